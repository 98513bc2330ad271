"""Timed cases of the retrieval library: what a program that uses it does, call by call.

Inputs are made on the GPU from a seed: tumour densities (logistic fronts inside an
ellipsoidal brain, the shapes and radii of the synthetic database), patient labels (a
simulation thresholded at both levels, 2 % of each mask's boundary voxels flipped), boxes
around the tumours, latents, encoder weights.

Kinds of cases:
  query    one patient against every entry (TumorDB.query)
  row_box  the same query over the rows both sides fill (TumorDB.query_sparse)
  batch    many patients, each inside a box of its own (TumorDB.query_batch)
  build    densities thresholded and packed into a new database (TumorDB.append)
  embed    labels -> packing, encoder, latent search, exact rerank: the top k
  encode   database entries -> latents (the database side of the latent search)
  knn      query latents quantised, then the nearest database latents (emb_knn)
  com      nearest centres of mass, then the exact rerank (TumorDB.query_com)
  train    one step of the autoencoder: forward, backward, Adam
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2205_04550_amd import nn
from paper_2205_04550_amd.binding import (EMB_BF16, EMB_FP8, LIB, Latents, TumorDB, emb_knn,
                                          knn_workspace)

T_LO, T_HI = 0.25, 0.675      # FLAIR / T1Gd levels
FLIP = 0.02                   # share of a mask's boundary voxels that a query has flipped
CHANNELS = (2, 8, 16, 32, 64)
LATENT = 512
VAE_BETA = 1e-5
FMT = {"bf16": EMB_BF16, "fp8": EMB_FP8}


def listed():
    return [
        # A small study: one patient against 1,000 simulations of 64^3. Launches and latency.
        dict(name="query_1k_64cube", kind="query", n=1000, nx=64, ny=64, nz=64, k=10),
        # The exhaustive search of the paper's database size, one patient.
        dict(name="query_50k_128cube", kind="query", n=50000, nx=128, ny=128, nz=128, k=10),
        # The same answer from the rows that both sides fill.
        dict(name="row_box_50k_128cube", kind="row_box", n=50000, nx=128, ny=128, nz=128, k=10),
        # A cohort, every patient with a region of interest, one call.
        dict(name="batch_256q_50k_128cube", kind="batch", n=50000, nx=128, ny=128, nz=128, nq=256,
             k=10),
        # One chunk of a database build.
        dict(name="build_2k_128cube", kind="build", n=2048, nx=128, ny=128, nz=128),
        # A cohort through the embedding search, top 15 after the exact rerank of 100.
        dict(name="embed_1024q_50k", kind="embed", n=50000, nq=1024, n_cand=100, k=15, fmt="bf16"),
        # One patient through the embedding search: a chain of small launches.
        dict(name="embed_1q_50k", kind="embed", n=50000, nq=1, n_cand=100, k=15, fmt="bf16"),
        # One chunk of a database being encoded.
        dict(name="encode_2k_entries", kind="encode", n=4096, batch=2048),
        # The latent search alone, over half a million FP8 latents.
        dict(name="knn_1024q_500k_fp8", kind="knn", n=500000, nq=1024, dim=512, k=100, fmt="fp8"),
        # The centre-of-mass prefilter on an uneven grid and count, 1,000 candidates.
        dict(name="com_200q_20011_96x112x77", kind="com", n=20011, nx=96, ny=112, nz=77, nq=200,
             n_cand=1000, k=15),
        # A training step at the usual batch.
        dict(name="train_32x64cube", kind="train", batch=32, grid=64, masks=2, latent=512,
             vae=False),
        # A training step of the single-mask variational encoder, small uneven batch and grid.
        dict(name="train_vae_7x48cube", kind="train", batch=7, grid=48, masks=1, latent=256,
             vae=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng):
    return dict(nx=rng.choice((32, 64, 96, 128)), ny=rng.randint(24, 128), nz=rng.randint(24, 128))


def draw(rng):
    kind = rng.choice(("query", "row_box", "batch", "build", "embed", "encode", "knn", "com",
                       "train"))
    if kind in ("query", "row_box"):
        return dict(kind=kind, n=_log(rng, 500, 50000), **_grid(rng), k=_log(rng, 1, 100))
    if kind == "batch":
        return dict(kind=kind, n=_log(rng, 500, 20000), **_grid(rng), nq=_log(rng, 2, 256),
                    k=_log(rng, 1, 50))
    if kind == "build":
        return dict(kind=kind, n=_log(rng, 64, 2048), **_grid(rng))
    if kind == "embed":
        n_cand = _log(rng, 20, 256)
        return dict(kind=kind, n=_log(rng, 2000, 50000), nq=_log(rng, 1, 1024), n_cand=n_cand,
                    k=min(n_cand, _log(rng, 1, 32)), fmt=rng.choice(("bf16", "fp8")))
    if kind == "encode":
        return dict(kind=kind, n=_log(rng, 1024, 4096), batch=_log(rng, 8, 2048))
    if kind == "knn":
        n = _log(rng, 1000, 500000)
        return dict(kind=kind, n=n, nq=_log(rng, 1, 1024), dim=rng.choice((64, 128, 256, 512, 1024)),
                    k=_log(rng, 1, 200), fmt=rng.choice(("bf16", "fp8")))
    if kind == "com":
        n_cand = _log(rng, 16, 1000)
        return dict(kind=kind, n=_log(rng, 1000, 20000), **_grid(rng), nq=_log(rng, 1, 400),
                    n_cand=n_cand, k=min(n_cand, _log(rng, 1, 50)))
    grid = rng.choice((16, 32, 48, 64))
    return dict(kind="train", batch=min(rng.randint(1, 96), 32 * 64 ** 3 // grid ** 3), grid=grid,
                masks=rng.choice((1, 2)), latent=rng.choice((64, 128, 256, 512)),
                vae=rng.random() < 0.5)


# ---- inputs -----------------------------------------------------------------------------------

def _params(seed: int, stream: int, n: int, dims) -> torch.Tensor:
    """[n][8] float32 on the GPU: centre, reciprocal anisotropy, radius, reciprocal width."""
    u = torch.from_numpy(np.random.RandomState((1000003 * seed + stream) % 2 ** 32).rand(n, 8))
    d = torch.tensor(dims, dtype=torch.float64)
    semi = torch.tensor((0.40, 0.46, 0.36), dtype=torch.float64) * d
    cos, phi = 2 * u[:, 6:7] - 1, 2 * math.pi * u[:, 7:8]
    sin = (1 - cos * cos).sqrt()
    way = torch.cat((sin * phi.cos(), sin * phi.sin(), cos), 1)
    p = torch.empty((n, 8), dtype=torch.float64)
    p[:, 0:3] = (d - 1) / 2 + way * semi * u[:, 0:1] ** (1 / 3)
    p[:, 3:6] = 1 / (0.7 + 0.6 * u[:, 1:4])
    m = min(dims)
    p[:, 6] = m / 16 + u[:, 4] * (m / 4)
    p[:, 7] = 1 / (m / 128 + u[:, 5] * (7 * m / 128))
    return p.float().cuda()


def _volumes(p: torch.Tensor, dims) -> torch.Tensor:
    """Densities float32 [n][nz][ny][nx]."""
    nx, ny, nz = dims
    ax = [torch.arange(s, device="cuda", dtype=torch.float32) for s in dims]
    semi = (0.40 * nx, 0.46 * ny, 0.36 * nz)
    bx, by, bz = [((a - (s - 1) / 2) / h) ** 2 for a, s, h in zip(ax, dims, semi)]
    brain = (bx[None, None, :] + by[None, :, None] + bz[:, None, None] <= 1).float()
    dx, dy, dz = [((ax[i][None, :] - p[:, i:i + 1]) * p[:, 3 + i:4 + i]) ** 2 for i in range(3)]
    c = (dx[:, None, None, :] + dy[:, None, :, None]) + dz[:, :, None, None]
    c = c.sqrt_().sub_(p[:, 6, None, None, None]).mul_(-p[:, 7, None, None, None])
    return c.sigmoid_().mul_(brain)


def _chunks(seed: int, stream: int, n: int, dims):
    p = _params(seed, stream, n, dims)
    step = max(1, min(512, (1 << 30) // (dims[0] * dims[1] * dims[2])))
    for s in range(0, n, step):
        yield s, _volumes(p[s:s + step], dims)


def _flip(mask: torch.Tensor, g) -> torch.Tensor:
    """mask with 2 % of its boundary voxels (a 6-neighbour of the other value) flipped."""
    b = torch.zeros_like(mask)
    for a in (1, 2, 3):
        n = mask.shape[a]
        d = mask.narrow(a, 1, n - 1) != mask.narrow(a, 0, n - 1)
        b.narrow(a, 1, n - 1).logical_or_(d)
        b.narrow(a, 0, n - 1).logical_or_(d)
    return mask ^ (b & (torch.rand(mask.shape, generator=g, device="cuda") < FLIP))


def _labels(seed: int, stream: int, nq: int, dims, of_db: bool = False) -> torch.Tensor:
    """uint8 [nq][nz][ny][nx]: held-out simulations, or (of_db) the database's first entries."""
    nx, ny, nz = dims
    g = torch.Generator(device="cuda").manual_seed(1000003 * seed + stream + 17)
    out = torch.empty((nq, nz, ny, nx), dtype=torch.uint8, device="cuda")
    p = _params(seed, 1 if of_db else stream, nq, dims)
    for s in range(0, nq, 64):
        c = _volumes(p[s:s + 64], dims)
        out[s:s + 64] = _flip(c >= T_LO, g).to(torch.uint8) | (_flip(c >= T_HI, g).to(torch.uint8) << 1)
    return out


def _rois(seed: int, labels: torch.Tensor) -> np.ndarray:
    """int32 [nq][6]: sides uniform in 24 .. the axis, centred on the FLAIR box, inside the grid."""
    r = np.random.RandomState(seed + 4552)
    fl = (labels & 1) != 0
    out = np.zeros((labels.shape[0], 6), dtype=np.int32)
    for i, (axis, others) in enumerate(((3, (1, 2)), (2, (1, 3)), (1, (2, 3)))):
        has = fl.any(dim=others[1]).any(dim=others[0]).cpu().numpy()
        n = has.shape[1]
        lo = np.where(has.any(1), has.argmax(1), 0)
        hi = np.where(has.any(1), n - has[:, ::-1].argmax(1), n)
        side = r.randint(min(24, n), n + 1, size=len(out))
        start = np.clip((lo + hi - side) // 2, 0, n - side)
        out[:, i], out[:, i + 3] = start, start + side
    return out


def _dims(case):
    return (case["nx"], case["ny"], case["nz"]) if "nx" in case else (128, 128, 128)


def _database(case, seed):
    dims = _dims(case)
    db = TumorDB(*dims, case["n"], T_LO, T_HI)
    for _, c in _chunks(seed, 1, case["n"], dims):
        db.append(c)
    return db


def _weights(shapes: dict, seed: int) -> dict:
    """He-uniform weights and small biases, float32 on the GPU, by parameter name."""
    g = torch.Generator().manual_seed(1000003 * seed + 5)
    out = {}
    for name in sorted(shapes):
        s = shapes[name]
        if name.endswith(".b"):
            w = (torch.rand(s, generator=g) * 2 - 1) * 0.02
        else:
            # Fan-in of a transposed convolution ([Cin][Cout][3][3][3]): Cin 27 / 8 taps.
            fan = (s[0] * 27 / 8 if name.startswith("dec") and len(s) == 5
                   else math.prod(s[1:]))
            w = (torch.rand(s, generator=g) * 2 - 1) * math.sqrt(6.0 / fan)
        out[name] = w.cuda()
    return out


def _shapes(grid, masks, latent, vae):
    ch = (masks,) + CHANNELS[1:]
    flat = ch[4] * (grid // 16) ** 3
    s = {}
    for i in range(4):
        s[f"enc{i}.w"], s[f"enc{i}.b"] = (ch[i + 1], ch[i], 3, 3, 3), (ch[i + 1],)
        s[f"dec{i}.w"], s[f"dec{i}.b"] = (ch[i + 1], ch[i], 3, 3, 3), (ch[i],)
    heads = 2 if vae else 1
    s["enc_fc.w"], s["enc_fc.b"] = (heads * latent, flat), (heads * latent,)
    s["dec_fc.w"], s["dec_fc.b"] = (flat, latent), (flat,)
    return s


def _model(seed, grid=64, masks=2, latent=LATENT, vae=False):
    model = nn.AutoEncoder(grid=grid, channels=(masks,) + CHANNELS[1:], latent=latent,
                           vae_beta=VAE_BETA if vae else None)
    w = _weights(_shapes(grid, masks, latent, vae), seed)
    with torch.no_grad():
        for name, p in model.params.items():
            p.copy_(w[name])
    model.refresh_working_weights()
    return model


def _pooled(seed, batch, grid, masks):
    """The masks of `batch` simulations of (2 grid)^3, mean-pooled by 2: [B][masks][grid^3]."""
    out = torch.empty((batch, masks, grid, grid, grid), device="cuda")
    for s, c in _chunks(seed, 3, batch, (2 * grid,) * 3):
        for m, t in enumerate((T_LO, T_HI)[:masks]):
            b = (c >= t).float().view(-1, grid, 2, grid, 2, grid, 2)
            out[s:s + len(c), m] = b.mean(dim=(2, 4, 6))
    return out


def _latents(seed, stream, n, dim):
    """Latents of a smooth map of the eight parameters of a tumour, float32 [n][dim]."""
    g = torch.Generator().manual_seed(1000003 * seed + 7)
    w1, w2 = torch.randn((8, 256), generator=g), torch.randn((256, dim), generator=g)
    g = torch.Generator().manual_seed(1000003 * seed + 7 + stream)
    h = torch.randn((n, 8), generator=g) @ w1 * 0.5
    return (torch.relu(h) @ w2 * 0.1 + 0.02 * torch.randn((n, dim), generator=g)).cuda()


def prepare(case, seed):
    kind, s = case["kind"], {"kind": case["kind"]}
    if kind in ("query", "row_box", "batch", "com"):
        s["db"] = db = _database(case, seed)
        s["k"] = case["k"]
        if kind == "batch":
            s["labels"] = _labels(seed, 1, case["nq"], _dims(case), of_db=True)
            s["rois"] = _rois(seed, s["labels"])
            s["ws"] = db.workspace(case["nq"], case["k"])
        elif kind == "com":
            s["labels"] = _labels(seed, 2, case["nq"], _dims(case))
            s["n_cand"] = case["n_cand"]
            s["ws"] = torch.empty(LIB.db_query_com_workspace_bytes(db._h, case["nq"], case["n_cand"]),
                                  dtype=torch.uint8, device="cuda")
        else:
            s["labels"] = _labels(seed, 1, 1, _dims(case), of_db=True)
            s["ws"] = db.workspace(1, case["k"])
    elif kind == "build":
        dims = _dims(case)
        s["dims"] = dims
        s["conc"] = torch.empty((case["n"], dims[2], dims[1], dims[0]), device="cuda")
        for at, c in _chunks(seed, 1, case["n"], dims):
            s["conc"][at:at + len(c)] = c
    elif kind == "embed":
        s["db"] = db = _database(case, seed)
        s["model"] = model = _model(seed)
        lat = [model.encode_planes_bf16(db.planes, db.dims, i.to(torch.int32))
               for i in torch.arange(case["n"], device="cuda").split(1024)]
        s["fmt"], s["k"], s["n_cand"] = FMT[case["fmt"]], case["k"], case["n_cand"]
        s["x"] = Latents(torch.cat(lat), s["fmt"])
        s["labels"] = _labels(seed, 2, case["nq"], db.dims)
        s["ws"] = db.rerank_workspace(case["nq"])
        s["knn_ws"] = knn_workspace(case["nq"], case["n"], case["n_cand"])
    elif kind == "encode":
        s["db"] = _database(case, seed)
        s["model"] = _model(seed)
        s["idx"] = _picked(case, seed)
    elif kind == "knn":
        s["q"] = _latents(seed, 2, case["nq"], case["dim"])
        s["fmt"], s["k"] = FMT[case["fmt"]], case["k"]
        s["x"] = Latents(_latents(seed, 1, case["n"], case["dim"]), s["fmt"])
        s["ws"] = knn_workspace(case["nq"], case["n"], case["k"])
    else:
        s["model"] = _model(seed, case["grid"], case["masks"], case["latent"], case["vae"])
        s["opt"] = nn.Adam(s["model"], lr=1e-3)
        s["x"] = _pooled(seed, case["batch"], case["grid"], case["masks"])
        s["eps"] = _eps(case, seed)
    return s


def _picked(case, seed):
    g = torch.Generator().manual_seed(1000003 * seed + 9)
    return torch.randint(case["n"], (case["batch"],), generator=g).to(torch.int32).cuda()


def _eps(case, seed):
    if not case["vae"]:
        return None
    g = torch.Generator().manual_seed(1000003 * seed + 11)
    return torch.randn((case["batch"], case["latent"]), generator=g).cuda()


# ---- one pass ---------------------------------------------------------------------------------

def run(s):
    kind = s["kind"]
    if kind == "query":
        return s["db"].query(s["labels"][0], s["k"], ws=s["ws"])
    if kind == "row_box":
        return s["db"].query_sparse(s["labels"][0], s["k"], ws=s["ws"])
    if kind == "batch":
        return s["db"].query_batch(s["labels"], s["rois"], s["k"], ws=s["ws"])
    if kind == "com":
        return s["db"].query_com(s["labels"], s["n_cand"], s["k"], ws=s["ws"])
    if kind == "build":
        db = TumorDB(*s["dims"], s["conc"].shape[0], T_LO, T_HI)
        db.append(s["conc"])
        return (db.planes, db.popcounts, db.boxes, db.tboxes, db.zranges, db.block_counts,
                db.moments)
    if kind == "embed":
        pooled = s["db"].rerank_pack_pool(s["labels"], s["ws"])
        lat = s["model"].encode_counts_bf16(pooled)
        cand, _ = emb_knn(Latents(lat, s["fmt"]), s["x"], s["n_cand"], ws=s["knn_ws"])
        return lat, s["db"].rerank_packed(s["ws"], cand, s["k"])
    if kind == "encode":
        return s["model"].encode_planes_bf16(s["db"].planes, s["db"].dims, s["idx"])
    if kind == "knn":
        return emb_knn(Latents(s["q"], s["fmt"]), s["x"], s["k"], ws=s["ws"])
    model = s["model"]
    loss = model.loss(s["x"], s["eps"])
    loss.backward()
    grads = {k: p.grad for k, p in model.params.items()}
    s["opt"].step()
    return loss.detach(), grads


# ---- the work of one pass ---------------------------------------------------------------------

def _macs(grid, masks, latent, vae):
    """(encoder, decoder) multiply-adds of one sample."""
    ch, e = (masks,) + CHANNELS[1:], 0
    for i in range(4):
        e += 27 * ch[i] * ch[i + 1] * (grid >> (i + 1)) ** 3
    fc = ch[4] * (grid // 16) ** 3 * latent
    return e + (2 if vae else 1) * fc, e + fc


def work(case):
    kind = case["kind"]
    if kind == "train":
        e, d = _macs(case["grid"], case["masks"], case["latent"], case["vae"])
        acts = sum(c * (case["grid"] >> i) ** 3
                   for i, c in enumerate((case["masks"],) + CHANNELS[1:]))
        par = sum(math.prod(v) for v in _shapes(case["grid"], case["masks"], case["latent"],
                                                case["vae"]).values())
        # Every activation of both halves written and read again by the backward; weights,
        # gradients and both moments.
        return {"bytes": 16.0 * acts * case["batch"] + 30.0 * par,
                "flops": 6.0 * case["batch"] * (e + d)}
    if kind == "knn":
        b = 2 if case["fmt"] == "bf16" else 1
        return {"bytes": b * case["dim"] * (case["n"] + case["nq"]) + 8 * case["nq"] * case["k"],
                "flops": 2.0 * case["nq"] * case["n"] * case["dim"]}
    nx, ny, nz = _dims(case)
    V = nx * ny * nz
    planes = case["n"] * V / 4
    if kind == "query":
        return {"bytes": planes + V, "flops": 0}
    if kind == "row_box":   # about 3 % of a database's bytes lie in rows that both sides fill
        return {"bytes": 0.03 * planes + V, "flops": 0}
    if kind == "batch":
        # An AND and two counts per packed word pair, over about a tenth of the grid's words.
        return {"bytes": planes + case["nq"] * V, "flops": 0.1 * 3 * case["nq"] * planes / 4}
    if kind == "build":
        return {"bytes": case["n"] * V * 4 + planes, "flops": 0}
    if kind == "com":
        # Labels, moments, the candidates' rows inside the query's box (about a tenth).
        return {"bytes": case["nq"] * V + 32 * case["n"] + 0.1 * case["nq"] * case["n_cand"] * V / 4,
                "flops": 0}
    enc = _macs(64, 2, LATENT, False)[0]
    if kind == "encode":
        return {"bytes": case["batch"] * (V / 4 + 4 * LATENT), "flops": 2.0 * case["batch"] * enc}
    b = 2 if case["fmt"] == "bf16" else 1
    return {"bytes": case["nq"] * V + b * LATENT * case["n"] +
            0.03 * case["nq"] * case["n_cand"] * V / 4,
            "flops": 2.0 * case["nq"] * (enc + case["n"] * LATENT)}


# ---- the same in 64 bits ----------------------------------------------------------------------

def _dice_sum(inter, a, b):
    """float64 sum over masks of 2 I / (A + B), 1 where both are empty; last axis = mask."""
    s = a + b
    d = torch.where(s > 0, 2 * inter / s.clamp(min=1), torch.ones_like(inter))
    return d[..., 1] + d[..., 0]


def _scores(case, seed, labels, rois=None):
    """float64 [nq][n] scores and, per side, (moments, count) of the FLAIR masks."""
    dims = _dims(case)
    nx, ny, nz = dims
    nq, V = labels.shape[0], nx * ny * nz
    R = torch.ones((nq, nz, ny, nx), dtype=torch.bool, device="cuda")
    if rois is not None:
        R.zero_()
        for q, (x0, y0, z0, x1, y1, z1) in enumerate(rois.tolist()):
            R[q, z0:z1, y0:y1, x0:x1] = True
    slab = lambda m: m.reshape(m.shape[0], nz, -1).transpose(0, 1).double().contiguous()  # noqa: E731
    Q = [slab(((labels >> m) & 1).bool() & R) for m in (0, 1)]
    box = slab(R) if rois is not None else None
    a = torch.stack([q.sum(dim=(0, 2)) for q in Q], -1)
    out = torch.empty((nq, case["n"]), dtype=torch.float64, device="cuda")
    mom = torch.empty((case["n"], 4), dtype=torch.float64, device="cuda")
    for s, c in _chunks(seed, 1, case["n"], dims):
        for t in range(0, len(c), 128):
            B = [slab(c[t:t + 128] >= v) for v in (T_LO, T_HI)]
            to = slice(s + t, s + t + B[0].shape[1])
            # [nz][entries][ny nx] x [nz][ny nx][nq]
            dot = lambda q, b: torch.stack([b[z] @ q[z].T for z in range(nz)]).sum(0).T  # noqa: E731
            inter = torch.stack([dot(q, b) for q, b in zip(Q, B)], -1)
            if box is None:
                cnt = torch.stack([b.sum(dim=(0, 2)) for b in B], -1)[None].expand_as(inter)
            else:
                cnt = torch.stack([dot(box, b) for b in B], -1)
            out[:, to] = _dice_sum(inter, a[:, None, :].expand_as(inter), cnt)
            mom[to] = _moments(B[0], ny, nx)
    return out, mom, _moments(Q[0], ny, nx)


def _moments(m, ny, nx):
    """[samples][4]: sum of x, y, z and the count, from slabs [nz][samples][ny nx]."""
    m = m.view(m.shape[0], m.shape[1], ny, nx)
    ar = lambda n: torch.arange(n, device="cuda", dtype=torch.float64)  # noqa: E731
    return torch.stack([m.sum(dim=(0, 2)) @ ar(nx), m.sum(dim=(0, 3)) @ ar(ny),
                        ar(m.shape[0]) @ m.sum(dim=(2, 3)), m.sum(dim=(0, 2, 3))], -1)


def _taps(x):
    """[B][C][D][H][W] -> [B][D/2][H/2][W/2][27 C] of a stride-2 window of 3 with padding 1."""
    B, C, D, H, W = x.shape
    p = torch.nn.functional.pad(x, (1, 1, 1, 1, 1, 1))
    t = [p[:, :, a:a + D:2, b:b + H:2, c:c + W:2] for a in range(3) for b in range(3)
         for c in range(3)]
    return torch.stack(t, 2).permute(0, 3, 4, 5, 1, 2).reshape(B, D // 2, H // 2, W // 2, 27 * C)


def _conv(x, w, b):
    y = _taps(x) @ w.reshape(w.shape[0], -1).T + b
    return y.permute(0, 4, 1, 2, 3)


def _conv_t(x, w, b):
    """conv_transpose3d(stride 2, padding 1, output_padding 1): each output parity from its taps."""
    B, C, D, H, W = x.shape
    cols = (x.permute(0, 2, 3, 4, 1).reshape(-1, C) @ w.reshape(C, -1)).view(B, D, H, W, -1, 3, 3, 3)
    out = x.new_zeros((B, w.shape[1], 2 * D + 1, 2 * H + 1, 2 * W + 1))
    for a in range(3):
        for e in range(3):
            for f in range(3):
                out[:, :, a:a + 2 * D:2, e:e + 2 * H:2, f:f + 2 * W:2] += \
                    cols[..., a, e, f].permute(0, 4, 1, 2, 3)
    return out[:, :, 1:, 1:, 1:] + b[None, :, None, None, None]


def _exact_train(case, seed):
    w = _weights(_shapes(case["grid"], case["masks"], case["latent"], case["vae"]), seed)
    # The weights of every layer are used in bfloat16, the biases as they are.
    w = {k: (v.bfloat16() if k.endswith(".w") else v).double().requires_grad_() for k, v in w.items()}
    x = _pooled(seed, case["batch"], case["grid"], case["masks"]).double()
    h = x
    for i in range(4):
        h = torch.relu(_conv(h, w[f"enc{i}.w"], w[f"enc{i}.b"]))
    z = h.reshape(h.shape[0], -1) @ w["enc_fc.w"].T + w["enc_fc.b"]
    more = 0.0
    if case["vae"]:
        mu, lv = z.chunk(2, dim=1)
        more = VAE_BETA * 0.5 * (mu * mu + lv.exp() - 1 - lv).sum(1).mean()
        z = mu + (lv / 2).exp() * _eps(case, seed).double()
    h = torch.relu(z @ w["dec_fc.w"].T + w["dec_fc.b"])
    g = case["grid"] // 16
    h = h.reshape(h.shape[0], CHANNELS[4], g, g, g)
    for i in reversed(range(4)):
        h = _conv_t(h, w[f"dec{i}.w"], w[f"dec{i}.b"])
        h = torch.relu(h) if i else h
    loss = ((h - x) ** 2).mean()
    (loss + more).backward()
    return loss.detach(), {k: v.grad for k, v in w.items()}


def _exact_encode(pooled, seed):
    """Latents of pooled masks [B][2][64^3]: layers 1 to 3 rounded to bfloat16, the rest not."""
    w = _weights(_shapes(64, 2, LATENT, False), seed)
    out = []
    for h in pooled.split(64):
        h = h.double()
        for i in range(4):
            h = torch.relu(_conv(h, w[f"enc{i}.w"].bfloat16().double(), w[f"enc{i}.b"].double()))
            h = h if i == 3 else h.float().bfloat16().double()
        out.append(h.reshape(len(h), -1) @ w["enc_fc.w"].bfloat16().double().T +
                   w["enc_fc.b"].double())
    return torch.cat(out)


def _pool_masks(f, t):
    B, n = f.shape[0], f.shape[1] // 2
    return torch.stack([m.float().view(B, n, 2, n, 2, n, 2).mean(dim=(2, 4, 6)) for m in (f, t)], 1)


def _stored(lat, fmt):
    if fmt == "bf16":
        return lat.bfloat16().double()
    s = lat.abs().amax(dim=1, keepdim=True) / 448
    s = torch.where(s > 0, s, torch.ones_like(s))
    return (lat / s).to(torch.float8_e4m3fn).double() * s.double()


def exact(case, seed):
    kind = case["kind"]
    if kind == "build":
        return None
    if kind in ("query", "row_box"):
        sc = _scores(case, seed, _labels(seed, 1, 1, _dims(case), of_db=True))[0][0]
        return None, sc.sort(descending=True, stable=True).values[:case["k"]], None
    if kind == "batch":
        if case["nq"] * case["n"] * math.prod(_dims(case)) > 6e12:
            return None
        labels = _labels(seed, 1, case["nq"], _dims(case), of_db=True)
        sc = _scores(case, seed, labels, _rois(seed, labels))[0]
        return None, sc.sort(dim=1, descending=True, stable=True).values[:, :case["k"]], None
    if kind == "com":
        sc, mx, mq = _scores(case, seed, _labels(seed, 2, case["nq"], _dims(case)))
        cx, cq = mx[:, :3] / mx[:, 3:], mq[:, :3] / mq[:, 3:]
        key = ((cq[:, None] - cx[None]) ** 2).sum(-1)
        key = torch.where((mq[:, None, 3] > 0) & (mx[None, :, 3] > 0), key,
                          torch.full_like(key, math.inf))
        d, i = key.float().sort(dim=1, stable=True)
        d, i = key.gather(1, i[:, :case["n_cand"]]), i[:, :case["n_cand"]]
        top = sc.gather(1, i).sort(dim=1, descending=True).values[:, :case["k"]]
        return None, top, None, None, d
    if kind == "knn":
        q = _stored(_latents(seed, 2, case["nq"], case["dim"]), case["fmt"])
        x = _stored(_latents(seed, 1, case["n"], case["dim"]), case["fmt"])
        xs, out = (x * x).sum(1), []
        for s in range(0, len(q), 64):
            D = (q[s:s + 64] ** 2).sum(1, keepdim=True) + xs - 2 * (q[s:s + 64] @ x.T)
            i = D.topk(case["k"], dim=1, largest=False).indices
            d = torch.stack([((q[s + r] - x[i[r]]) ** 2).sum(1) for r in range(len(i))])
            out.append(d.sort(dim=1).values)
        return None, torch.cat(out)
    if kind == "embed":
        lab = _labels(seed, 2, case["nq"], _dims(case))
        lat = [_exact_encode(_pool_masks(b & 1, b >> 1), seed) for b in lab.split(64)]
        return torch.cat(lat), None
    if kind == "encode":
        p = _params(seed, 1, case["n"], _dims(case))[_picked(case, seed).long()]
        lat = []
        for s in range(0, len(p), 64):
            c = _volumes(p[s:s + 64], _dims(case))
            lat.append(_exact_encode(_pool_masks(c >= T_LO, c >= T_HI), seed))
        return torch.cat(lat)
    return _exact_train(case, seed)
