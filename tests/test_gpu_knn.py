"""The fused nearest-latent search (emb_knn): distances and the k nearest per query in one
pass, with no distance matrix. Its indices and expanded-form values must equal, bit for
bit, emb_distances followed by emb_topk_min (and the oracle's stable sort of those
distances); its direct-form distances must be within 1e-5 relative of the float64
direct form of the stored vectors, and exactly 0 for a query equal to a database row."""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu, say
from oracle import encoder as E

pytestmark = pytest.mark.gpu


def _dequant(L, rows=None):
    from paper_2205_04550_amd import binding as b
    codes = L.codes if rows is None else L.codes[rows]
    if L.fmt == b.EMB_BF16:
        return E.bf16_decode(codes.view(torch.int16).cpu().numpy())
    sc = (L.scale if rows is None else L.scale[rows]).cpu().numpy().astype(np.float64)
    return E.e4m3_decode(codes.cpu().numpy()) * sc[..., None]


def _check_equal(Q, X, k):
    from paper_2205_04550_amd import binding as b
    D = b.emb_distances(Q, X)
    i0, v0 = b.emb_topk_min(D, k)
    i1, v1 = b.emb_knn(Q, X, k, direct=False)
    torch.cuda.synchronize()
    assert torch.equal(i0, i1), k
    assert torch.equal(v0.view(torch.int32), v1.view(torch.int32)), k
    return D, i1


@pytest.mark.parametrize("fmt,M,N,dim,ks", [
    (0, 77, 1301, 512, (1, 10, 100, 256)),       # ragged M and N against the 128 x 256 tiles
    (1, 77, 1301, 512, (1, 10, 100, 256)),
    (0, 5, 3000, 48, (7, 100)),                  # K not a whole number of 32-value slices
    (0, 300, 50_021, 64, (1, 100)),              # many tiles per split, lists compacted
    (1, 9, 50_021, 64, (10, 256)),
    (0, 3, 150, 32, (1, 150)),                   # one partial tile: k = N
    (0, 5, 40_000, 48, (7, 100)),                # sampled bound, K with a partial slice
    (1, 130, 32_767, 64, (100,)),                # just below the sample size: own bounds
    (1, 130, 32_768, 64, (100, 256)),            # smallest database with the sampled bound
])
def test_knn_equals_distances_then_topk(fmt, M, N, dim, ks):
    need_gpu()
    from paper_2205_04550_amd import binding as b
    g = torch.Generator(device="cuda").manual_seed(41)
    base = torch.randn(701, dim, generator=g, device="cuda")
    Xf = base.repeat(N // 701 + 1, 1)[:N].contiguous()     # repeated rows: exact ties
    Qf = torch.randn(M, dim, generator=g, device="cuda")
    Qf[min(1, M - 1)] = base[3]
    Q, X = b.Latents(Qf, fmt), b.Latents(Xf, fmt)
    for k in ks:
        say(f"knn fmt {fmt} {M} x {N} x {dim} k = {k}")
        D, i1 = _check_equal(Q, X, k)
    want = E.topk_by_distance(D.cpu().numpy(), ks[-1])
    assert np.array_equal(i1.cpu().numpy(), want)


@pytest.mark.parametrize("fmt,N", [(0, 20_000), (1, 20_000), (0, 40_000), (1, 40_000)])
def test_knn_all_distances_equal(fmt, N):
    """Every database row identical: every distance of a query row ties, so each list's
    bound must fall back to the exact k-th entry; the lowest indices win. At 40,000 the
    sampled bound (the sample's k-th group minimum) admits every entry."""
    need_gpu()
    from paper_2205_04550_amd import binding as b
    g = torch.Generator(device="cuda").manual_seed(5)
    Xf = torch.randn(1, 64, generator=g, device="cuda").repeat(N, 1)
    Qf = torch.randn(6, 64, generator=g, device="cuda")
    Q, X = b.Latents(Qf, fmt), b.Latents(Xf, fmt)
    for k in (1, 100, 256):
        _, i1 = _check_equal(Q, X, k)
        assert np.array_equal(i1.cpu().numpy(), np.tile(np.arange(k), (6, 1)))


@pytest.mark.parametrize("fmt,N", [(0, 50_000), (1, 50_000), (1, 500_000)])
def test_knn_direct_form_distances(fmt, N):
    """direct = 1: each reported distance within 1e-5 of the float64 direct form of the
    stored vectors, and 0 exactly for the queries that are copies of database rows."""
    need_gpu()
    from paper_2205_04550_amd import binding as b
    g = torch.Generator(device="cuda").manual_seed(9)
    M, dim, k = 300, 512, 100
    Xf = torch.randn(N, dim, generator=g, device="cuda")
    Qf = torch.randn(M, dim, generator=g, device="cuda")
    self_rows = [0, 17, 299]
    Qf[self_rows] = Xf[[5, N // 2, N - 1]]
    Q, X = b.Latents(Qf, fmt), b.Latents(Xf, fmt)
    idx, d = b.emb_knn(Q, X, k, direct=True)
    i_exp, _ = b.emb_knn(Q, X, k, direct=False)
    torch.cuda.synchronize()
    assert torch.equal(idx, i_exp)
    q = _dequant(Q)
    idx_h = idx.cpu().numpy()
    x = _dequant(X, idx.view(-1).to(torch.int64)).reshape(M, k, dim)
    d64 = ((x - q[:, None, :]) ** 2).sum(axis=2)
    got = d.cpu().numpy().astype(np.float64)
    err = np.abs(got - d64)
    say(f"knn direct fmt {fmt} N {N}: max |d - d64| / d64 = {(err / np.maximum(d64, 1e-300)).max():.3g}")
    assert np.all(err <= 1e-5 * d64)
    for qi, xi in zip(self_rows, [5, N // 2, N - 1]):
        assert idx_h[qi, 0] == xi and got[qi, 0] == 0.0


@pytest.mark.parametrize("fmt,N", [(0, 50_000), (1, 500_000)])
def test_knn_workload_shapes(fmt, N):
    """The embedding workloads' shapes: 1,024 queries x 50,000 BF16 / 500,000 FP8 latents of
    dimension 512, top-100: the fused search equals distances + top-k bit for bit."""
    need_gpu()
    from paper_2205_04550_amd import binding as b
    g = torch.Generator(device="cuda").manual_seed(77)
    Xf = torch.randn(N, 512, generator=g, device="cuda")
    Qf = torch.randn(1024, 512, generator=g, device="cuda") * 0.5 + Xf[:1024] * 0.5
    Q, X = b.Latents(Qf, fmt), b.Latents(Xf, fmt)
    del Xf
    say(f"knn workload fmt {fmt}: 1024 x {N}")
    _check_equal(Q, X, 100)


@pytest.mark.parametrize("fmt,M,N,dim,ks", [
    (0, 1, 1, 16, (1,)), (1, 1, 256, 64, (1, 256)), (0, 32, 257, 16, (1, 200)),    # one tile and one row more
    (0, 33, 2_000, 512, (1, 256)), (1, 64, 3_333, 1024, (100,)),                   # 64-row tile, its widest rows
    (0, 65, 3_000, 64, (10,)), (1, 128, 33_000, 512, (256,)), (0, 100, 90_000, 16, (100,)),  # 128-row tile
    (0, 129, 3_000, 64, (10,)), (0, 33, 1_500, 1040, (10,)),                       # back to the tiled kernel
    (0, 32, 2_100, 2048, (256,)), (1, 31, 40_001, 1024, (1, 256)),                 # 32-row tile, its widest rows
    (0, 2, 32_769, 144, (256,)), (1, 64, 140_000, 64, (256,)), (0, 1, 70_000, 80, (1, 100)),
])
def test_knn_few_queries(fmt, M, N, dim, ks):
    """The kernel for up to 128 queries at the edges of its row tiles, its LDS (32 rows of 2,048
    values, 64 of 1,024, 128 of 512), chunks of loads with a rest and lists that are tightened, with and without
    the sampled bound, on rows with exact ties and an infinite and a NaN distance."""
    need_gpu()
    from paper_2205_04550_amd import binding as b
    g = torch.Generator(device="cuda").manual_seed(M + N + dim)
    base = torch.randn(min(N, 997), dim, generator=g, device="cuda")
    Xf = base.repeat(N // len(base) + 1, 1)[:N].contiguous()
    Qf = torch.randn(M, dim, generator=g, device="cuda")
    Q, X = b.Latents(Qf, fmt), b.Latents(Xf, fmt)
    if N > 300:
        X.sq[299], X.sq[123] = float("inf"), float("nan")
    for k in ks:
        say(f"knn few queries fmt {fmt} {M} x {N} x {dim} k = {k}")
        _check_equal(Q, X, k)


@pytest.mark.parametrize("fmt,M", [(0, 5), (0, 40), (0, 70), (1, 5)])
@pytest.mark.parametrize("N", [5000, 40_000])
def test_knn_of_few_queries_leaves_nans_out(fmt, M, N):
    """Queries and entries with infinities and NaNs: the nearest by the distances that are numbers,
    infinite ones too, below and above the size of the sampled bound."""
    need_gpu()
    from paper_2205_04550_amd import binding as b
    g = torch.Generator(device="cuda").manual_seed(43)
    Xf, Qf = (torch.randn(n, 64, generator=g, device="cuda") for n in (N, M))
    if fmt == 0:
        Qf[3, 1] = float("inf")                    # half the distances infinite, half NaN
    Qf[4, 2] = float("nan")
    Xf[7::9, 5] = float("nan")
    Q, X = b.Latents(Qf, fmt), b.Latents(Xf, fmt)
    k = 6
    say(f"knn with special values fmt {fmt} {M} x {N}")
    D = b.emb_distances(Q, X).cpu()
    idx, d = b.emb_knn(Q, X, k, direct=False)
    idx, d = idx.cpu(), d.cpu()
    for q in range(M):
        ok = torch.nonzero(~torch.isnan(D[q]))[:, 0]
        order = ok[torch.sort(D[q][ok], stable=True).indices][:k]
        if len(order) < k:
            assert len(order) == 0 and (idx[q] == -1).all()
            continue
        assert torch.equal(idx[q].long(), order), q
        assert torch.equal(d[q], D[q][order]), q


@pytest.mark.parametrize("M,N,k", [(40, 300, 100), (41, 1967, 20), (41, 1968, 20), (64, 3071, 128), (64, 3072, 128),
                                   (80, 7680, 64), (81, 7776, 64), (81, 7776, 100), (128, 12_288, 100), (4, 767, 256),
                                   (4, 768, 129), (100, 19_200, 200)])
def test_knn_either_side_of_the_small_database_rule(M, N, k):
    """Databases below the sampled size, where M, N and k decide between the kernel of few queries
    and the tiled one: equal to the distances' smallest on both sides."""
    need_gpu()
    from paper_2205_04550_amd import binding as b
    g = torch.Generator(device="cuda").manual_seed(47)
    Xf = torch.randn(N, 64, generator=g, device="cuda")
    Xf[N // 2:] = Xf[:N - N // 2].clone()                   # ties
    Qf = torch.randn(M, 64, generator=g, device="cuda")
    for fmt in (0, 1):
        say(f"knn rule fmt {fmt} {M} x {N} k = {k}")
        _check_equal(b.Latents(Qf, fmt), b.Latents(Xf, fmt), k)


@pytest.mark.parametrize("M,N,k", [(128, 2000, 256), (64, 600, 200), (128, 2000, 100)])
def test_knn_of_few_queries_takes_no_longer_than_of_more(M, N, k):
    """A search of up to 128 queries takes at most one and a half times as long as of 192."""
    need_gpu()
    from paper_2205_04550_amd import binding as b
    g = torch.Generator(device="cuda").manual_seed(48)
    X = b.Latents(torch.randn(N, 64, generator=g, device="cuda"), 0)
    best = {}
    for m in (M, 192):
        Q = b.Latents(torch.randn(m, 64, generator=g, device="cuda"), 0)
        ws = b.knn_workspace(m, N, k)
        times = []
        for _ in range(6):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(5):
                b.emb_knn(Q, X, k, direct=False, ws=ws)
            e1.record()
            e1.synchronize()
            times.append(e0.elapsed_time(e1))
        best[m] = min(times[1:])
    assert best[M] < 1.5 * best[192], best
