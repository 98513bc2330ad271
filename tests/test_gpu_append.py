"""Everything db_append stores of an entry, in its one pass, against numpy on the thresholded
volumes: grids whose words do not fill a wave's group or a row a word pair, plane padding, one
slice, and the pass that deeper grids take."""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu, unpack_planes

pytestmark = pytest.mark.gpu


def _range(any_y):
    """y0 | y1 << 16 of the set rows, per slice."""
    out = np.zeros(any_y.shape[:-1], dtype=np.int64)
    has = any_y.any(-1)
    lo, hi = any_y.argmax(-1), any_y.shape[-1] - any_y[..., ::-1].argmax(-1)
    out[has] = (lo | (hi << 16))[has]
    return out


def _box(rows):
    z, y = np.nonzero(rows)
    return [z.min(), z.max() + 1, y.min(), y.max() + 1] if len(z) else [0, 0, 0, 0]


@pytest.mark.parametrize("dims,n,t_lo", [((128, 17, 9), 3, 0.25), ((32, 3, 1), 5, 0.25), ((96, 5, 7), 4, -1.0),
                                         ((64, 33, 20), 1100, 0.25), ((32, 2, 600), 2, 0.25),
                                         ((160, 21, 18), 2, 0.25), ((256, 256, 130), 1, 0.25)])
def test_append_one_pass(dims, n, t_lo):
    need_gpu()
    from paper_2205_04550_amd import TumorDB
    nx, ny, nz = dims
    rng = np.random.default_rng(nx + ny + nz)
    c = np.zeros((n, nz, ny, nx), dtype=np.float32)
    for e in range(n):                       # a box of random densities, some entries empty
        if e % 5 == 4:
            continue
        a = [sorted(rng.integers(0, d + 1, 2)) for d in (nz, ny, nx)]
        sl = tuple(slice(lo, hi) for lo, hi in a)
        c[e][sl] = rng.random(c[e][sl].shape, dtype=np.float32)
    c[0].ravel()[-1] = 1.0                   # the last voxel of the first entry
    c[0].ravel()[0] = np.nan
    db = TumorDB(nx, ny, nz, n + 1, t_lo, 0.675)
    half = n // 2                            # two calls: the second starts past the first
    for part in (c[:half], c[half:]):
        if len(part):
            db.append(torch.from_numpy(part).cuda())
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore"):
        m = np.stack([c >= t_lo, c >= 0.675], 1)             # [n][2][nz][ny][nx]
    V = nx * ny * nz
    got = unpack_planes(db.planes[:n].cpu().numpy(), V).reshape(m.shape)
    assert np.array_equal(got, m)
    assert not db.planes[:n, :, V // 32:].any()              # padding words
    assert np.array_equal(db.popcounts[:n].cpu().numpy(), m.sum((2, 3, 4)))
    rows = m.any(-1)                                         # [n][2][nz][ny]
    assert np.array_equal(db.boxes[:n].cpu().numpy(), [_box(r.any(0)) for r in rows])
    assert np.array_equal(db.tboxes[:n].cpu().numpy(), [_box(r[1]) for r in rows])
    assert np.array_equal(db.zranges[:n].cpu().numpy(), _range(rows).transpose(0, 2, 1))
    f = m[:, 0]
    mom = np.stack([(f.sum((1, 2)) * np.arange(nx)).sum(-1), (f.sum((1, 3)) * np.arange(ny)).sum(-1),
                    (f.sum((2, 3)) * np.arange(nz)).sum(-1), f.sum((1, 2, 3))], -1)
    assert np.array_equal(db.moments[:n].cpu().numpy(), mom)
    nbx, nby, nbz, nbp = db.block_dims()
    if nbp:
        p = np.pad(m, ((0, 0), (0, 0), (0, 16 * nbz - nz), (0, 16 * nby - ny), (0, 0)))
        b = p.reshape(n, 2, nbz, 16, nby, 16, nbx, 16).sum((3, 5, 7)).reshape(n, 2, -1)
        want = np.zeros((n, 2, nbp), dtype=np.int64)
        want[:, :, :b.shape[2]] = b
        assert np.array_equal(db.block_counts[:n].cpu().numpy().astype(np.uint16), want)


@pytest.mark.parametrize("dims,n", [((32, 4, 8), 7), ((32, 8, 9), 1030), ((64, 8, 13), 6), ((32, 2, 100), 5),
                                    ((32, 33, 8), 1025)])
def test_append_with_few_waves(dims, n):
    """Grids of fewer word groups than a block has waves elsewhere: one wave to all of them."""
    test_append_one_pass(dims, n, 0.25)


def test_append_of_millions_of_tiny_entries():
    """More entries than one launch takes threads for, in one call."""
    need_gpu()
    from paper_2205_04550_amd import TumorDB
    n = 8_400_000
    g = torch.Generator(device="cuda").manual_seed(1)
    c = torch.rand((n, 1, 1, 32), generator=g, device="cuda")
    db = TumorDB(32, 1, 1, n, 0.25, 0.675)
    db.storage.fill_(0xa5)
    db.append(c)
    torch.cuda.synchronize()
    bit = 2 ** torch.arange(32, device="cuda", dtype=torch.int64)
    for m, t in enumerate((0.25, 0.675)):
        on = c.view(n, 32) >= t
        word = (on.long() * bit).sum(1)
        assert torch.equal(db.planes[:, m, 0].long() & 0xffffffff, word)
        assert torch.equal(db.popcounts[:, m].long(), on.sum(1))
    assert torch.equal(db.moments[:, 3], (c.view(n, 32) >= 0.25).sum(1))
