"""GPU parity of the batched, box-restricted scan (one kernel launch replayed from a HIP graph).

Each query q is cut to its box R_q on both sides: I = |A n B n R|,
A = |A n R|, B = |B n R| (the paper compares whole volumes; the box is this
library's extension). Bar: bit-exact counts, score bits and indices.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import build_db_from_host, need_gpu, say

pytestmark = pytest.mark.gpu

T_LO, T_HI = synth.T_LO, synth.T_HI


def _host(t):
    return t.detach().cpu().numpy()


def _oracle_batch(conc, labels, rois, k):
    out = []
    for q in range(labels.shape[0]):
        roi = None if rois is None else rois[q]
        cnt, sc = oracle.scan_block(conc, labels[q], T_LO, T_HI, roi=roi)
        out.append((cnt, sc, oracle.rank(sc, k)))
    return out


def _compare(res, ref, k):
    idx, score, counts = (_host(t) for t in res)
    for q, (cnt, sc, top) in enumerate(ref):
        assert list(idx[q]) == top, f"query {q}"
        assert np.array_equal(score[q].view(np.uint64), sc[top].view(np.uint64)), f"query {q}"
        c = counts[q].view(np.uint32).astype(np.uint64)
        assert np.array_equal(c, cnt[top]), f"query {q}"


def _edge_rois(dims, nq, rng):
    nx, ny, nz = dims
    fixed = [
        (0, 0, 0, nx, ny, nz),              # whole grid
        (31, 3, 2, 33, 9, 7),               # spans a word boundary in x
        (5, 4, 3, 6, 5, 4),                 # single voxel
        (32, 0, 0, 64, ny, nz),             # word-aligned slab
        (nx - 1, ny - 1, nz - 1, nx, ny, nz),
        (1, 1, 1, nx - 1, ny - 1, nz - 1),
    ]
    rois = list(fixed)
    while len(rois) < nq:
        lo = [int(rng.integers(0, d)) for d in dims]
        hi = [int(rng.integers(l + 1, d + 1)) for l, d in zip(lo, dims)]
        rois.append((*lo, *hi))
    return np.array(rois[:nq], dtype=np.int32)


def test_batch_small_grid_parity():
    need_gpu()
    gen = synth.GenConfig(128, 24, 20, 2.0, 10.0, 0.5, 3.0, 31)
    n, nq, k = 203, 14, 10        # ragged tile count; k <= n
    say(f"batch: build n={n} on {gen.nx}x{gen.ny}x{gen.nz}")
    db, conc = build_db_from_host(gen, n, T_LO, T_HI)
    labels, _ = synth.make_queries(gen, n, nq, synth.BATCH_QUERY_SEED)
    rng = np.random.default_rng(1)
    rois = _edge_rois((gen.nx, gen.ny, gen.nz), nq, rng)
    ref = _oracle_batch(conc, labels, rois, k)
    lab_d = torch.from_numpy(labels).cuda()
    ws = db.workspace(nq, k)
    out = (torch.empty((nq, k), dtype=torch.int32, device="cuda"),
           torch.empty((nq, k), dtype=torch.float64, device="cuda"),
           torch.empty((nq, k, 6), dtype=torch.int32, device="cuda"))
    # First call records the graph, later calls replay it; eager work in between.
    for rep in range(3):
        say(f"batch: replay {rep}")
        for t in out:
            t.fill_(-1)
        res = db.query_batch(lab_d, rois, k, out=out, ws=ws)
        db.sync()
        _compare(res, ref, k)
        _ = (lab_d.float().sum() + 1).item()
    # New boxes through the same graph (only the uploaded plan changes).
    rois2 = _edge_rois((gen.nx, gen.ny, gen.nz), nq, np.random.default_rng(2))[::-1].copy()
    ref2 = _oracle_batch(conc, labels, rois2, k)
    res = db.query_batch(lab_d, rois2, k, out=out, ws=ws)
    db.sync()
    _compare(res, ref2, k)


def test_batch_whole_grid_equals_single_query():
    need_gpu()
    gen = synth.SMALL
    n, nq, k = 300, 5, 10
    say("batch vs single")
    db, conc = build_db_from_host(gen, n, T_LO, T_HI)
    labels, _ = synth.make_queries(gen, n, nq, synth.BATCH_QUERY_SEED)
    lab_d = torch.from_numpy(labels).cuda()
    bi, bs, bc = db.query_batch(lab_d, None, k)
    db.sync()
    for q in range(nq):
        si, ss, sc = db.query(lab_d[q], k)
        db.sync()
        assert torch.equal(bi[q], si) and torch.equal(bs[q], ss) and torch.equal(bc[q], sc)


def test_batch_boxes_of_the_workload_generator():
    need_gpu()
    gen = synth.SMALL
    n, nq, k = 256, 16, 10
    say("batch: workload-style boxes on 64^3")
    db, conc = build_db_from_host(gen, n, T_LO, T_HI)
    labels, _ = synth.make_queries(gen, n, nq, synth.BATCH_QUERY_SEED)
    rois = synth.make_rois(labels, synth.ROI_SEED)
    ref = _oracle_batch(conc, labels, rois, k)
    res = db.query_batch(torch.from_numpy(labels).cuda(), rois, k)
    db.sync()
    _compare(res, ref, k)


def test_batch_results_do_not_depend_on_launch_shape():
    """Every launch shape the autotuner may pick (slab depth, block size, entries per tile,
    queries per chunk) and the kernel that reads the database through L2 (slab_planes
    = -1) give the same bytes."""
    need_gpu()
    gen = synth.GenConfig(128, 24, 20, 2.0, 10.0, 0.5, 3.0, 31)
    n, nq, k = 75, 9, 7
    db, conc = build_db_from_host(gen, n, T_LO, T_HI)
    labels, _ = synth.make_queries(gen, n, nq, synth.BATCH_QUERY_SEED)
    rois = _edge_rois((gen.nx, gen.ny, gen.nz), nq, np.random.default_rng(3))
    ref = _oracle_batch(conc, labels, rois, k)
    lab_d = torch.from_numpy(labels).cuda()
    for shape in [(0, 0, 0, 0), (1, 256, 4, 0), (2, 512, 8, 0), (3, 1024, 8, 4), (7, 512, 4, 2),
                  (20, 1024, 8, 1), (0, 1024, 8, 9), (-1, 0, 0, 0)]:
        say(f"shape planes, threads, tile, chunk = {shape}")
        db.tune_batch(*shape)
        res = db.query_batch(lab_d, rois, k)
        db.sync()
        _compare(res, ref, k)


@pytest.mark.parametrize("planes,tile", [(0, 4), (0, 8), (-1, 0)])
def test_batch_more_queries_than_one_chunk(planes, tile):
    """300 queries (more than the 256 of one query chunk: two chunks, each an item of the
    block per tile) with uneven boxes, against the oracle's loop over every entry;
    also through the kernel that reads the database through L2."""
    need_gpu()
    gen = synth.GenConfig(128, 24, 20, 2.0, 10.0, 0.5, 3.0, 37)
    n, nq, k = 61, 300, 5
    say(f"batch: {nq} queries, planes {planes}, tile {tile}")
    db, conc = build_db_from_host(gen, n, T_LO, T_HI)
    labels, _ = synth.make_queries(gen, n, nq, synth.BATCH_QUERY_SEED)
    rois = _edge_rois((gen.nx, gen.ny, gen.nz), nq, np.random.default_rng(5))
    cnt, sc = oracle.scan_block_multi(conc, labels, T_LO, T_HI, rois)
    db.tune_batch(planes, 0, tile, 0)
    res = db.query_batch(torch.from_numpy(labels).cuda(), rois, k)
    db.sync()
    _compare(res, [(cnt[q], sc[q], oracle.rank(sc[q], k)) for q in range(nq)], k)


@pytest.mark.parametrize("nq,n,dims", [(96, 61, (128, 64, 96)), (128, 130, (128, 45, 136)), (129, 63, (128, 128, 48)),
                                       (257, 65, (128, 6, 1024)), (300, 5, (128, 101, 61))])
def test_batch_matrix_core_kernel(nq, n, dims):
    """The matrix-core kernel (96 queries and more on rows of 128 voxels) with each split of its
    waves, groups of 32 queries and tiles of 64 entries with a rest, uneven boxes and empty
    entries, against the oracle's loop; the vector kernel asked for gives the same bytes."""
    need_gpu()
    gen = synth.GenConfig(*dims, 2.0, min(dims) / 2, 0.5, 3.0, 41)
    k = 5
    say(f"batch on matrix cores: {nq} queries, {n} entries, {dims}")
    conc = gen.conc_cpu(0, n)
    conc[3] = 0.0
    db, conc = build_db_from_host(gen, n, T_LO, T_HI, conc=conc)
    labels, _ = synth.make_queries(gen, n, nq, synth.BATCH_QUERY_SEED)
    rng = np.random.default_rng(nq)
    rois = _edge_rois(dims, nq, rng) if min(dims) > 9 else np.tile((0, 0, 0) + dims, (nq, 1)).astype(np.int32)
    for q in range(6, nq, 2):                            # every other box nearly the whole grid
        rois[q] = [*(int(rng.integers(0, d // 8 + 1)) for d in dims),
                   *(d - int(rng.integers(0, d // 8 + 1)) for d in dims)]
    cnt, sc = oracle.scan_block_multi(conc, labels, T_LO, T_HI, rois)
    ref = [(cnt[q], sc[q], oracle.rank(sc[q], k)) for q in range(nq)]
    lab_d = torch.from_numpy(labels).cuda()
    res = db.query_batch(lab_d, rois, k)
    db.sync()
    _compare(res, ref, k)
    db.tune_batch(0, 1024, 4, 0)
    res = db.query_batch(lab_d, rois, k)
    db.sync()
    _compare(res, ref, k)


def test_batch_kinds_alternate_on_one_handle():
    """Calls that take the matrix-core kernel (many whole-grid queries) and the vector kernel (a few)
    in turn, and after an append: the oracle's results, and the handle's tile order is one of all
    its entries after each."""
    need_gpu()
    dims = (128, 80, 80)
    gen = synth.GenConfig(*dims, 2.0, 20.0, 0.5, 3.0, 41)
    n, k = 70, 5
    db, conc = build_db_from_host(gen, 61, T_LO, T_HI, capacity=n)
    conc = np.concatenate([conc, gen.conc_cpu(61, n - 61)])
    labels, _ = synth.make_queries(gen, n, 96, synth.BATCH_QUERY_SEED)
    whole = np.tile((0, 0, 0) + dims, (96, 1)).astype(np.int32)
    lab_d = torch.from_numpy(labels).cuda()
    for have in (61, n):
        db.append(torch.from_numpy(conc[len(db):have]).cuda())
        cnt, sc = oracle.scan_block_multi(conc[:have], labels, T_LO, T_HI, whole)
        ref = [(cnt[q], sc[q], oracle.rank(sc[q], k)) for q in range(96)]
        for nq in (96, 7, 96, 7, 7, 96):
            say(f"batch kinds in turn: {have} entries, {nq} queries")
            res = db.query_batch(lab_d[:nq], whole[:nq], k)
            db.sync()
            _compare(res, ref[:nq], k)
            assert sorted(_host(db.tile_order[:have])) == list(range(have))


def test_batch_matrix_core_kernel_counts_up_to_its_limit():
    """The largest grid that the matrix-core kernel takes (16.77 of 2^24 voxels), masks that fill it
    and boxes of all or nearly all of it, with tiles enough that none is split over blocks: every
    voxel adds one to a float accumulator, and the counts are the boxes' voxels exactly."""
    need_gpu()
    from paper_2205_04550_amd import TumorDB
    nx, ny, nz = dims = (128, 362, 362)
    n, nq, k = 8192, 2048, 384                              # 128 tiles of 64 x 8 chunks of 256
    if torch.cuda.mem_get_info()[0] < (100 << 30):
        pytest.skip("needs 100 GiB")
    say(f"batch on matrix cores: {nq} queries, {n} entries, {dims}")
    conc = torch.ones((64, nz, ny, nx), device="cuda")
    for e in range(64):                                     # entry e lacks its first e slices
        conc[e, :e] = 0.0
    db = TumorDB(*dims, n, T_LO, T_HI)
    for _ in range(n // 64):
        db.append(conc)
    torch.cuda.synchronize()
    del conc
    labels = torch.full((nq, nz, ny, nx), 3, dtype=torch.uint8, device="cuda")
    rois = np.tile((0, 0, 0) + dims, (nq, 1)).astype(np.int32)
    rois[1::3, 0] = 1
    rois[2::3, 4] = ny - 5
    idx, score, counts = (_host(t) for t in db.query_batch(labels, rois, k))
    db.sync()
    # The best: the 128 entries without a slice less, then those that lack one, then two.
    order = [e + 64 * i for e in range(3) for i in range(n // 64)]
    lacks = np.repeat(np.arange(3), n // 64)
    side = (rois[:, 3:] - rois[:, :3]).astype(np.int64)
    box = side.prod(1)
    b = box[:, None] - lacks[None] * (side[:, 0] * side[:, 1])[:, None]
    assert (idx == np.array(order)).all()
    c = counts.view(np.uint32).astype(np.int64)
    assert (c[..., 0:2] == b[..., None]).all() and (c[..., 4:6] == b[..., None]).all()
    assert (c[..., 2:4] == box[:, None, None]).all()
    want = 2.0 * b / (box[:, None] + b)
    assert np.array_equal(score, want + want)
    del db, labels
    torch.cuda.empty_cache()
