"""The C ABI library loads, exports what include/tumordb.h declares, and rejects bad
arguments before touching the GPU (CPU-only checks)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADERS = [os.path.join(ROOT, "include", h) for h in ("tumordb.h", "tumornn.h")]


def declared_functions():
    names = set()
    for h in HEADERS:
        text = re.sub(r"/\*.*?\*/", "", open(h).read(), flags=re.S)
        names |= set(re.findall(r"\b((?:db|emb|nn|labels)_[a-z0-9_]+)\s*\(", text))
    return sorted(names)


def test_header_declares_the_boundary():
    names = declared_functions()
    for n in ("db_build", "db_append", "db_query", "db_query_batch", "db_scan", "db_sync",
              "db_free", "db_last_error", "db_storage_bytes", "db_query_workspace_bytes"):
        assert n in names


def test_library_exports_every_declared_symbol():
    from paper_2205_04550_amd import binding, nn
    lib = ctypes.CDLL(binding.LIB_PATH)
    for n in declared_functions():
        assert hasattr(lib, n), n
    # The Python binding covers exactly the declared C entry points.
    assert set(declared_functions()) == set(binding.SYMBOLS) | set(nn.NN_SYMBOLS)


def test_library_never_allocates_device_memory():
    """No device allocation among the functions that the library calls (the header's promise:
    every device buffer is the caller's)."""
    import subprocess
    from paper_2205_04550_amd import binding
    names = subprocess.run(["nm", "-D", "--undefined-only", binding.LIB_PATH], capture_output=True,
                           text=True, check=True).stdout.split()
    called = {n.split("@")[0] for n in names if n.startswith("hip")}
    assert "hipMemcpyAsync" in called
    assert not {n for n in called if n.startswith(("hipMalloc", "hipExtMalloc", "hipMemPool")) or
                n in ("hipFree", "hipFreeAsync")}


def test_storage_bytes():
    from paper_2205_04550_amd import binding
    # 128^3: 65,536 words per mask plane, 2 planes, 4 bytes; popcounts 8 bytes per entry;
    # row boxes 16, moments 32, the tile order 4, the T1Gd row boxes 16, the per-slice
    # y-ranges 8 nz bytes and the 16^3-block counts 2 masks x 512 blocks x 2 bytes per entry;
    # each piece 256-byte aligned.
    up = lambda b: (b + 255) // 256 * 256
    planes = 50000 * 2 * 65536 * 4
    meta = (up(50000 * 8) + up(50000 * 16) + up(50000 * 32) + up(50000 * 4) + up(50000 * 16) +
            up(50000 * 128 * 8) + up(50000 * 2 * 512 * 2))
    assert binding.storage_bytes(128, 128, 128, 50000) == planes + meta
    # Ragged plane: 32x3x1 = 3 words, padded to 4: 10*2*4*4 = 320 -> 512; then 80, 160,
    # 320, 40, 160 and 80 bytes -> 256, 256, 512, 256, 256 and 256; 2 x 1 x 1 blocks padded
    # to 8: 10*2*8*2 = 320 -> 512.
    assert binding.storage_bytes(32, 3, 1, 10) == 512 + 256 + 256 + 512 + 256 + 256 + 256 + 512
    # 512^3: 32^3 blocks, more than the bound keeps: no block counts.
    assert binding.storage_bytes(512, 512, 512, 1) == (
        up(2 * 512 ** 3 // 8) + 256 * 5 + up(512 * 8))
    assert binding.storage_bytes(33, 4, 4, 10) == 0      # nx not a multiple of 32
    assert binding.storage_bytes(32, 0, 4, 10) == 0
    assert binding.storage_bytes(32, 4, 4, 0) == 0


def test_build_rejects_bad_arguments_before_any_gpu_call():
    from paper_2205_04550_amd import binding as b
    h = ctypes.c_void_p()
    assert b.LIB.db_build(None, 64, 64, 64, 0.25, 0.675, 10, 256, 1 << 30) == b.DB_EINVAL
    assert b"NULL" in b.LIB.db_last_error()
    assert b.LIB.db_build(ctypes.byref(h), 63, 64, 64, 0.25, 0.675, 10, 256, 1 << 30) == b.DB_EINVAL
    assert b.LIB.db_build(ctypes.byref(h), 64, 64, 64, 0.7, 0.25, 10, 256, 1 << 30) == b.DB_EINVAL
    assert b.LIB.db_build(ctypes.byref(h), 64, 64, 64, 0.25, 0.675, 10, None, 1 << 30) == b.DB_EINVAL
    assert b.LIB.db_build(ctypes.byref(h), 64, 64, 64, 0.25, 0.675, 10, 257, 1 << 30) == b.DB_EINVAL
    assert b.LIB.db_build(ctypes.byref(h), 64, 64, 64, 0.25, 0.675, 10, 256, 100) == b.DB_ENOSPC
    assert b"needed" in b.LIB.db_last_error()
    assert h.value is None


def test_calls_on_invalid_handle():
    from paper_2205_04550_amd import binding as b
    assert b.LIB.db_size(None) == -1
    assert b.LIB.db_query(None, 256, 1, 256, 256, None, 256, 1 << 20, None) == b.DB_ESTATE
    assert b.LIB.db_query_batch(None, 1, 256, None, 1, 256, 256, None, 256, 1 << 20, None) == b.DB_ESTATE
    assert b.LIB.db_scan(None, 256, 256, None, 256, 1 << 20, None) == b.DB_ESTATE
    assert b.LIB.db_append(None, 256, 1, None) == b.DB_ESTATE
    assert b.LIB.db_sync(None, None) == b.DB_ESTATE
    assert b.LIB.db_query_workspace_bytes(None, 1, 10) == 0
    b.LIB.db_free(None)  # no-op


def test_group_path_sizes_and_argument_errors_before_any_gpu_call():
    from paper_2205_04550_amd import binding as b
    # tau (M words, 256-byte aligned) + the group minima [M][N / 16] (whole groups only).
    assert b.LIB.emb_groups_workspace_bytes(1024, 50_000) == 4096 + 1024 * 3125 * 4
    assert b.LIB.emb_groups_workspace_bytes(3, 50_021) == 256 + 3 * 3126 * 4
    assert b.LIB.emb_groups_workspace_bytes(0, 100) == 0
    fake = 1 << 20                                  # aligned non-null pointers, never dereferenced
    assert b.LIB.emb_topk_groups(4, 100, None, 5, fake, fake, fake, 1 << 20, None) == b.DB_EINVAL
    assert b.LIB.emb_topk_groups(4, 100, fake, 101, fake, fake, fake, 1 << 20, None) == b.DB_EINVAL
    assert b.LIB.emb_topk_groups(4, 100, fake, 5, fake, fake, None, 1 << 20, None) == b.DB_ENOSPC
    assert b.LIB.emb_topk_groups(4, 100, fake, 5, fake, fake, fake, 16, None) == b.DB_ENOSPC
    sq = fake
    assert b.LIB.emb_distances_groups(b.EMB_BIN, 4, 100, 64, fake, None, None, fake, None, None,
                                      fake, fake, 1 << 20, None) == b.DB_EINVAL
    assert b.LIB.emb_distances_groups(b.EMB_BF16, 4, 100, 64, fake, None, sq, fake, None, sq,
                                      fake, fake, 16, None) == b.DB_ENOSPC
    assert b"needed" in b.LIB.db_last_error()
    # Query codes of 2 GiB or more are refused (32-bit row offsets in the distance kernel).
    assert b.LIB.emb_distances(b.EMB_BF16, 1 << 20, 100, 1024, fake, None, sq, fake, None, sq,
                               fake, None) == b.DB_EINVAL


# A HIP runtime whose launches fail: the error is reported once and cleared, as the real one does.
FAILING_RUNTIME = r"""
static int last;
int __hipPushCallConfiguration() { return 0; }
int __hipPopCallConfiguration() { return 0; }
int hipLaunchKernel() { last = 9; return 9; }
int hipGetLastError(void) { int e = last; last = 0; return e; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { *v = 256; return 0; }
"""
FAILING_CALLS = r"""
import ctypes, sys
ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
from paper_2205_04550_amd import binding as b, nn
L, p, n, f32 = b.LIB, 1 << 20, 1 << 40, nn.NN_F32
conv, lin = (f32, 2, 8, 16, 8, 8, 8), (f32, 32, 512, 256)
adam = (1e-3, 0.9, 0.999, 1e-8, 1, None)
for name, args in (("nn_conv3d_s2_fwd", (*conv, p, p, f32, p, 0, p, None)),
                   ("nn_conv3d_s2_bwd_data", (*conv, p, p, f32, None, 0, p, None)),
                   ("nn_conv3d_s2_bwd_weight", (*conv, p, p, p, p, p, n, None)),
                   ("nn_conv3d_s2_backward", (*conv, p, p, f32, p, p, None, p, p, p, n, None)),
                   ("nn_conv3d_s2_backward", (*conv, p, p, f32, p, p, p, p, p, p, n, None)),
                   ("nn_conv3d_t_s2_backward", (*conv, p, p, f32, p, p, p, p, p, p, n, None)),
                   ("nn_linear_fwd", (*lin, p, p, f32, p, 0, p, None)),
                   ("nn_linear_bwd_data", (*lin, p, p, f32, p, None)),
                   ("nn_linear_bwd_weight", (*lin, p, p, p, p, None)),
                   ("nn_linear_backward", (*lin, p, p, f32, p, p, p, p, p, p, n, None)),
                   ("nn_adam_step", (100, p, p, p, p, None, *adam)),
                   ("emb_knn", (b.EMB_BF16, 4, 40000, 64, p, None, p, p, None, p, 10, 0, p, p, p, n, None))):
    print(name, getattr(L, name)(*args) == b.DB_EHIP)
"""


def test_calls_report_a_launch_that_failed(tmp_path):
    """Each call whose launch fails returns DB_EHIP, not DB_OK (over a runtime that launches
    nothing, so the aligned, non-null pointers are never dereferenced)."""
    import subprocess
    import sys
    src, lib = tmp_path / "hip.c", tmp_path / "libfailing.so"
    src.write_text(FAILING_RUNTIME)
    subprocess.run(["gcc", "-w", "-shared", "-fPIC", str(src), "-o", str(lib)], check=True)
    out = subprocess.run([sys.executable, "-c", FAILING_CALLS, str(lib)], cwd=ROOT, check=True,
                         capture_output=True, text=True).stdout.split()
    assert len(out) == 24
    assert [n for n, ok in zip(out[::2], out[1::2]) if ok != "True"] == []


RECORDING_RUNTIME = r"""
#include <stdio.h>
struct d3 { unsigned x, y, z; };
struct tensor { long long n; char *w, *m, *v, *g, *wb; };
struct table { int count; unsigned first[33]; struct tensor t[32]; };
int __hipPushCallConfiguration() { return 0; }
int __hipPopCallConfiguration(struct d3 *g, struct d3 *b, unsigned long *l, void **s)
{
    static const struct d3 one = {1, 1, 1};
    *g = *b = one;
    *l = 0;
    *s = 0;
    return 0;
}
int hipLaunchKernel(const void *f, struct d3 grid, struct d3 block, void **args, unsigned long l, void *s)
{
    const struct table *t = args[0];
    printf("launch %d\n", t->count);
    for (int i = 0; i < t->count; ++i)
        printf("%u %lld %llu %llu\n", t->first[i], t->t[i].n, (unsigned long long)t->t[i].w,
               (unsigned long long)t->t[i].wb);
    fflush(stdout);
    return 0;
}
int hipGetLastError(void) { return 0; }
"""
ADAM_OF_LARGE_TENSORS = r"""
import ctypes, sys
ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
from paper_2205_04550_amd.nn import LIB
n = [int(a) for a in sys.argv[2:]]
k = len(n)
col = lambda c: (ctypes.c_void_p * k)(*(((i + 1) << 44) + (c << 40) for i in range(k)))
sys.exit(LIB.nn_adam_step_multi(k, (ctypes.c_int64 * k)(*n), col(0), col(1), col(2), col(3), col(4),
                                1e-3, 0.9, 0.999, 1e-8, 1, None))
"""


@pytest.mark.parametrize("sizes", [(5, 1024, 1025), (2 ** 34 + 5, 3, 2 ** 33, 1025), (7,) * 70,
                                   (2 ** 33 - 1024, 2048, 2 ** 35)])
def test_adam_launches_take_fewer_threads_than_a_grid_holds(tmp_path, sizes):
    """Every element of every tensor in exactly one launch, in order, in launches of at most 2^31
    threads (blocks of 256 for 1,024 elements; nothing runs)."""
    import subprocess
    import sys
    src, lib = tmp_path / "hip.c", tmp_path / "librecording.so"
    src.write_text(RECORDING_RUNTIME)
    subprocess.run(["gcc", "-w", "-shared", "-fPIC", str(src), "-o", str(lib)], check=True)
    out = subprocess.run([sys.executable, "-c", ADAM_OF_LARGE_TENSORS, str(lib), *map(str, sizes)], cwd=ROOT,
                         check=True, capture_output=True, text=True).stdout.splitlines()
    done, i = 0, 0
    while out:
        count = int(out.pop(0).split()[1])
        blocks = 0
        for _ in range(count):
            first, n, w, wb = map(int, out.pop(0).split())
            assert first == blocks and n > 0
            assert w == ((i + 1) << 44) + 4 * done and wb == ((i + 1) << 44) + (4 << 40) + 2 * done
            blocks += -(-n // 1024)
            done += n
            if done == sizes[i]:
                i, done = i + 1, 0
        assert blocks * 256 <= 2 ** 31
    assert i == len(sizes) and done == 0
