// train.hip — the autoencoder's training kernels (float activations).
//
// One training step (paper Sec. 2.4 "Implementation": strided convolutions, kernel 3, stride
// 2, and their transposes) is three maps per convolution: the forward, the adjoint and the
// weight gradient. "Coarse" is the strided side of a layer (Co channels), "fine" the other one
// (Ci channels, twice the size along each axis).
//
// Every sum here is formed term by term in the order of the direct loops (conv_fwd_kernel,
// conv_bwd_data_kernel, conv_bwd_weight_partial in nn.hip): an FP32 matrix product of this
// architecture is the chain of its four (or two) fused multiply-adds in k order, rounded after
// each, so an implicit GEMM whose k runs in a loop's order gives that loop's bits. A training
// step passes through ReLU kinks, where a last-bit change of a sum can switch a unit: the same
// order keeps whole steps reproducible across these kernels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "../../include/tumornn.h"
#include "common.hpp"
#include "internal.hpp"

namespace tdb {

namespace {

typedef __amdgpu_buffer_rsrc_t rsrc_t;

// A buffer over at most 2 GiB - 4 bytes from p: loads at kOut (or past the end) give 0.
constexpr uint32_t kOut = 0x80000000u;
__device__ __forceinline__ rsrc_t make_rsrc(const void *p, int64_t bytes)
{
    const int n = (int)(bytes < 0x7ffffffc ? bytes : 0x7ffffffc);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, n, 0x00020000);
}
__device__ __forceinline__ float buf_f32(rsrc_t r, uint32_t off, uint32_t soff = 0)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0));
}
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float2 buf_f32x2(rsrc_t r, uint32_t off, uint32_t soff = 0)
{
    const u32x2_t u = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0));
    return make_float2(__uint_as_float(u.x), __uint_as_float(u.y));
}

// Weight i of a buffer, or 0 unless ok (a plain conditional load would become a branch that waits
// for the load before the next one is issued).
__device__ __forceinline__ uint16_t buf_w(rsrc_t r, bool ok, uint32_t i, uint16_t)
{
    return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, ok ? 2 * i : kOut, 0, 0);
}
__device__ __forceinline__ float buf_w(rsrc_t r, bool ok, uint32_t i, float)
{
    return buf_f32(r, ok ? 4 * i : kOut);
}

typedef float f32x2_u __attribute__((ext_vector_type(2), aligned(4)));   // 4-byte aligned pair

// ---- wave sums of many values ------------------------------------------------------------------
//
// The sum over the 64 lanes of each of N values, as the butterfly (lane ^ 32, ^ 16, ... ^ 1)
// adds it, but halving the values with the lanes: of two values a and b, half of the lanes go
// on with a and half with b, so N values take about 2 N exchanges and adds instead of 6 N.
// On return lane l of v[m] holds the total of value 64 m + reverse6(l).
__device__ __forceinline__ void swap32(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap16(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
template <int N>
__device__ __forceinline__ void wave_sums(float (&v)[N], int lane)
{
    constexpr int n1 = (N + 1) / 2, n2 = (n1 + 1) / 2, n3 = (n2 + 1) / 2, n4 = (n3 + 1) / 2,
                  n5 = (n4 + 1) / 2, n6 = (n5 + 1) / 2;
#pragma unroll
    for (int m = 0; m < n1; ++m) {
        float a = v[2 * m], b = 2 * m + 1 < N ? v[2 * m + 1] : 0.f;
        swap32(a, b);
        v[m] = a + b;
    }
#pragma unroll
    for (int m = 0; m < n2; ++m) {
        float a = v[2 * m], b = 2 * m + 1 < n1 ? v[2 * m + 1] : 0.f;
        swap16(a, b);
        v[m] = a + b;
    }
#define TDB_HALVE(n_out, n_in, bit, exchange)                                                      \
    _Pragma("unroll") for (int m = 0; m < n_out; ++m) {                                            \
        const float a = v[2 * m], b = 2 * m + 1 < n_in ? v[2 * m + 1] : 0.f;                       \
        const float keep = (lane & bit) ? b : a, send = (lane & bit) ? a : b;                      \
        v[m] = keep + exchange;                                                                    \
    }
#define TDB_DPP(ctrl) __uint_as_float(dpp_u32<ctrl>(__float_as_uint(send)))
    TDB_HALVE(n3, n2, 8, TDB_DPP(0x128))                  // row_ror:8
    TDB_HALVE(n4, n3, 4, __shfl_xor(send, 4, 64))
    TDB_HALVE(n5, n4, 2, TDB_DPP(0x4e))                   // quad_perm [2,3,0,1]
    TDB_HALVE(n6, n5, 1, TDB_DPP(0xb1))                   // quad_perm [1,0,3,2]
#undef TDB_DPP
#undef TDB_HALVE
}

// A number of coarse voxels in mixed radix, to advance a position without divisions.
struct Step {
    int b, z, y, x;
};
Step step_of(int n, int OD, int OH, int OW)
{
    return {n / OW / OH / OD, n / OW / OH % OD, n / OW % OH, n % OW};
}
__device__ __forceinline__ void advance(int &b, int &z, int &y, int &x, const Step &st, int OD,
                                        int OH, int OW)
{
    x += st.x;
    y += st.y;
    z += st.z;
    b += st.b;
    if (x >= OW) { x -= OW; ++y; }
    if (y >= OH) { y -= OH; ++z; }
    if (z >= OD) { z -= OD; ++b; }
}

// ---- weight gradient ------------------------------------------------------------------------
//
// dW[co][ci][tap] = sum over (sample, coarse voxel o) of dY[co][o] X[ci][2 o + tap - 1]. Grid
// (chunks of kWgChunkF positions, Ci, ceil(Co / CB)); a thread takes every 256th position of
// the chunk, CB coarse channels and all 27 taps (and the sum of dY, tap 27), 28 CB sums in
// registers. MASK: dY counts only where Y > 0 (the layer's ReLU), so that the gradient before the
// ReLU need not be written where only this kernel reads it. Per position the fine values come as nine pairs (x = 2 ow, 2 ow + 1) by buffer
// loads, whose out-of-range answer 0 is the padding; the left column (2 ow - 1) is the second
// value of the lane before (SHIFT: rows of 64 / n voxels, so that a wave starts a row) or a
// load of its own. Positions advance by 256 in mixed radix: no division in the loop, and a
// position's loads are all issued before the first product (waiting for each row in turn
// made the 2 -> 8 channel layer 107 us). Bound by vector issue and the loads' latency at three
// waves per SIMD; the sums of a wave are formed halving the values with the lanes. Batch 32:
// 42 / 38 / 20 / 12 us for the layers 2 -> 8 (64^3), 8 -> 16, 16 -> 32, 32 -> 64, against
// 132 / 128 / 66 / 47 us for conv_bwd_weight_partial (27 bounds-checked loads per position
// and channel, six exchanges per summed value); the eight layers of a step with their final
// sums 270 us instead of 900 us.
constexpr int kWgChunkF = 4096;
constexpr int kWgCBF = 4;



template <bool SHIFT, bool MASK>
__global__ void __launch_bounds__(256, 3) conv_wgrad_kernel(int B, int Ci, int Co, int D, int H,
                                                            int W, Step st,
                                                            const float *__restrict__ X,
                                                            const float *__restrict__ dY,
                                                            const float *__restrict__ Y,
                                                            float *__restrict__ partial)
{
    constexpr int CB = kWgCBF, NV = CB * 28, NR = (NV + 63) / 64;
    __shared__ float red[4][NR * 64];
    const int OD = D / 2, OH = H / 2, OW = W / 2;
    const int64_t osp = (int64_t)OD * OH * OW, isp = 8 * osp;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int co0 = blockIdx.z * CB, ci = blockIdx.y;
    const int64_t P = (int64_t)B * osp, p0 = (int64_t)blockIdx.x * kWgChunkF;
    const int64_t b0 = p0 / osp;
    // Buffers from this chunk's first sample on; the host checks that its samples stay below 2 GiB.
    const rsrc_t xr = make_rsrc(X + (b0 * Ci + ci) * isp, ((B - b0) * Ci - ci) * isp * 4);
    const rsrc_t yr = make_rsrc(dY + (b0 * Co + co0) * osp, ((B - b0) * Co - co0) * osp * 4);
    const rsrc_t mr = make_rsrc((MASK ? Y : dY) + (b0 * Co + co0) * osp, ((B - b0) * Co - co0) * osp * 4);
    int o = (int)(p0 - b0 * osp) + tid;
    int x = o % OW, y = (o / OW) % OH, z = o / (OW * OH), b = z / OD;
    z -= b * OD;
    float acc[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) acc[i] = 0.f;
    const uint32_t rowB = 4u * W, planeB = 4u * W * H, bX = 4u * (uint32_t)(Ci * isp),
                   bY = 4u * (uint32_t)(Co * osp);
    const int n = (int)min((int64_t)kWgChunkF, P - p0);
    for (int i = tid; i - tid < n; i += 256) {
        const bool in = i < n;                           // past the end: both sides read zeros
        const uint32_t xo = (uint32_t)b * bX + 2u * z * planeB + 2u * y * rowB + 8u * x;
        const uint32_t yo = in ? (uint32_t)b * bY + 4u * ((z * OH + y) * OW + x) : kOut;
        float g[CB];
#pragma unroll
        for (int c = 0; c < CB; ++c)                     // a channel past the last is not stored
            g[c] = buf_f32(yr, yo, 4u * (uint32_t)min(c, Co - 1 - co0) * (uint32_t)osp);
        float mk[CB];
#pragma unroll
        for (int c = 0; MASK && c < CB; ++c)
            mk[c] = buf_f32(mr, yo, 4u * (uint32_t)min(c, Co - 1 - co0) * (uint32_t)osp);
        float2 p[9];                                     // all loads before their first use
        float l[9];
#pragma unroll
        for (int kd = 0; kd < 3; ++kd)
#pragma unroll
            for (int kh = 0; kh < 3; ++kh) {             // low edges only: 2 o + 1 is in range
                const bool ok = in & ((kd != 0) | (z != 0)) & ((kh != 0) | (y != 0));
                const uint32_t ro = ok ? xo + (kd - 1) * planeB + (kh - 1) * rowB : kOut;
                p[kd * 3 + kh] = buf_f32x2(xr, ro);
                if (!SHIFT) l[kd * 3 + kh] = buf_f32(xr, ok & (x != 0) ? ro - 4 : kOut);
            }
        float v[9][3];
#pragma unroll
        for (int r = 0; r < 9; ++r) {
            if (SHIFT) {
                l[r] = __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(p[r].y), 0x138,
                                                                   0xf, 0xf, true));   // wave_shr:1
                l[r] = x ? l[r] : 0.f;
            }
            v[r][0] = l[r];
            v[r][1] = p[r].x;
            v[r][2] = p[r].y;
        }
#pragma unroll
        for (int c = 0; MASK && c < CB; ++c) g[c] = mk[c] > 0.f ? g[c] : 0.f;
#pragma unroll
        for (int c = 0; c < CB; ++c) {
#pragma unroll
            for (int r = 0; r < 27; ++r) acc[c * 28 + r] = __builtin_fmaf(g[c], v[r / 3][r % 3], acc[c * 28 + r]);
            acc[c * 28 + 27] += g[c];
        }
        advance(b, z, y, x, st, OD, OH, OW);
    }
    wave_sums(acc, lane);
    const int at = (int)(__brev((unsigned)lane) >> 26);
#pragma unroll
    for (int m = 0; m < NR; ++m) red[wave][64 * m + at] = acc[m];
    __syncthreads();
    if (tid < NV) {
        const int c = tid / 28, k = tid - c * 28;
        if (co0 + c < Co)
            partial[(((int64_t)blockIdx.x * Co + co0 + c) * Ci + ci) * 28 + k] =
                ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
    }
}

// Adds the chunks in order: a block takes 32 of the Co Ci 28 sums, loads them from up to 256
// chunks at a time with all its threads and adds them with one thread per sum: 9 us for the
// 256 chunks of the first layer at batch 32, where one thread per sum that loaded as it added
// took 60 us.
__global__ void __launch_bounds__(512) conv_wgrad_final_kernel(int chunks, int Ci, int64_t N,
                                                               const float *__restrict__ partial,
                                                               float *__restrict__ dW,
                                                               float *__restrict__ dbias)
{
    __shared__ float buf[256][32];
    const int o = threadIdx.x & 31, g = threadIdx.x >> 5;
    const int64_t i = (int64_t)blockIdx.x * 32 + o;
    float s = 0.f;
    for (int c0 = 0; c0 < chunks; c0 += 256) {
        const int nc = min(256, chunks - c0);
#pragma unroll 16
        for (int c = g; c < nc; c += 16) buf[c][o] = i < N ? partial[(c0 + c) * N + i] : 0.f;
        __syncthreads();
        if (g == 0) {
#pragma unroll 8
            for (int c = 0; c < nc; ++c) s += buf[c][o];
        }
        __syncthreads();
    }
    if (g != 0 || i >= N) return;
    const int64_t cc = i / 28;
    const int k = (int)(i - cc * 28);
    if (k < 27) dW[cc * 27 + k] = s;
    else if (dbias && cc % Ci == 0) dbias[cc / Ci] = s;
}

}  // namespace

bool conv_wgrad_ok(int Ci, int Co, int D, int H, int W)
{
    // A chunk's samples, from the first one's start, are addressed with 31-bit byte offsets.
    const int64_t osp = (int64_t)(D / 2) * (H / 2) * (W / 2), samples = (kWgChunkF - 1) / osp + 2;
    return samples * std::max<int64_t>((int64_t)Ci * 8, Co) * osp * 4 < ((int64_t)1 << 31);
}

hipError_t launch_conv_wgrad(int B, int Ci, int Co, int D, int H, int W, const float *X,
                             const float *dY, const float *Y, float *dW, float *dbias, float *ws,
                             hipStream_t s)
{
    const int OD = D / 2, OH = H / 2, OW = W / 2;
    const int64_t P = (int64_t)B * OD * OH * OW;
    const int chunks = (int)((P + kWgChunkF - 1) / kWgChunkF);
    const Step st = step_of(256, OD, OH, OW);
    const dim3 grid((unsigned)chunks, (unsigned)Ci, (unsigned)((Co + kWgCBF - 1) / kWgCBF));
#define TDB_WGRAD(SHIFT_, MASK_)                                                                   \
    hipLaunchKernelGGL((conv_wgrad_kernel<SHIFT_, MASK_>), grid, dim3(256), 0, s, B, Ci, Co, D, H, W, \
                       st, X, dY, Y, ws)
    if (64 % OW == 0) {
        if (Y) TDB_WGRAD(true, true); else TDB_WGRAD(true, false);
    } else {
        if (Y) TDB_WGRAD(false, true); else TDB_WGRAD(false, false);
    }
#undef TDB_WGRAD
    const int64_t N = (int64_t)Co * Ci * 28;
    hipLaunchKernelGGL(conv_wgrad_final_kernel, dim3((unsigned)((N + 31) / 32)), dim3(512), 0, s,
                       chunks, Ci, N, (const float *)ws, dW, dbias);
    return hipGetLastError();
}

namespace {

// ---- adjoint (input gradient; transposed-convolution forward) ----------------------------------
//
// dX[ci][i] = bias[ci] + sum over co and the taps with i + 1 - tap even of W[co][ci][tap]
// dY[co][(i + 1 - tap) / 2], in the order co, kd, kh, kw. Along an axis the even fine voxel 2 j
// has tap 1 on coarse voxel j, the odd one 2 j + 1 has tap 0 on j + 1, then tap 2 on j. So for 16
// coarse voxels (the N of a product) the eight parities of the fine voxels are rows of M, k runs
// over co and the neighbours j + 1, j of each odd axis, and a row whose parity lacks a neighbour
// has weight zero there: the sum's terms keep their order.
//   few fine channels (Ci <= 2): the 16 rows are (pz, py, ci, px), one tile, 8 Co terms;
//   otherwise a tile is (pz, py) and eight fine channels, rows (ci, px), and k has only the
//   neighbours its z and y parities use: 2, 4, 4 or 8 terms per co.
// A wave keeps a tile's weights in registers (through LDS, which the four waves of a block
// fill once) and walks its share of the voxels; lane l needs dY at voxel l % 16 and neighbour
// l / 16, one buffer load per product straight from the caches, with no vector instruction
// in between: the lane's offset is fixed per voxel (out of range where the neighbour is) and
// the channel is the load's scalar offset. Zero weights times an infinity would leave a NaN
// that the direct loop does not have: a wave that finds a NaN in its results redoes them as
// that loop. Loads run three batches of eight products ahead (one batch: the 32 -> 64 layer took
// 32 us, the latency of each batch being longer than its products). Batch 32, transposes of
// the layers 2 -> 8 (64^3), 8 -> 16, 16 -> 32, 32 -> 64: 40 / 28 / 18 / 15 us, where a thread
// per fine voxel with its weights broadcast from LDS (conv_bwd_data_kernel, kept for the sizes
// launch_conv_adjoint does not take and for double) took 262 / 73 / 55 / 79 us. The first is
// bound by its writes (67 MB), the others by the matrix products and the first loads' latency.
__device__ __forceinline__ float wt_f32(uint16_t w) { return __uint_as_float((uint32_t)w << 16); }
__device__ __forceinline__ float wt_f32(float w) { return w; }

struct AdjArgs {
    int B, Ci, Co, D, H, W, relu, groups, gpw;   // groups of 16 coarse voxels; groups per wave
    Step st;                                     // kAdjNG groups
    const float *dY, *bias;
    float *dX;
};
constexpr int kAdjNG = 2;                        // groups that go together (shared weights)

// One output by the direct loop, a coarse channel's loads before their sums: along an axis an odd voxel has tap 0
// on coarse voxel j + 1, then tap 2 on j, an even one tap 1 on j.
template <class WT>
__device__ float adjoint_direct(const AdjArgs &a, const WT *Wt, int b, int ci, int id, int ih, int iw)
{
    const int OD = a.D / 2, OH = a.H / 2, OW = a.W / 2, osp = OD * OH * OW;
    const int z0 = (id + 1) >> 1, y0 = (ih + 1) >> 1, x0 = (iw + 1) >> 1;
    const int tap0 = (id & 1 ? 0 : 9) + (ih & 1 ? 0 : 3) + (iw & 1 ? 0 : 1);
    const float *g = a.dY + (int64_t)b * a.Co * osp + (z0 * OH + y0) * OW + x0;
    const WT *w = Wt + (int64_t)ci * 27 + tap0;
    float s = a.bias ? a.bias[ci] : 0.f;
#pragma unroll 1
    for (int co = 0; co < a.Co; ++co) {
        float gv[8], wv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int dz = e >> 2, dy = e >> 1 & 1, dx = e & 1;
            const bool ok = (dz ? id & 1 : z0 < OD) && (dy ? ih & 1 : y0 < OH) && (dx ? iw & 1 : x0 < OW);
            gv[e] = ok ? g[-(dz * OH + dy) * OW - dx] : 0.f;
            wv[e] = ok ? wt_f32(w[18 * dz + 6 * dy + 2 * dx]) : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) s = __builtin_fmaf(wv[e], gv[e], s);   // zero by zero adds nothing
        g += osp;
        w += (int64_t)a.Ci * 27;
    }
    return s;
}

// Tap of parity p for neighbour i (0: j + 1, 1: j); -1: none.
__device__ __forceinline__ int adj_tap(int p, int i) { return p ? 2 * i : (i ? 1 : -1); }

// PZ, PY = 1, 1 with ROWS8: the tile of few fine channels (all eight parities); otherwise the
// tile of z and y parity PZ, PY. CO: Co rounded up to the registers' size.
template <class WT, int PZ, int PY, bool ROWS8, int CO>
__device__ __forceinline__ void adjoint_tile(const AdjArgs &a, const WT *Wt, const WT *wsh, int ci0)
{
    constexpr int CIB = ROWS8 ? 2 : 8;
    constexpr int NK = PZ && PY ? 2 * CO : (PZ || PY ? CO : CO / 2);   // products per 16 voxels
    constexpr int KC = NK < 8 ? NK : 8, NG = kAdjNG, NCH = NK / KC, R = 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, kq = lane >> 4;
    const int OD = a.D / 2, OH = a.H / 2, OW = a.W / 2;
    const int osp = OD * OH * OW;
    const int nci = min(CIB, a.Ci - ci0);
    // Row of this lane's weights, and its neighbours: x always by kq's low bit; z and y by the
    // high bit or the product's parity.
    const int cil = ROWS8 ? (l16 >> 1) & 1 : l16 >> 1, px = l16 & 1;
    const int pz = ROWS8 ? l16 >> 3 : PZ, py = ROWS8 ? (l16 >> 2) & 1 : PY;
    const int xi = kq & 1, hi = kq >> 1;
    float w[NK];
#pragma unroll
    for (int s = 0; s < NK; ++s) {
        int co, zi, yi;
        if (PZ && PY) { co = s / 2; zi = s & 1; yi = hi; }
        else if (PZ) { co = s; zi = hi; yi = 1; }
        else if (PY) { co = s; zi = 1; yi = hi; }
        else { co = 2 * s + hi; zi = 1; yi = 1; }
        const int tz = adj_tap(pz, zi), ty = adj_tap(py, yi), tx = adj_tap(px, xi);
        const bool ok = tz >= 0 && ty >= 0 && tx >= 0 && cil < nci && co < a.Co;
        w[s] = wt_f32(wsh[ok ? (co * CIB + cil) * 27 + tz * 9 + ty * 3 + tx : CO * CIB * 27]);
    }
    float binit[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = ROWS8 ? r >> 1 : 2 * kq + (r >> 1);
        binit[r] = a.bias && c < nci ? a.bias[ci0 + c] : 0.f;
    }
    const int g0 = (blockIdx.x * 4 + wave) * a.gpw, g1 = min(a.groups, g0 + a.gpw);
    // The buffer starts at this block's first sample; the host checks the block's samples.
    const int64_t pb = (int64_t)blockIdx.x * 4 * a.gpw * 16;
    const int b0 = (int)(pb / osp);
    const rsrc_t yr = make_rsrc(a.dY + (int64_t)b0 * a.Co * osp, (int64_t)(a.B - b0) * a.Co * osp * 4);
    const int64_t fsp = 8 * (int64_t)osp;
    int vb[NG], vz[NG], vy[NG], vx[NG];
#pragma unroll
    for (int j = 0; j < NG; ++j) {
        const int o = (int)((int64_t)(g0 + j) * 16 + l16 - (int64_t)b0 * osp);
        vx[j] = o % OW;
        vy[j] = o / OW % OH;
        vz[j] = o / (OW * OH);
        vb[j] = vz[j] / OD;
        vz[j] -= vb[j] * OD;
    }
    for (int g = g0; g < g1; g += NG) {
        uint32_t off[NG][2];
        f32x4 acc[NG];
#pragma unroll
        for (int j = 0; j < NG; ++j) {
            const bool in = g + j < g1 && b0 + vb[j] < a.B;
            const int nx = 1 - xi;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                int ny, nz, dc = 0;
                if (PZ && PY) { nz = 1 - e; ny = 1 - hi; }
                else if (PZ) { nz = 1 - hi; ny = 0; }
                else if (PY) { nz = 0; ny = 1 - hi; }
                else { nz = ny = 0; dc = hi; }
                const bool ok = in & (vz[j] + nz < OD) & (vy[j] + ny < OH) & (vx[j] + nx < OW);
                off[j][e] = ok ? 4u * (uint32_t)((vb[j] * a.Co + dc) * osp +
                                                 ((vz[j] + nz) * OH + vy[j] + ny) * OW + vx[j] + nx)
                               : kOut;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[j][r] = binit[r];
        }
        float v[R][KC][NG];                      // loads three batches of products ahead
        auto load = [&](int c) {
#pragma unroll
            for (int k = 0; k < KC; ++k) {
                const int s = c * KC + k;
                const int co = PZ && PY ? s / 2 : (PZ || PY ? s : 2 * s);
                const uint32_t so = 4u * (uint32_t)osp * (uint32_t)min(co, a.Co - 1);
#pragma unroll
                for (int j = 0; j < NG; ++j)
                    v[c % R][k][j] = buf_f32(yr, off[j][PZ && PY ? s & 1 : 0], so);
            }
        };
#pragma unroll
        for (int c = 0; c < R - 1 && c < NCH; ++c) load(c);
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if (c + R - 1 < NCH) load(c + R - 1);
#pragma unroll
            for (int k = 0; k < KC; ++k)
#pragma unroll
                for (int j = 0; j < NG; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[c * KC + k], v[c % R][k][j], acc[j], 0, 0, 0);
        }
        int redo = 0;                            // groups in which this lane found a NaN
#pragma unroll
        for (int j = 0; j < NG; ++j) {
            const bool in = g + j < g1 && b0 + vb[j] < a.B;
            const int oz = ROWS8 ? kq >> 1 : PZ, oy = ROWS8 ? kq & 1 : PY;
            float *d = a.dX + ((int64_t)(b0 + vb[j]) * a.Ci + ci0) * fsp +
                       ((int64_t)(2 * vz[j] + oz) * a.H + 2 * vy[j] + oy) * a.W + 2 * vx[j];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int c = ROWS8 ? e : 2 * kq + e;
                float r0 = acc[j][2 * e], r1 = acc[j][2 * e + 1];
                if (in && c < nci && (!(r0 == r0) || !(r1 == r1))) redo |= 1 << j;
                if (a.relu && r0 < 0.f) r0 = 0.f;
                if (a.relu && r1 < 0.f) r1 = 0.f;
                if (in && c < nci) *reinterpret_cast<f32x2_u *>(d + c * fsp) = (f32x2_u){r0, r1};
            }
            advance(vb[j], vz[j], vy[j], vx[j], a.st, OD, OH, OW);
        }
        if (__any(redo)) {
#pragma unroll 1
            for (int q = 0; q < 4 * NG; ++q) {
                if (!(redo >> (q >> 2) & 1)) continue;
                const int o = (int)((int64_t)(g + (q >> 2)) * 16 + l16 - (int64_t)b0 * osp);
                const int b = b0 + o / osp, e = (q >> 1) & 1, c = ROWS8 ? e : 2 * kq + e;
                const int id = 2 * (o / (OW * OH) % OD) + (ROWS8 ? kq >> 1 : PZ);
                const int ih = 2 * (o / OW % OH) + (ROWS8 ? kq & 1 : PY), iw = 2 * (o % OW) + (q & 1);
                if (c >= nci) continue;
                float r = adjoint_direct(a, Wt, b, ci0 + c, id, ih, iw);
                if (a.relu && r < 0.f) r = 0.f;
                a.dX[((int64_t)b * a.Ci + ci0 + c) * fsp + ((int64_t)id * a.H + ih) * a.W + iw] = r;
            }
        }
    }
}

// grid (shares of the voxels, tiles): tiles of one fine-channel block are (pz, py) = (1, 1),
// (1, 0), (0, 1), (0, 0), the longest first.
// Waves per SIMD for the compiler to schedule for: with more, by its own choice, it issues fewer of the
// loads ahead (2 <- 8, 16 <- 32: 20 to 60 % slower). Left alone (8) it keeps them for 32 and 64 channels.
template <class WT, bool ROWS8, int CO>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(
    ROWS8 && CO == 64 ? 2 : 1, ROWS8 ? (CO == 8 ? 5 : 2) : CO == 16 ? (sizeof(WT) == 2 ? 6 : 4) : 8)))
conv_adjoint_kernel(AdjArgs a, const WT *__restrict__ Wt)
{
    constexpr int CIB = ROWS8 ? 2 : 8;
    __shared__ WT wsh[CO * CIB * 27 + 1];                // and a zero for the taps a row lacks
    const int ci0 = (ROWS8 ? 0 : blockIdx.y / 4) * CIB, nci = min(CIB, a.Ci - ci0);
    // Loads in batches: one at a time, their latency was most of the small layers' time.
    constexpr int N = CO * CIB * 27, NB = (N + 255) / 256, U = 18;
    const rsrc_t wr = make_rsrc(Wt, (int64_t)a.Co * a.Ci * 27 * sizeof(WT));
    if (threadIdx.x == 0) wsh[N] = (WT)0;
#pragma unroll
    for (int k0 = 0; k0 < NB; k0 += U) {
        WT v[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int t = (k0 + k) * 256 + threadIdx.x, co = t / (CIB * 27), r = t - co * (CIB * 27);
            v[k] = buf_w(wr, k0 + k < NB && co < a.Co && r < nci * 27,
                         (uint32_t)((co * a.Ci + ci0) * 27 + r), (WT)0);
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int t = (k0 + k) * 256 + threadIdx.x;
            if (t < N) wsh[t] = v[k];
        }
    }
    __syncthreads();
    if (ROWS8) adjoint_tile<WT, 1, 1, true, CO>(a, Wt, wsh, ci0);
    else if (blockIdx.y % 4 == 0) adjoint_tile<WT, 1, 1, false, CO>(a, Wt, wsh, ci0);
    else if (blockIdx.y % 4 == 1) adjoint_tile<WT, 1, 0, false, CO>(a, Wt, wsh, ci0);
    else if (blockIdx.y % 4 == 2) adjoint_tile<WT, 0, 1, false, CO>(a, Wt, wsh, ci0);
    else adjoint_tile<WT, 0, 0, false, CO>(a, Wt, wsh, ci0);
}

template <class WT>
hipError_t adjoint_launch(const AdjArgs &a, const WT *Wt, hipStream_t s)
{
    const unsigned gx = (unsigned)((a.groups + 4 * a.gpw - 1) / (4 * a.gpw));
    const unsigned gy = a.Ci <= 2 ? 1 : 4 * ((a.Ci + 7) / 8);
#define TDB_ADJ(ROWS8_, CO_)                                                                       \
    hipLaunchKernelGGL((conv_adjoint_kernel<WT, ROWS8_, CO_>), dim3(gx, gy), dim3(256), 0, s, a, Wt)
    if (a.Ci <= 2) {
        if (a.Co <= 8) TDB_ADJ(true, 8);
        else TDB_ADJ(true, 64);
    } else {
        if (a.Co <= 16) TDB_ADJ(false, 16);
        else if (a.Co <= 32) TDB_ADJ(false, 32);
        else TDB_ADJ(false, 64);
    }
#undef TDB_ADJ
    return hipGetLastError();
}

}  // namespace

bool conv_adjoint_ok(int B, int Ci, int Co, int D, int H, int W)
{
    const int64_t osp = (int64_t)(D / 2) * (H / 2) * (W / 2), P = (int64_t)B * osp;
    // More coarse channels would not fit the registers; an odd count would pair its last one
    // with a channel past the end.
    if (Co > 64 || (Co & 1) || P >= ((int64_t)1 << 31) - 65536) return false;
    // Two coarse channels use an eighth of the 16 that the registers and products are laid out for. This
    // kernel / the general one, batch 4, 64 <- 2 on 16^3 36 / 22 us, batch 16, 9 <- 2 28 / 20; but on 2 to 31
    // coarse voxels batch 32, 8 <- 2 on 2^3 8.4 / 12.5, on 3^3 9.0 / 9.9. Four channels are faster here, with
    // inputs not in the L2, but for 1 shape in 30 (by 17 % at most).
    if (Ci > 2 && Co <= 2 && (osp == 1 || osp >= 32)) return false;
    // A block's voxels (at most 1,024, see launch_conv_adjoint) and their neighbours lie in
    // these samples, addressed with 31-bit byte offsets.
    return (1023 / osp + 2) * Co * osp * 4 < ((int64_t)1 << 31);
}

hipError_t launch_conv_adjoint(bool bf16w, int B, int Ci, int Co, int D, int H, int W,
                               const float *dY, const void *Wt, const float *bias, int relu,
                               float *dX, hipStream_t s)
{
    const int64_t P = (int64_t)B * (D / 2) * (H / 2) * (W / 2);
    AdjArgs a = {B, Ci, Co, D, H, W, relu, (int)((P + 15) / 16), kAdjNG,
                 step_of(16 * kAdjNG, D / 2, H / 2, W / 2), dY, bias, dX};
    // Two 16-voxel groups go together; up to 16 per wave while 1,024 blocks remain.
    const int tiles = Ci <= 2 ? 1 : 4 * ((Ci + 7) / 8);
    while (a.gpw < 16 && (int64_t)a.groups * tiles / (8 * a.gpw) >= 1024) a.gpw *= 2;
    return bf16w ? adjoint_launch(a, (const uint16_t *)Wt, s)
                 : adjoint_launch(a, (const float *)Wt, s);
}

namespace {

// ---- forward (also the transposed convolution's input gradient) ---------------------------------
//
// Y[co][o] = sum over ci and taps of W[co][ci][tap] X[ci][2 o + tap - 1]: M = 16 coarse channels,
// N = 16 coarse voxels, one tile per wave at a time. Two orders of k, those of the kernels in
// nn.hip that this one stands in for:
//   by channel (CHUNK4 = false; conv_fwd_kernel): from bias[co], over ci, then the taps. Lane
//     group kq of product s has term 4 s + kq, so its channel and tap differ by lane: a table of
//     27 offsets per lane repeats every 27 products (4 channels).
//   by chunk (CHUNK4 = true; conv_mfma_kernel): from 0, over chunks of four channels, the taps,
//     the four channels; the bias last. Lane group kq is channel kq of the chunk.
// A block's weights lie in LDS as floats in product order (64 consecutive floats per product);
// lane l needs X at voxel l % 16: one buffer load per product straight from the caches. The
// padding is a load out of range; it can only be at the low edge of an axis (2 o + 1 is in
// range), so eight offsets per voxel (by chunk) or three bit masks per lane (by channel) hold
// all of it. The buffer starts one plane, row and element before X, which the masked taps alone
// would read, so that every tap is a positive offset. Batch 32: 20 / 21 us for 16 -> 32 and
// 32 -> 64, where the staged kernel's few blocks (one 4^3 box of all channels each) took 28 / 67;
// 32 -> 64 on 6^3 (rows not of fours) 19 us, where the vector kernel took 112. Bound by the chain
// of its products (216 of 32 cycles for 32 fine channels) and the first loads.
struct FwdArgs {
    int B, Ci, Co, D, H, W, relu, groups, gpw, NK;   // NK: products per tile
    Step st;
    const float *X, *bias;
    float *Y;
};
constexpr int kFwdMaxNK = 216;   // 32 fine channels: 55 KB of weights

template <class WT, bool CHUNK4, bool PAST, int NG>
__global__ void __launch_bounds__(256) conv_fwd_direct_kernel(FwdArgs a, const WT *__restrict__ Wt)
{
    extern __shared__ float wsh[];                       // [NK][64]: product, lane
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, kq = lane >> 4;
    const int OD = a.D / 2, OH = a.H / 2, OW = a.W / 2, HW = a.H * a.W;
    const int osp = OD * OH * OW, isp = a.D * HW;
    const int co0 = blockIdx.y * 16, K = a.Ci * 27;
    const rsrc_t wr = make_rsrc(Wt, (int64_t)a.Co * K * sizeof(WT));
    // Weights of the tile: thread t takes channel t / 16 of it, terms t % 16 + 16 i.
    for (int i0 = 0; i0 * 16 < K; i0 += 18) {
        WT v[18];
#pragma unroll
        for (int i = 0; i < 18; ++i) {
            const int k = (i0 + i) * 16 + (tid & 15), co = co0 + (tid >> 4);
            v[i] = buf_w(wr, k < K && co < a.Co, (uint32_t)(co * K + k), (WT)0);
        }
#pragma unroll
        for (int i = 0; i < 18; ++i) {
            const int k = (i0 + i) * 16 + (tid & 15);
            int s, q;
            if (CHUNK4) {
                const int ci = k / 27;
                s = (ci >> 2) * 27 + k - ci * 27;
                q = ci & 3;
            } else {
                s = k >> 2;
                q = k & 3;
            }
            if (s < a.NK) wsh[s * 64 + q * 16 + (tid >> 4)] = wt_f32(v[i]);
        }
    }
    __syncthreads();

    // By channel: this lane's terms of the 27 products of a period.
    int tap[CHUNK4 ? 1 : 27];
    uint32_t mz = 0, my = 0, mx = 0;
    // PAST (fine channels not in fours): terms of the last period past the last channel. Their weights
    // are zero, but what they would load is the next sample, whose infinities and NaNs times zero are
    // NaN. The mask costs 2 to 6 % (31 channels on a few voxels 20 %), so whole fours go without.
    const int last = (a.NK - 1) / 27;
    uint32_t past = 0;
    if (!CHUNK4) {
#pragma unroll
        for (int s = 0; s < 27; ++s) {
            const int k = 4 * s + kq, ci = k / 27, t = k - ci * 27;
            if (PAST) past |= (uint32_t)(4 * last + ci >= a.Ci) << s;
            tap[s] = 4 * (ci * isp + (t / 9) * HW + (t / 3 % 3) * a.W + t % 3);
            mz |= (uint32_t)(t / 9 == 0) << s;
            my |= (uint32_t)(t / 3 % 3 == 0) << s;
            mx |= (uint32_t)(t % 3 == 0) << s;
        }
    }
    const int g0 = (blockIdx.x * 4 + wave) * a.gpw, g1 = min(a.groups, g0 + a.gpw);
    const int64_t pb = (int64_t)blockIdx.x * 4 * a.gpw * 16;
    const int b0 = (int)(pb / osp);
    const int before = HW + a.W + 1;
    const rsrc_t xr = make_rsrc(a.X + (int64_t)b0 * a.Ci * isp - before,
                                ((int64_t)(a.B - b0) * a.Ci * isp + before) * 4);
    int vb[NG], vz[NG], vy[NG], vx[NG];
#pragma unroll
    for (int j = 0; j < NG; ++j) {
        const int o = (int)((int64_t)(g0 + j) * 16 + l16 - (int64_t)b0 * osp);
        vx[j] = o % OW;
        vy[j] = o / OW % OH;
        vz[j] = o / (OW * OH);
        vb[j] = vz[j] / OD;
        vz[j] -= vb[j] * OD;
    }
    float bq[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int co = co0 + 4 * kq + r;
        bq[r] = a.bias && co < a.Co ? a.bias[co] : 0.f;
    }
    constexpr int KC = 9, R = 8 / NG;                    // NK is padded to whole batches
    for (int g = g0; g < g1; g += NG) {
        uint32_t off[NG][8], inv[NG];
        f32x4 acc[NG];
#pragma unroll
        for (int j = 0; j < NG; ++j) {
            const bool in = g + j < g1 && b0 + vb[j] < a.B;
            const uint32_t o = 4u * (uint32_t)((vb[j] * a.Ci + (CHUNK4 ? kq : 0)) * isp +
                                               2 * vz[j] * HW + 2 * vy[j] * a.W + 2 * vx[j]);
            if (CHUNK4) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const bool ok = in & (!(e & 4) | (vz[j] != 0)) & (!(e & 2) | (vy[j] != 0)) &
                                    (!(e & 1) | (vx[j] != 0));
                    off[j][e] = ok ? o : kOut;
                }
            } else {
                off[j][0] = o;
                inv[j] = in ? (vz[j] ? 0u : mz) | (vy[j] ? 0u : my) | (vx[j] ? 0u : mx) : ~0u;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[j][r] = CHUNK4 ? 0.f : bq[r];
        }
        float v[R][KC][NG];
        // Batch c: products 9 c .. 9 c + 8, a third of a period, e = c % 3.
        auto load = [&](int c, int e, float (&d)[KC][NG]) {
            const uint32_t s0 = 16u * (uint32_t)isp * (uint32_t)(c / 3);
            if (PAST && e == 0) {                        // a period begins
#pragma unroll
                for (int j = 0; j < NG; ++j) inv[j] |= c == 3 * last ? past : 0u;
            }
#pragma unroll
            for (int k = 0; k < KC; ++k)
#pragma unroll
                for (int j = 0; j < NG; ++j) {
                    if (CHUNK4) {
                        const int t = 9 * e + k;         // the tap
                        const uint32_t so = s0 + 4u * (uint32_t)((t / 9) * HW + (t / 3 % 3) * a.W + t % 3);
                        d[k][j] = buf_f32(xr, off[j][(t / 9 == 0) * 4 + (t / 3 % 3 == 0) * 2 + (t % 3 == 0)], so);
                    } else {
                        const int t = 9 * e + k;         // product of the period
                        d[k][j] = buf_f32(xr, (inv[j] >> t & 1) ? kOut : off[j][0] + (uint32_t)tap[t], s0);
                    }
                }
        };
        const int nch = a.NK / KC;
        // Unrolled by lcm(3, R) batches so that every register index is a constant.
        constexpr int U = R * 3;
#pragma unroll
        for (int c = 0; c < R - 1; ++c)
            if (c < nch) load(c, c % 3, v[c]);
        for (int cb = 0; cb < nch; cb += U) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = cb + u;
                if (c < nch) {
                    if (c + R - 1 < nch) load(c + R - 1, (u + R - 1) % 3, v[(u + R - 1) % R]);
                    const float *w = wsh + c * KC * 64 + lane;
#pragma unroll
                    for (int k = 0; k < KC; ++k) {
                        const float wk = w[k * 64];
#pragma unroll
                        for (int j = 0; j < NG; ++j)
                            acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wk, v[u % R][k][j], acc[j], 0, 0, 0);
                    }
                }
            }
        }
#pragma unroll
        for (int j = 0; j < NG; ++j) {
            const bool in = g + j < g1 && b0 + vb[j] < a.B;
            float *d = a.Y + ((int64_t)(b0 + vb[j]) * a.Co + co0 + 4 * kq) * osp +
                       (vz[j] * OH + vy[j]) * OW + vx[j];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float y = CHUNK4 ? acc[j][r] + bq[r] : acc[j][r];
                if (a.relu && y < 0.f) y = 0.f;
                if (in && co0 + 4 * kq + r < a.Co) d[(int64_t)r * osp] = y;
            }
            advance(vb[j], vz[j], vy[j], vx[j], a.st, OD, OH, OW);
        }
    }
}

// The first layer's forward (at most two fine channels, rows of whole fours): the matrix cores
// would work on half-empty tiles and lanes would fetch every second element, so here a thread
// takes four voxels of a row and eight coarse channels: per fine row one pair of 16-byte loads
// (and the element before them, from the lane before where a wave starts a row), 96 multiply-adds
// against weights broadcast from LDS. The order is by channel, as above, from the bias. 26 us for
// 2 -> 8 at 64^3, batch 32 (two voxels per thread with an element per load: 49 us); the
// multiply-adds alone are 12 us.
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
template <class WT, bool SHIFT>
__global__ void __launch_bounds__(256) conv_fwd_first_kernel(FwdArgs a, const WT *__restrict__ Wt)
{
    __shared__ __attribute__((aligned(16))) float wsh[2 * 27 * 8];   // [ci][tap][co]
    const int tid = threadIdx.x, lane = tid & 63;
    const int OD = a.D / 2, OH = a.H / 2, OW = a.W / 2, HW = a.H * a.W, Q = OW / 4;
    const int osp = OD * OH * OW, isp = a.D * HW, qsp = osp / 4;
    const int co0 = blockIdx.y * 8, nco = min(8, a.Co - co0);
    for (int t = tid; t < a.Ci * 27 * 8; t += 256) {
        const int c = t & 7, r = t >> 3;
        wsh[t] = c < nco ? wt_f32(Wt[(int64_t)(co0 + c) * a.Ci * 27 + r]) : 0.f;
    }
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * 256;
    const int b0 = (int)(t0 / qsp);
    const int t = (int)(t0 - (int64_t)b0 * qsp) + tid;
    const int b = t / qsp, q = t - b * qsp;
    const int x = q % Q, y = q / Q % OH, z = q / (Q * OH);
    const bool in = b0 + b < a.B;
    const rsrc_t xr = make_rsrc(a.X + (int64_t)b0 * a.Ci * isp, (int64_t)(a.B - b0) * a.Ci * isp * 4);
    float acc[4][8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const float bc = a.bias && c < nco ? a.bias[co0 + c] : 0.f;
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v][c] = bc;
    }
    for (int ci = 0; ci < a.Ci; ++ci) {
        const uint32_t base = 4u * (uint32_t)((b * a.Ci + ci) * isp + 2 * z * HW + 2 * y * a.W + 8 * x);
        u32x4 lo[9], hi[9];
        float l[9];
#pragma unroll
        for (int r = 0; r < 9; ++r) {
            const bool ok = in & ((r / 3 != 0) | (z != 0)) & ((r % 3 != 0) | (y != 0));
            const uint32_t o = ok ? base + 4 * ((r / 3 - 1) * HW + (r % 3 - 1) * a.W) : kOut;
            lo[r] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, o, 0, 0));
            hi[r] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, ok ? o + 16 : kOut, 0, 0));
            if (!SHIFT) l[r] = buf_f32(xr, ok & (x != 0) ? o - 4 : kOut);
        }
#pragma unroll
        for (int r = 0; r < 9; ++r) {
            if (SHIFT) {
                l[r] = __uint_as_float(__builtin_amdgcn_update_dpp(0, hi[r].w, 0x138, 0xf, 0xf, true));   // wave_shr:1
                l[r] = x ? l[r] : 0.f;
            }
            const float e[9] = {l[r], __uint_as_float(lo[r].x), __uint_as_float(lo[r].y),
                                __uint_as_float(lo[r].z), __uint_as_float(lo[r].w),
                                __uint_as_float(hi[r].x), __uint_as_float(hi[r].y),
                                __uint_as_float(hi[r].z), __uint_as_float(hi[r].w)};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const f32x4 *w = reinterpret_cast<const f32x4 *>(wsh + ((ci * 9 + r) * 3 + k) * 8);
                const f32x4 w0 = w[0], w1 = w[1];
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int c = 0; c < 8; ++c)
                        acc[v][c] = __builtin_fmaf(c < 4 ? w0[c & 3] : w1[c & 3], e[2 * v + k], acc[v][c]);
            }
        }
    }
    if (!in) return;
    float *d = a.Y + ((int64_t)(b0 + b) * a.Co + co0) * osp + 4 * q;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        if (c >= nco) break;
        f32x4_u o;
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = a.relu && acc[v][c] < 0.f ? 0.f : acc[v][c];
        *reinterpret_cast<f32x4_u *>(d + (int64_t)c * osp) = o;
    }
}

template <class WT>
hipError_t fwd_first_launch(const FwdArgs &a, const WT *Wt, hipStream_t s)
{
    const int64_t T = (int64_t)a.B * (a.D / 2) * (a.H / 2) * (a.W / 8);
    const dim3 grid((unsigned)((T + 255) / 256), (unsigned)((a.Co + 7) / 8));
    if (64 % (a.W / 8) == 0)
        hipLaunchKernelGGL((conv_fwd_first_kernel<WT, true>), grid, dim3(256), 0, s, a, Wt);
    else
        hipLaunchKernelGGL((conv_fwd_first_kernel<WT, false>), grid, dim3(256), 0, s, a, Wt);
    return hipGetLastError();
}

template <class WT, bool CHUNK4, bool PAST>
hipError_t fwd_launch(FwdArgs a, const WT *Wt, hipStream_t s)
{
    const int tiles = (a.Co + 15) / 16;
    // Two groups of voxels share a product's weights where there are waves enough; fewer leave
    // the small layers' chains side by side.
    const bool two = (int64_t)a.groups * tiles >= 8192;
    a.gpw = two ? 2 : 1;
    while (a.gpw < 16 && (int64_t)a.groups * tiles / (8 * a.gpw) >= 1024) a.gpw *= 2;
    a.st = step_of(two ? 32 : 16, a.D / 2, a.H / 2, a.W / 2);
    const dim3 grid((unsigned)((a.groups + 4 * a.gpw - 1) / (4 * a.gpw)), (unsigned)tiles);
    const size_t lds = (size_t)a.NK * 64 * sizeof(float);
    if (two)
        hipLaunchKernelGGL((conv_fwd_direct_kernel<WT, CHUNK4, PAST, 2>), grid, dim3(256), lds, s, a, Wt);
    else
        hipLaunchKernelGGL((conv_fwd_direct_kernel<WT, CHUNK4, PAST, 1>), grid, dim3(256), lds, s, a, Wt);
    return hipGetLastError();
}

// Products per tile, in whole batches of nine.
int fwd_products(int Ci, bool chunk4)
{
    const int n = chunk4 ? Ci / 4 * 27 : (Ci * 27 + 3) / 4;
    return (n + 8) / 9 * 9;
}

}  // namespace

// Times of the forward kernels in us, fitted to 1,400 shapes and more of each weight type with inputs not
// in the L2 (within 5 to 13 %): the rule below compares them. A chain of dependent steps while the waves
// fit the chip side by side, else the rate of its products. groups: groups of 16 voxels; nt, nb: tiles
// of 16 (blocks of 8 or 16) coarse channels.
static double direct_us(double groups, int nt, int NK, int Ci, int64_t isp, int OW, bool chunk4)
{
    const bool big = groups * nt >= 8192;                // two groups per wave
    if (!chunk4) return 5.3 + .125 * Ci + NK * std::max(Ci % 4 ? .03 : .021, groups * nt * 53e-6);
    // Channels a multiple of 2 KB apart lie on the same few L2 channels.
    const bool same = isp % 512 == 0;
    const double chain = NK * (OW < 4 ? .054 : same ? .048 : .036) + .17 * Ci;
    const double rate = groups * nt * NK * (big ? 44e-6 : 54e-6) * (same ? 1.22 : 1);
    return 7.5 + .07 * nt + std::cbrt(chain * chain * chain + rate * rate * rate);
}
// conv_mfma_kernel: its boxes of voxels, npb of a sample in turn per block, a stage per four fine
// channels, most of it the wait for its loads; BF16 weights are widened on their way into LDS.
static double staged_us(bool bf16w, int B, int Ci, int OD, int OH, int OW, int nt)
{
    static const double stage[2][3][4] = {
        {{1.1, 1.7, 2.4, 3.15}, {1.8, 3.25, 4.5, 5.7}, {2.0, 3.4, 4.75, 6.2}},     // float weights
        {{1.7, 3.3, 4.7, 6.0}, {2.4, 4.6, 6.45, 8.25}, {2.4, 4.5, 6.4, 8.3}}};
    const int box = OW >= 16 ? 2 : OW >= 8 ? 1 : 0, td = box == 2 ? 2 : 4, tw = 4 << box, stages = Ci / 4;
    const int64_t T = (int64_t)((OD + td - 1) / td) * ((OH + 3) / 4) * ((OW + tw - 1) / tw);
    const int npb = T >= 64 ? 4 : T >= 16 ? 2 : 1;
    const double boxes = (double)B * T * td * 4 * tw / 16384, chain = npb * stages * stage[bf16w][box][std::min(nt, 4) - 1];
    const double start = bf16w ? 5.8 + 1.2 * nt : 6.1 + .65 * nt;
    return start + std::max(chain + (bf16w ? .75 : 1.5) * npb, boxes * stages * nt);
}
// conv_fwd_kernel.
static double vector_us(double P, int Ci, int Co, bool wide)
{
    const int cb = wide ? 16 : 8, nb = (Co + cb - 1) / cb;
    return 3.5 + std::hypot(Ci * (.98 + .12 * cb), Ci * P * nb * (8 + cb) * 1e-6);
}

bool conv_fwd_direct_ok(bool bf16w, int B, int Ci, int Co, int D, int H, int W, bool chunk4)
{
    const int OD = D / 2, OH = H / 2, OW = W / 2;
    const int64_t osp = (int64_t)OD * OH * OW, P = (int64_t)B * osp;
    const int NK = fwd_products(Ci, chunk4);
    if (P >= ((int64_t)1 << 31) - 65536) return false;
    // A block's voxels (at most 1,024) lie in these samples, addressed with 31-bit byte offsets.
    if (((1023 / osp + 2) * Ci + 4) * (8 * osp) * 4 >= ((int64_t)1 << 31)) return false;
    // The first layer's kernel takes rows of whole fours. Other rows of two channels leave the lanes of
    // the matrix products half idle (72 us against 49 for the vector kernel, 2 -> 8 at 64^3).
    if (Ci <= 2) return W % 8 == 0;
    if (NK > kFwdMaxNK || Co > 1024) return false;
    // By chunk, rows of 16 and more voxels fill the staged kernel's boxes (24 us against 26, 8 -> 16 at
    // batch 32). Otherwise the estimates decide, with a margin for their errors: short sums of few
    // channels and many samples whose boxes are full go to the other kernels (float weights, 12 -> 16 on
    // 4^3, batch 100: staged 8 / direct 12; 28 -> 8 on 8^3, batch 100: 29 / 54; 3 -> 24 on 10 x 10 x 11:
    // vector 25 / 36), batch 32, BF16 weights, 16 -> 32 on 8^3 and 32 -> 64 on 4^3 stay (28 / 20 and 67 / 21).
    const double direct = direct_us((double)((P + 15) / 16), (Co + 15) / 16, NK, Ci, 8 * osp, OW, chunk4);
    if (chunk4) return OW % 16 != 0 && 1.05 * direct < staged_us(bf16w, B, Ci, OD, OH, OW, (Co + 15) / 16);
    return 1.15 * direct < vector_us((double)P, Ci, Co, Co >= 16 && (int64_t)D * H * W <= 4096);
}

hipError_t launch_conv_fwd_direct(bool bf16w, bool chunk4, int B, int Ci, int Co, int D, int H,
                                  int W, const float *X, const void *Wt, const float *bias, int relu,
                                  float *Y, hipStream_t s)
{
    const int64_t P = (int64_t)B * (D / 2) * (H / 2) * (W / 2);
    const FwdArgs a = {B, Ci, Co, D, H, W, relu, (int)((P + 15) / 16), 0, fwd_products(Ci, chunk4),
                       {}, X, bias, Y};
    if (Ci <= 2 && !chunk4)
        return bf16w ? fwd_first_launch(a, (const uint16_t *)Wt, s) : fwd_first_launch(a, (const float *)Wt, s);
    const auto launch = [&](auto *W) {
        using WT = std::remove_cv_t<std::remove_pointer_t<decltype(W)>>;
        return chunk4        ? fwd_launch<WT, true, false>(a, W, s)
               : Ci % 4 == 0 ? fwd_launch<WT, false, false>(a, W, s)
                             : fwd_launch<WT, false, true>(a, W, s);
    };
    return bf16w ? launch((const uint16_t *)Wt) : launch((const float *)Wt);
}

namespace {

// ---- linear layers of a small batch --------------------------------------------------------------
//
// C[m][n] = act(bias[n] + sum over k of A[m][k] W(k, n)), W [N][K] (forward) or [K][N] (input
// gradient, KN). The order of linear_mfma_kernel, bit for bit: two chains over k, wave kh of a
// pair taking of every 64 terms 16 kh + s and 32 + 16 kh + s alternately (s = 0 .. 15), added at
// the end. That kernel's 64 x 64 tiles leave a batch of 32 eight blocks; here a pair of waves
// takes 16 rows and NT x 16 columns straight from the caches, so the same batch runs 64 to 256
// pairs side by side, each as long as its chain of products. In product p of 64 terms lane group
// kq holds term 32 (kq & 1) + 2 p + (kq >> 1): it loads its 16 consecutive terms and uses every
// second. KN: lane n holds columns 4 (l % 16) .. + 3 (NT = 4), one for each of four tiles.
// Batch 32: 33 / 13 us forward (4096 -> 512 / 512 -> 4096; 128 / 19 for the 64 x 64 tiles), 16 / 31
// us for the input gradients (25 / 171). The long chains (4,096 terms) run at half a microsecond
// per 64 terms, five times their products: every row starts at a multiple of 8 KB, so the blocks,
// all at the same k, read from few of the L2's channels at a time.
template <class WT>
struct Frag;   // 16 consecutive values, loaded in fours
template <>
struct Frag<uint16_t> {
    u32x2_t v[4];
    __device__ void load4(rsrc_t r, int i, uint32_t off)
    {
        v[i] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(r, off, 8 * i, 0));
    }
    // Element 2 p or (odd) 2 p + 1.
    __device__ float get(int p, bool odd) const
    {
        const uint32_t u = v[p >> 1][p & 1];
        return __uint_as_float(odd ? u & 0xffff0000u : u << 16);
    }
};
template <>
struct Frag<float> {
    u32x4 v[4];
    __device__ void load4(rsrc_t r, int i, uint32_t off)
    {
        v[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 16 * i, 0));
    }
    __device__ float get(int p, bool odd) const
    {
        const uint32_t a = v[p >> 1][2 * (p & 1)], b = v[p >> 1][2 * (p & 1) + 1];
        return __uint_as_float(odd ? b : a);
    }
};

struct LinArgs {
    int M, N, K, relu;
    const float *A, *bias;
    float *C;
};

template <class WT, bool KN, int NT>
__global__ void __launch_bounds__(128) linear_small_kernel(LinArgs a, const WT *__restrict__ Wt)
{
    __shared__ f32x4 other[NT][64];
    const int lane = threadIdx.x & 63, kh = threadIdx.x >> 6, l16 = lane & 15, kq = lane >> 4;
    const int m0 = blockIdx.y * 16, n0 = blockIdx.x * 16 * NT;
    const rsrc_t ar = make_rsrc(a.A, (int64_t)a.M * a.K * 4);
    const rsrc_t wr = make_rsrc(Wt, (int64_t)a.N * a.K * sizeof(WT));
    const int m = m0 + l16, n = KN ? n0 + NT * l16 : n0 + l16;
    const bool odd = kq >> 1;
    const int kb = 16 * kh + 32 * (kq & 1);              // first of this lane's 16 terms of 64
    constexpr int R = NT == 4 ? 4 : 8;                   // 64-term chunks in flight
    Frag<float> fa[R];
    Frag<WT> fb[KN ? 1 : R];
    uint32_t kw[KN ? R : 1][8][NT];                      // KN: the lane's eight terms, raw
    const int nch = (a.K + 63) / 64;
    auto load = [&](int c, int u) {
        const int k = 64 * c + kb;
        // K is a multiple of 4: a group of four terms is inside or outside as a whole.
        const uint32_t e = (uint32_t)m * (uint32_t)a.K + k;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            fa[u].load4(ar, i, m < a.M && k + 4 * i < a.K ? 4 * e : kOut);
        if (!KN) {
            const uint32_t w = (uint32_t)n * (uint32_t)a.K + k;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                fb[u].load4(wr, i, n < a.N && k + 4 * i < a.K ? (uint32_t)sizeof(WT) * w : kOut);
        } else {
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const int kk = k + 2 * p + (odd ? 1 : 0);
                const uint32_t w = (uint32_t)kk * (uint32_t)a.N + n;
                const bool in = kk < a.K && n < a.N;
                if (NT == 4 && sizeof(WT) == 2) {
                    const u32x2_t v = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(
                        wr, in ? 2 * w : kOut, 0, 0));
                    kw[u][p][0] = v.x;
                    kw[u][p][1 % NT] = v.y;
                } else if (NT == 4) {
                    const u32x4 v = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                        wr, in ? 4 * w : kOut, 0, 0));
#pragma unroll
                    for (int t = 0; t < NT; ++t) kw[u][p][t] = v[t % 4];
                } else if (sizeof(WT) == 2) {
                    kw[u][p][0] = (uint32_t)buf_w(wr, in, w, (WT)0);
                } else {
                    kw[u][p][0] = __float_as_uint((float)buf_w(wr, in, w, (WT)0));
                }
            }
        }
    };
    // Column t of term p of chunk slot u.
    auto bval = [&](int u, int p, int t) {
        if (!KN) return fb[KN ? 0 : u].get(p, odd);
        if (sizeof(WT) == 4) return __uint_as_float(kw[KN ? u : 0][p][t]);
        if (NT == 1) return __uint_as_float(kw[KN ? u : 0][p][0] << 16);
        const uint32_t v = kw[KN ? u : 0][p][(t >> 1) % NT];
        return __uint_as_float(t & 1 ? v & 0xffff0000u : v << 16);
    };
    f32x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    // Loads are unconditional (zeros past the end), so that each wait counts those in flight.
#pragma unroll
    for (int u = 0; u < R - 1; ++u) load(u, u);
    for (int cb = 0; cb < nch; cb += R) {
#pragma unroll
        for (int u = 0; u < R; ++u) {
            load(cb + u + R - 1, (u + R - 1) % R);
            if (cb + u < nch) {
#pragma unroll
                for (int p = 0; p < 8; ++p) {
                    const float av = fa[u].get(p, odd);
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bval(u, p, t), acc[t], 0, 0, 0);
                }
            }
        }
    }
    if (kh) {
#pragma unroll
        for (int t = 0; t < NT; ++t) other[t][lane] = acc[t];
    }
    __syncthreads();
    if (kh) return;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int nn = KN ? n + t : n0 + l16;
        if (nn >= a.N) continue;
        const f32x4 o = other[t][lane];
        const float bn = a.bias ? a.bias[nn] : 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int mm = m0 + 4 * kq + r;
            float v = acc[t][r] + o[r];
            v += bn;
            if (a.relu && v < 0.f) v = 0.f;
            if (mm < a.M) a.C[(int64_t)mm * a.N + nn] = v;
        }
    }
}

// dW[j][i] = sum over b of dY[b][j] X[b][i], b ascending as in linear_bwd_weight_kernel, and
// dbias[j]. A wave takes 16 rows j and 64 columns i: four products per four samples, lane n
// holding columns 4 (l % 16) .. + 3 as one 16-byte load; dbias is a fifth product with ones, in
// the first columns' waves. Bound by the writes of dW: 5 us for 512 x 4096 at batch 32 (one thread
// per element: 32 us).
__global__ void __launch_bounds__(256) linear_wgrad_kernel(int B, int In, int Out,
                                                           const float *__restrict__ X,
                                                           const float *__restrict__ dY,
                                                           float *__restrict__ dW,
                                                           float *__restrict__ dbias)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, kq = lane >> 4;
    const int i = (blockIdx.x * 4 + wave) * 64 + 4 * l16, j0 = blockIdx.y * 16;
    const rsrc_t xr = make_rsrc(X, (int64_t)B * In * 4), yr = make_rsrc(dY, (int64_t)B * Out * 4);
    f32x4 acc[4], ab = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = ab;
    const bool first = blockIdx.x == 0 && wave == 0 && dbias;
    constexpr int U = 8;                                 // loads of 32 samples before their use
    for (int b0 = 0; b0 < B; b0 += 4 * U) {
        u32x4 x[U];
        float y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int b = b0 + 4 * u + kq;
            y[u] = buf_f32(yr, b < B && j0 + l16 < Out ? 4u * ((uint32_t)b * Out + j0 + l16) : kOut);
            x[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                xr, b < B && i < In ? 4u * ((uint32_t)b * In + i) : kOut, 0, 0));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(y[u], __uint_as_float(x[u][t]), acc[t], 0, 0, 0);
            if (first) ab = __builtin_amdgcn_mfma_f32_16x16x4f32(y[u], 1.f, ab, 0, 0, 0);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int j = j0 + 4 * kq + r;
        if (j >= Out) continue;
        if (i < In)
            *reinterpret_cast<f32x4_u *>(dW + (int64_t)j * In + i) =
                (f32x4_u){acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
        if (first && l16 == 0) dbias[j] = ab[r];
    }
}

template <class WT, bool KN>
hipError_t linear_small_launch(const LinArgs &a, const WT *Wt, hipStream_t s)
{
    const unsigned my = (unsigned)((a.M + 15) / 16);
    // Four column tiles per wave where that still gives 128 pairs (the weights' rows are read in
    // wider pieces), one otherwise.
    if (KN && (int64_t)my * ((a.N + 63) / 64) >= 128)
        hipLaunchKernelGGL((linear_small_kernel<WT, KN, KN ? 4 : 1>), dim3((unsigned)((a.N + 63) / 64), my),
                           dim3(128), 0, s, a, Wt);
    else
        hipLaunchKernelGGL((linear_small_kernel<WT, KN, 1>), dim3((unsigned)((a.N + 15) / 16), my),
                           dim3(128), 0, s, a, Wt);
    return hipGetLastError();
}

}  // namespace

bool linear_small_ok(bool kn, int M, int N, int K)
{
    if ((int64_t)M * K * 4 >= ((int64_t)1 << 31) || (int64_t)N * K * 4 >= ((int64_t)1 << 31)) return false;   // 31-bit byte offsets
    // While the pairs of waves run side by side (256 CUs, a second round hidden by long chains) a
    // launch takes as long as one chain, which the 64 x 64 tiles walk at a third of the pace; with
    // more of them the tiles' reuse wins. 64 x 64 tiles / pairs, forward: 256 pairs, K = 68: 5.8 / 4.8
    // us, K = 4,096: 88 / 33; 512 pairs, K = 256: 8.4 / 8.8, K = 320: 9.7 / 9.6, K = 4,096: 87 / 62; 1,024
    // pairs, K = 4,096: 89 / 120. A chain of one chunk of 64 pays only for rows past the first tile:
    // 4 rows 4.2 / 4.7, 32 rows 5.3 / 4.8.
    const int64_t my = (M + 15) / 16;
    if (!kn) return (K > 64 || M >= 32) && my * ((N + 15) / 16) <= (K > 256 ? 512 : 256);
    // Input gradient, in groups of 64 columns (BF16 weights, the tiles' better type): 256 groups, K = 256:
    // 10.9 / 9.7; 512, K = 256: 11.2 / 12.9, K = 1,024: 35 / 31, K = 4,096: 150 / 104; 1,024, K = 1,024 (float)
    // 34 / 46. Two chunks of 64: 4 rows 5.9 / 5.9, 32 rows in pairs of one column tile 7.1 / 6.2, of four (128
    // groups and more) 6.7 / 8.0.
    const int64_t groups = my * ((N + 63) / 64);
    return K > 128 ? groups <= (K > 256 ? 512 : 256) : K > 64 && M >= 32 && groups < 128;
}

hipError_t launch_linear_small(bool bf16w, bool kn, int M, int N, int K, const float *A, const void *Wt,
                               const float *bias, int relu, float *C, hipStream_t s)
{
    const LinArgs a = {M, N, K, relu, A, bias, C};
    if (bf16w)
        return kn ? linear_small_launch<uint16_t, true>(a, (const uint16_t *)Wt, s)
                  : linear_small_launch<uint16_t, false>(a, (const uint16_t *)Wt, s);
    return kn ? linear_small_launch<float, true>(a, (const float *)Wt, s)
              : linear_small_launch<float, false>(a, (const float *)Wt, s);
}

bool linear_wgrad_ok(int B, int In, int Out)
{
    return In % 4 == 0 && (int64_t)B * std::max(In, Out) * 4 < ((int64_t)1 << 31);
}

hipError_t launch_linear_wgrad(int B, int In, int Out, const float *X, const float *dY, float *dW,
                               float *dbias, hipStream_t s)
{
    hipLaunchKernelGGL(linear_wgrad_kernel, dim3((unsigned)((In + 255) / 256), (unsigned)((Out + 15) / 16)),
                       dim3(256), 0, s, B, In, Out, X, dY, dW, dbias);
    return hipGetLastError();
}

}  // namespace tdb
