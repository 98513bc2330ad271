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

// ---- weight gradient ------------------------------------------------------------------------
//
// dW[co][ci][tap] = sum over (sample, coarse voxel o) of dY[co][o] X[ci][2 o + tap - 1]. Grid
// (chunks of kWgChunkF positions, Ci, ceil(Co / CB)); a thread takes every 256th position of
// the chunk, CB coarse channels and all 27 taps (and the sum of dY, tap 27), 28 CB sums in
// registers. Per position the fine values come as nine pairs (x = 2 ow, 2 ow + 1) by buffer
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

struct WgStep {   // 256 positions as (samples, z, y, x)
    int b, z, y, x;
};

template <bool SHIFT>
__global__ void __launch_bounds__(256, 3) conv_wgrad_kernel(int B, int Ci, int Co, int D, int H,
                                                            int W, WgStep st,
                                                            const float *__restrict__ X,
                                                            const float *__restrict__ dY,
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
        for (int c = 0; c < CB; ++c) {
#pragma unroll
            for (int r = 0; r < 27; ++r) acc[c * 28 + r] = __builtin_fmaf(g[c], v[r / 3][r % 3], acc[c * 28 + r]);
            acc[c * 28 + 27] += g[c];
        }
        x += st.x;
        y += st.y;
        z += st.z;
        b += st.b;
        if (x >= OW) { x -= OW; ++y; }
        if (y >= OH) { y -= OH; ++z; }
        if (z >= OD) { z -= OD; ++b; }
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
                             const float *dY, float *dW, float *dbias, float *ws, hipStream_t s)
{
    const int OD = D / 2, OH = H / 2, OW = W / 2;
    const int64_t P = (int64_t)B * OD * OH * OW;
    const int chunks = (int)((P + kWgChunkF - 1) / kWgChunkF);
    const WgStep st = {256 / (OW * OH * OD), 256 / (OW * OH) % OD, 256 / OW % OH, 256 % OW};
    const dim3 grid((unsigned)chunks, (unsigned)Ci, (unsigned)((Co + kWgCBF - 1) / kWgCBF));
    if (64 % OW == 0)
        hipLaunchKernelGGL((conv_wgrad_kernel<true>), grid, dim3(256), 0, s, B, Ci, Co, D, H, W, st,
                           X, dY, ws);
    else
        hipLaunchKernelGGL((conv_wgrad_kernel<false>), grid, dim3(256), 0, s, B, Ci, Co, D, H, W, st,
                           X, dY, ws);
    const int64_t N = (int64_t)Co * Ci * 28;
    hipLaunchKernelGGL(conv_wgrad_final_kernel, dim3((unsigned)((N + 31) / 32)), dim3(512), 0, s,
                       chunks, Ci, N, (const float *)ws, dW, dbias);
    return hipGetLastError();
}

}  // namespace tdb
