// query_parts.hpp — one query's counts, row boxes and moments from the partials its pack blocks
// left, by one wave: a kernel of its own (pack.hip), or a block of the exact scan (scan.hip).
#pragma once

#include <limits.h>

#include "common.hpp"
#include "internal.hpp"

namespace tdb {

// A row box as [z0, z1) x [y0, y1) from the extreme rows (all zero when there is none).
__device__ __forceinline__ void write_box(int32_t *bx, int zlo, int zhi, int ylo, int yhi)
{
    if (zhi < 0) {
        bx[0] = bx[1] = bx[2] = bx[3] = 0;
    } else {
        bx[0] = zlo;
        bx[1] = zhi + 1;
        bx[2] = ylo;
        bx[3] = yhi + 1;
    }
}

// Combine the kQueryParts partials of query q (threads 0 .. 63).
__device__ __forceinline__ void sum_query_parts(const QueryPart *__restrict__ qpart, int q,
                                                uint32_t *__restrict__ acnt,
                                                int32_t *__restrict__ qbox,
                                                uint64_t *__restrict__ qmom,
                                                int32_t *__restrict__ qtbox)
{
    uint32_t a = 0, b = 0;
    int zlo = INT_MAX, zhi = -1, ylo = INT_MAX, yhi = -1;
    int tzlo = INT_MAX, tzhi = -1, tylo = INT_MAX, tyhi = -1;
    uint64_t sx = 0, sy = 0, sz = 0;
    for (int i = threadIdx.x; i < kQueryParts; i += 64) {
        const QueryPart &p = qpart[(int64_t)q * kQueryParts + i];
        a += p.cnt[0];
        b += p.cnt[1];
        zlo = min(zlo, p.box[0]);
        zhi = max(zhi, p.box[1]);
        ylo = min(ylo, p.box[2]);
        yhi = max(yhi, p.box[3]);
        tzlo = min(tzlo, p.tbox[0]);
        tzhi = max(tzhi, p.tbox[1]);
        tylo = min(tylo, p.tbox[2]);
        tyhi = max(tyhi, p.tbox[3]);
        sx += p.mom[0];
        sy += p.mom[1];
        sz += p.mom[2];
    }
    a = wave_sum(a);
    b = wave_sum(b);
    zlo = wave_min(zlo);
    ylo = wave_min(ylo);
    zhi = wave_max(zhi);
    yhi = wave_max(yhi);
    tzlo = wave_min(tzlo);
    tylo = wave_min(tylo);
    tzhi = wave_max(tzhi);
    tyhi = wave_max(tyhi);
    sx = wave_sum64(sx);
    sy = wave_sum64(sy);
    sz = wave_sum64(sz);
    if (threadIdx.x == 0) {
        acnt[2 * q] = a;
        acnt[2 * q + 1] = b;
        write_box(qbox + 4 * q, zlo, zhi, ylo, yhi);
        if (qtbox) write_box(qtbox + 4 * q, tzlo, tzhi, tylo, tyhi);
        uint64_t *m = qmom + 4 * q;
        m[0] = sx;
        m[1] = sy;
        m[2] = sz;
        m[3] = a;
    }
}

}  // namespace tdb
