// Demons iterations on a region held by one workgroup (multi-resolution demons,
// arXiv:1907.05993 section 1, Eq. (1)): the device code shared by the
// level-resident kernel (the region is a whole coarse level) and the tile
// kernel (the region is an output tile with a halo).
//
// A wavefront owns 64 consecutive columns of RPT consecutive rows (lane =
// column) and keeps, in registers, the field of its pixels and what an
// iteration needs of the reference there: its value and its gradient, which do
// not change from one iteration to the next.  An iteration is then
//   1. the bilinear gathers of the test pattern for all of the rows (issued
//      together), the force, v = u + a grad R / (|grad R|^2 + a^2);
//   2. horizontal Gaussian taps across the lanes: the neighbours' v come by
//      shifts of the wavefront by one lane (DPP, in the vector ALU), so the
//      horizontal pass needs no LDS and no barrier; the end lanes keep their
//      own value, which is the replicated border where the wavefront ends at
//      the image's border;
//   3. the filtered rows into one of two LDS buffers, one workgroup barrier, and
//      the vertical taps over the rows around the wavefront's own.
// Every pixel's arithmetic is that of the row-marching kernels (gradient,
// gather, blend, reciprocal, tap order), so the fields are equal bit for bit.
#pragma once

#include "dev_util.h"

namespace ebsd {

// src of the previous / next lane; `end` in the first / last lane.
__device__ __forceinline__ float from_prev(float src, float end)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, end),
                                                                 __builtin_bit_cast(int, src), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float from_next(float src, float end)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, end),
                                                                 __builtin_bit_cast(int, src), 0x130, 0xf, 0xf, false));
}

// Horizontal taps of v across the lanes of a wavefront (all lanes active), C
// consecutive columns per lane, in place; the end columns repeat outside.
template <int C, int RAD>
__device__ __forceinline__ void lane_taps(float (&v)[C], const Taps& tp)
{
    float e[C + 2 * RAD];
#pragma unroll
    for (int c = 0; c < C; c++) e[RAD + c] = v[c];
#pragma unroll
    for (int j = 1; j <= RAD; j++) {
        // the columns j to the left of the first and j to the right of the last: C columns
        // further in for each lane passed
        e[RAD - j] = from_prev(j <= C ? v[j <= C ? C - j : 0] : e[RAD - j + C], v[0]);
        e[RAD + C - 1 + j] = from_next(j <= C ? v[j <= C ? j - 1 : 0] : e[RAD - 1 + j], v[C - 1]);
    }
#pragma unroll
    for (int c = 0; c < C; c++) {
        float a = 0.0f;
#pragma unroll
        for (int j = 0; j <= 2 * RAD; j++) a = fmaf(tp.w[j], e[c + j], a);
        v[c] = a;
    }
}
template <int RAD>
__device__ __forceinline__ float lane_taps(float v, const Taps& tp)
{
    float t[1] = {v};
    lane_taps<1, RAD>(t, tp);
    return t[0];
}

// A wavefront's rows of a region: rows y .. y + RPT - 1 of the level at column
// x (both may lie outside the image; values there are those of the nearest
// pixel and only ever feed pixels that are not written).
template <int RPT>
struct RegionRows {
    float ux[RPT], uy[RPT];          // field
    float r[RPT], gx[RPT], gy[RPT];  // reference and its gradient
};

// R, u: the level's reference and field (u: 2 channels of h w).
template <int RPT>
__device__ __forceinline__ void region_load(RegionRows<RPT>& s, const float* __restrict__ Rg,
                                            const float* __restrict__ ug, int h, int w, int x, int y)
{
    const EBSD_GLOBAL float* __restrict__ R = gptr(Rg);
    const EBSD_GLOBAL float* __restrict__ u = gptr(ug);
    const int xc = clampi(x, 0, w - 1);
    const int xm = max(xc - 1, 0), xp = min(xc + 1, w - 1);
    const float sx = (xp - xm == 2) ? 0.5f : 1.0f;
#pragma unroll
    for (int k = 0; k < RPT; k++) {
        const int yc = clampi(y + k, 0, h - 1);
        const int ym = max(yc - 1, 0), yp = min(yc + 1, h - 1);
        const float sy = (yp - ym == 2) ? 0.5f : 1.0f;
        const int o = yc * w + xc;
        s.ux[k] = u[o];
        s.uy[k] = u[(int64_t)h * w + o];
        s.r[k] = R[o];
        s.gx[k] = (R[yc * w + xp] - R[yc * w + xm]) * sx;
        s.gy[k] = (R[yp * w + xc] - R[ym * w + xc]) * sy;
    }
}

// The force at one pixel: v = u + du from the gathered test value wv.
__device__ __forceinline__ void demons_force(float wv, float r, float gx, float gy, float ux, float uy, float& vx,
                                             float& vy)
{
    const float a = r - wv;
    const float den = fmaf(gx, gx, fmaf(gy, gy, a * a));
    vx = ux;
    vy = uy;
    if (den > 1e-9f) {
        const float q = a * __builtin_amdgcn_rcpf(den);
        vx = fmaf(q, gx, ux);
        vy = fmaf(q, gy, uy);
    }
}

// Gather of a bilinear cell from an LDS copy of the level (at least 2 x 2 px).
struct LdsImage {
    const float* t;
    int w;
};
__device__ __forceinline__ Bilin region_gather(const LdsImage& T, const BilGeom& g, float x, float y)
{
    Bilin b;
    const float xc = fminf(fmaxf(x, 0.0f), g.wm1);
    const float yc = fminf(fmaxf(y, 0.0f), g.hm1);
    const float xf = fminf(floorf(xc), g.wm2), yf = fminf(floorf(yc), g.hm2);
    b.fx = xc - xf;
    b.fy = yc - yf;
    const int o = (int)fmaf(yf, g.wf, xf);
    b.v00 = T.t[o];
    b.v01 = T.t[o + 1];
    b.v10 = T.t[o + T.w];
    b.v11 = T.t[o + T.w + 1];
    return b;
}
__device__ __forceinline__ Bilin region_gather(const GatherBase& T, const BilGeom& g, float x, float y)
{
    return bilinear_issue_g(T, g, x, y);
}

// Phases 1 and 2 for a wavefront's rows; the filtered rows go to hrow[k * 64]
// (the wavefront's first row at this lane).  fix: the lane whose v this lane
// takes (a lane outside the image takes the border column's), < 0 where the
// whole wavefront keeps its own.
template <int RAD, int RPT, class Img>
__device__ __forceinline__ void region_rows(const RegionRows<RPT>& s, const Img& T, const BilGeom& g, const Taps& tp,
                                            float x, float y, bool fix, int fix_lane, float2* __restrict__ hrow)
{
    Bilin b[RPT];
#pragma unroll
    for (int k = 0; k < RPT; k++) b[k] = region_gather(T, g, x + s.ux[k], (y + (float)k) + s.uy[k]);
#pragma unroll
    for (int k = 0; k < RPT; k++) {
        float vx, vy;
        demons_force(bilinear_blend_g(b[k]), s.r[k], s.gx[k], s.gy[k], s.ux[k], s.uy[k], vx, vy);
        if (fix) {
            vx = __shfl(vx, fix_lane, 64);
            vy = __shfl(vy, fix_lane, 64);
        }
        hrow[k * 64] = make_float2(lane_taps<RAD>(vx, tp), lane_taps<RAD>(vy, tp));
    }
}

// Phase 3: vertical taps over the filtered rows into the field; off[t] is the
// float2 index of row y - RAD + t at this lane.  Returns the squared update of
// the rows k with bit k of `count` set.
template <int RAD, int RPT>
__device__ __forceinline__ float region_cols(RegionRows<RPT>& s, const float2* __restrict__ hb,
                                             const int (&off)[RPT + 2 * RAD], const Taps& tp, unsigned count)
{
    float2 t[RPT + 2 * RAD];
#pragma unroll
    for (int j = 0; j < RPT + 2 * RAD; j++) t[j] = hb[off[j]];
    float ss = 0.0f;
#pragma unroll
    for (int k = 0; k < RPT; k++) {
        float ox = 0.0f, oy = 0.0f;
#pragma unroll
        for (int j = 0; j <= 2 * RAD; j++) {
            ox = fmaf(tp.w[j], t[k + j].x, ox);
            oy = fmaf(tp.w[j], t[k + j].y, oy);
        }
        if (count & (1u << k)) {
            const float dx = ox - s.ux[k], dy = oy - s.uy[k];
            ss = fmaf(dx, dx, fmaf(dy, dy, ss));
        }
        s.ux[k] = ox;
        s.uy[k] = oy;
    }
    return ss;
}

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

}  // namespace ebsd
