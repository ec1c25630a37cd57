// Two demons iterations per launch by wavefronts that march down a strip on
// their own (multi-resolution demons, section 1, Eq. (1)).
//
// A wavefront (a workgroup of one) owns 64 C columns, C consecutive columns per
// lane (C = 4 for levels of more than 128 px, 2 up to 128; wider levels in
// segments whose halo columns are recomputed), and a strip of output rows.
// Stage 1 takes the rows of u from the top down: force, horizontal taps across
// the lanes (shifts of the wavefront, see demons_region.h), and adds the
// filtered row into the 2r + 1 output rows it is a tap of, which are kept as
// running sums in registers; the row that has all its taps is a row of u1,
// which stage 2 treats in the same way one row step later.  Nothing passes
// between wavefronts: no LDS, no barrier, and a row is one 16-byte load per
// channel and lane.  An output row's taps are added in row order as in the row
// kernels, so the fields are theirs bit for bit.
//
// Bound: vector ALU and its single wavefront's waits (four columns: 318 registers,
// one wavefront per SIMD; a step issues about 690 instructions, 2760 cycles, and
// took 3200 with the batch in the last-level cache, 4500 with 1024 pairs of 256 x
// 256 in memory).  Per iteration against the two-iteration row kernel, which
// executes as many vector instructions per pixel but waits on barriers and the
// LDS exchange for half of the time: 1024 pairs of 256 x 256 259 us (270), 512
// pairs 136 (149), 128 pairs 33 (41), 192 pairs of 400 x 400 186 (217), 1024
// pairs of 128 x 128 59 (80).  Three variants were slower: whole rows by several
// two-column wavefronts with their edge columns through LDS (390 us for the
// 1024 pairs), the next rows touched ahead (281), two wavefronts per SIMD with
// spilled registers.
//
// Border rows: the first image row enters the sums once for itself and once
// for every replicated row above it, the last one likewise, so no row is
// computed twice.  Border columns: the shifts leave a value of choice in the
// end lane; lanes past the last column (levels that do not fill the wavefront)
// take the border column's value.
#include "demons_region.h"
#include "ebsd_internal.h"

namespace ebsd {

namespace {

template <int C>
struct VecOf {
    typedef float type __attribute__((ext_vector_type(C)));
};

// C floats at byte voff + soff of a buffer, naturally aligned (the buffer unit
// drops the low address bits).
template <int C>
__device__ __forceinline__ void load_row(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, float (&v)[C])
{
    typedef unsigned U __attribute__((ext_vector_type(C)));
    U t;
    if constexpr (C == 4) t = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0);
    else t = __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0);
#pragma unroll
    for (int c = 0; c < C; c++) v[c] = __builtin_bit_cast(float, (unsigned)t[c]);
}
template <int C>
__device__ __forceinline__ void store_row(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, const float (&v)[C])
{
    typedef unsigned U __attribute__((ext_vector_type(C)));
    U t;
#pragma unroll
    for (int c = 0; c < C; c++) t[c] = __builtin_bit_cast(unsigned, v[c]);
    if constexpr (C == 4) __builtin_amdgcn_raw_buffer_store_b128(t, r, (int)voff, (int)soff, 0);
    else __builtin_amdgcn_raw_buffer_store_b64(t, r, (int)voff, (int)soff, 0);
}

template <int C>
struct MarchCtx {
    __amdgpu_buffer_rsrc_t R, U, UN;
    GatherBase T;
    BilGeom gg;
    int h;
    unsigned uw4, x4;  // row bytes; byte offset of the lane's first column (inside the row)
    unsigned ch1;      // bytes of a channel
    float x;           // the lane's first column
    float s0, s1;      // gradient scales of the lane's first and last column
    bool edge;         // the lane's last column is the image's last, or lies past it
    bool virt;         // the lane's columns lie past the image
    bool any_virt;     // uniform
    int last_lane;     // uniform: lane of the image's last column
    bool own;          // the lane's columns are written
    __device__ unsigned row(int y) const { return (unsigned)clampi(y, 0, h - 1) * uw4; }
    __device__ void load_u(int y, float (&vx)[C], float (&vy)[C]) const
    {
        const unsigned o = row(y);
        load_row<C>(U, x4, o, vx);
        load_row<C>(U, x4, o + ch1, vy);
    }
    __device__ void load_r(int y, float (&v)[C]) const { load_row<C>(R, x4, row(y), v); }
};

// A stage: the running sums of its output rows, and of the row it takes next the
// field, the gathers in flight and the reference rows around it.
template <int C, int RAD>
struct MarchStage {
    float ax[2 * RAD + 1][C], ay[2 * RAD + 1][C];
    float ux[C], uy[C];
    Bilin g[C];
    float rm[C], rc[C], rp[C];
};

template <int C, int RAD>
__device__ __forceinline__ void march_gather(const MarchCtx<C>& k, MarchStage<C, RAD>& s, int y)
{
#pragma unroll
    for (int c = 0; c < C; c++)
        s.g[c] = bilinear_issue_g(k.T, k.gg, (k.x + (float)c) + s.ux[c], (float)y + s.uy[c]);
}

// v of row y from the gathers of its field.
template <int C, int RAD>
__device__ __forceinline__ void march_force(const MarchCtx<C>& k, const MarchStage<C, RAD>& s, int y, float (&vx)[C],
                                            float (&vy)[C])
{
    const float sy = (y > 0 && y < k.h - 1) ? 0.5f : 1.0f;
    const float left = from_prev(s.rc[C - 1], s.rc[0]);
    float right = from_next(s.rc[0], s.rc[C - 1]);
    if (k.edge) right = s.rc[C - 1];
#pragma unroll
    for (int c = 0; c < C; c++) {
        const float rl = c == 0 ? left : s.rc[c > 0 ? c - 1 : 0], rr = c == C - 1 ? right : s.rc[c < C - 1 ? c + 1 : c];
        const float gx = (rr - rl) * (c == 0 ? k.s0 : (c == C - 1 ? k.s1 : 0.5f));
        const float gy = (s.rp[c] - s.rm[c]) * sy;
        demons_force(bilinear_blend_g(s.g[c]), s.rc[c], gx, gy, s.ux[c], s.uy[c], vx[c], vy[c]);
    }
    if (k.any_virt) {
        const float bx = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, vx[C - 1]),
                                                                             k.last_lane));
        const float by = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, vy[C - 1]),
                                                                             k.last_lane));
#pragma unroll
        for (int c = 0; c < C; c++) {
            vx[c] = k.virt ? bx : vx[c];
            vy[c] = k.virt ? by : vy[c];
        }
    }
}

// Add the filtered row at phase PH into its 2r + 1 output rows.  FIRST: the
// image's first row, which also stands for the r replicated rows above it.
template <int C, int RAD, int PH, bool FIRST>
__device__ __forceinline__ void march_add(MarchStage<C, RAD>& s, const float (&hx)[C], const float (&hy)[C],
                                          const Taps& tp)
{
    constexpr int NR = 2 * RAD + 1;
    if constexpr (FIRST) {
#pragma unroll
        for (int m = 0; m <= RAD; m++)
#pragma unroll
            for (int c = 0; c < C; c++) {
                float a = 0.0f, b = 0.0f;
#pragma unroll
                for (int j = 0; j <= RAD - m; j++) {
                    a = fmaf(tp.w[j], hx[c], a);
                    b = fmaf(tp.w[j], hy[c], b);
                }
                s.ax[(PH + m) % NR][c] = a;
                s.ay[(PH + m) % NR][c] = b;
            }
    } else {
#pragma unroll
        for (int j = 0; j <= 2 * RAD; j++)
#pragma unroll
            for (int c = 0; c < C; c++) {
                constexpr int B = PH + RAD + NR;
                float& a = s.ax[(B - j) % NR][c];
                float& b = s.ay[(B - j) % NR][c];
                a = fmaf(tp.w[j], hx[c], j == 0 ? 0.0f : a);
                b = fmaf(tp.w[j], hy[c], j == 0 ? 0.0f : b);
            }
    }
}
// The image's last row once more for every replicated row below it: row y - m
// lacks its taps r + m + 1 .. 2r.
template <int C, int RAD, int PH>
__device__ __forceinline__ void march_bottom(MarchStage<C, RAD>& s, const float (&hx)[C], const float (&hy)[C],
                                             const Taps& tp)
{
    constexpr int NR = 2 * RAD + 1;
#pragma unroll
    for (int m = 0; m < RAD; m++)
#pragma unroll
        for (int j = RAD + m + 1; j <= 2 * RAD; j++)
#pragma unroll
            for (int c = 0; c < C; c++) {
                float& a = s.ax[(PH + NR - m) % NR][c];
                float& b = s.ay[(PH + NR - m) % NR][c];
                a = fmaf(tp.w[j], hx[c], a);
                b = fmaf(tp.w[j], hy[c], b);
            }
}

// Sum of squared updates of a row against its old field.
template <int C>
__device__ __forceinline__ void march_ss(const float (&ox)[C], const float (&oy)[C], const float (&ux)[C],
                                         const float (&uy)[C], float& ss)
{
#pragma unroll
    for (int c = 0; c < C; c++) {
        const float dx = ox[c] - ux[c], dy = oy[c] - uy[c];
        ss = fmaf(dx, dx, fmaf(dy, dy, ss));
    }
}

template <int C>
__device__ __forceinline__ void march_store(const MarchCtx<C>& k, int y, const float (&ox)[C], const float (&oy)[C])
{
    const unsigned o = (unsigned)y * k.uw4;
    store_row<C>(k.UN, k.x4, o, ox);
    store_row<C>(k.UN, k.x4, o + k.ch1, oy);
}

// Keeps the compiler from moving work of one part of a step into another (the
// live registers of two parts do not fit).
#define EBSD_SCHED() __builtin_amdgcn_sched_barrier(0)

// Pipeline registers besides the stages.
template <int C>
struct MarchNext {
    float ux[C], uy[C];  // field of row y + 1 of stage 1
};

// The lane's words of a ring of kMarchHist rows in LDS: u for the first
// iteration's squared update, u1 for the second's (u read from memory again
// took 1024 pairs of 256 x 256 from 70.2 to 72.0 ms per call).
constexpr int kMarchHist = 8;
template <int C>
__device__ __forceinline__ void hist_put(float* h, int y, const float (&x)[C], const float (&v)[C])
{
    float* p = h + (y & (kMarchHist - 1)) * 2 * C * 64;
#pragma unroll
    for (int c = 0; c < C; c++) {
        p[c * 64] = x[c];
        p[(C + c) * 64] = v[c];
    }
}
template <int C>
__device__ __forceinline__ void hist_get(const float* h, int y, float (&x)[C], float (&v)[C])
{
    const float* p = h + (y & (kMarchHist - 1)) * 2 * C * 64;
#pragma unroll
    for (int c = 0; c < C; c++) {
        x[c] = p[c * 64];
        v[c] = p[(C + c) * 64];
    }
}

// Step at stage-1 row y, phase PH.  TWO: the second iteration follows in stage 2
// (row j = y - r - 1, same phase); otherwise stage 1's rows are the output.
// F1, O1, D2, F2, O2: the row is the image's first, a row completes, stage 2 runs,
// its row is the first, it completes one; all compile-time, so the running sums
// are fixed registers.  END: the image's last row may be reached.  hist: LDS ring
// of the lane's u1 rows (SS with TWO).
template <int C, int RAD, int PH, bool SS, bool TWO, bool F1, bool O1, bool D2, bool F2, bool O2, bool END>
__device__ __forceinline__ void march_step(const MarchCtx<C>& k, const Taps& tp, MarchStage<C, RAD>& a,
                                           MarchStage<C, RAD>& b, MarchNext<C>& n, int y, int y0, int y1, float& ss1,
                                           float& ss2, float* hist)
{
    constexpr int NR = 2 * RAD + 1, HR = kMarchHist;
    static_assert(RAD + 2 <= HR, "history too short");
    // ---- stage 1: force of row y, then the gathers of row y + 1
    float hx[C], hy[C];
    march_force(k, a, y, hx, hy);
    float oldx[C], oldy[C];
    // the field of the row that completes below
    if constexpr (SS && O1) hist_get<C>(hist + HR * 2 * C * 64, y - RAD, oldx, oldy);
#pragma unroll
    for (int c = 0; c < C; c++) {
        a.ux[c] = n.ux[c];
        a.uy[c] = n.uy[c];
        a.rm[c] = a.rc[c];
        a.rc[c] = a.rp[c];
    }
    if constexpr (SS) hist_put<C>(hist + HR * 2 * C * 64, y + 1, a.ux, a.uy);
    march_gather(k, a, y + 1);
    k.load_u(y + 2, n.ux, n.uy);
    k.load_r(y + 2, a.rp);
    EBSD_SCHED();
    // taps of row y; past the image the sums are complete
    if (!END || y < k.h) {
        lane_taps<C, RAD>(hx, tp);
        lane_taps<C, RAD>(hy, tp);
        march_add<C, RAD, PH, F1>(a, hx, hy, tp);
        if (END && y == k.h - 1) march_bottom<C, RAD, PH>(a, hx, hy, tp);
    }
    constexpr int DONE = (PH + RAD + 1) % NR;  // slot of output row y - r
    if constexpr (!TWO) {
        if constexpr (O1) {
            const int yo = y - RAD;
            if (k.own && yo < y1) {
                march_store<C>(k, yo, a.ax[DONE], a.ay[DONE]);
                if (SS) march_ss<C>(a.ax[DONE], a.ay[DONE], oldx, oldy, ss1);
            }
        }
        return;
    }
    EBSD_SCHED();
    // ---- stage 2: force of row j, then u1 of row j + 1 = y - r and its gathers
    const int j = y - RAD - 1;
    if constexpr (D2) march_force(k, b, j, hx, hy);
    if constexpr (O1) {
        const int yo = y - RAD;
        if constexpr (SS) {
            if (k.own && yo >= y0 && yo < y1) march_ss<C>(a.ax[DONE], a.ay[DONE], oldx, oldy, ss1);
            hist_put<C>(hist, yo, a.ax[DONE], a.ay[DONE]);
        }
#pragma unroll
        for (int c = 0; c < C; c++) {
            b.ux[c] = a.ax[DONE][c];
            b.uy[c] = a.ay[DONE][c];
        }
        march_gather(k, b, yo);
    }
    EBSD_SCHED();
    if constexpr (D2) {
#pragma unroll
        for (int c = 0; c < C; c++) {
            b.rm[c] = b.rc[c];
            b.rc[c] = b.rp[c];
        }
        k.load_r(j + 2, b.rp);
        EBSD_SCHED();
        if (!END || j < k.h) {
            lane_taps<C, RAD>(hx, tp);
            lane_taps<C, RAD>(hy, tp);
            march_add<C, RAD, PH, F2>(b, hx, hy, tp);
            if (END && j == k.h - 1) march_bottom<C, RAD, PH>(b, hx, hy, tp);
        }
        if constexpr (O2) {
            const int yo = j - RAD;
            if (k.own && yo < y1) {
                march_store<C>(k, yo, b.ax[DONE], b.ay[DONE]);
                if constexpr (SS) {
                    hist_get<C>(hist, yo, oldx, oldy);
                    march_ss<C>(b.ax[DONE], b.ay[DONE], oldx, oldy, ss2);
                }
            }
        }
    }
}

template <int B, int E, class F>
__device__ __forceinline__ void march_for(F&& f)
{
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        march_for<B + 1, E>(f);
    }
}

// Fill the pipeline of a stage whose first row is y.
template <int C, int RAD>
__device__ __forceinline__ void march_refs(const MarchCtx<C>& k, MarchStage<C, RAD>& s, int y)
{
    k.load_r(y - 1, s.rm);
    k.load_r(y, s.rc);
    k.load_r(y + 1, s.rp);
}

// One (TWO = false) or two iterations over output rows [y0, y1).  Phases: stage
// 1's row y is at phase (y - y0 + r [+ r with TWO]) mod (2r + 1).  A strip that
// starts at the image's first row begins there; its strip height is at least
// 2r + 1, so that no other strip reaches the first row's replicated rows.
template <int C, int RAD, bool SS, bool TWO>
__device__ __forceinline__ void march_strip(const MarchCtx<C>& k, const Taps& tp, int y0, int y1, float* hist,
                                            float& ss1, float& ss2)
{
    constexpr int NR = 2 * RAD + 1;
    MarchStage<C, RAD> a, b;
    MarchNext<C> n;
    const bool top = y0 == 0;
    int y = top ? 0 : y0 - (TWO ? 2 : 1) * RAD;
    {
        k.load_u(y, a.ux, a.uy);
        k.load_u(y + 1, n.ux, n.uy);
        march_refs(k, a, y);
        if (TWO) march_refs(k, b, max(0, y0 - RAD));
        if constexpr (SS) hist_put<C>(hist + kMarchHist * 2 * C * 64, y, a.ux, a.uy);
        march_gather(k, a, y);
#pragma unroll
        for (int s = 0; s < NR; s++)
#pragma unroll
            for (int c = 0; c < C; c++) {
                a.ax[s][c] = a.ay[s][c] = 0.0f;
                b.ax[s][c] = b.ay[s][c] = 0.0f;
            }
#pragma unroll
        for (int c = 0; c < C; c++) {
            b.ux[c] = b.uy[c] = 0.0f;
            b.g[c] = a.g[c];
        }
    }
    // last stage-1 row: the one whose step completes output row y1 - 1
    const int ye = y1 - 1 + (TWO ? 2 * RAD + 1 : RAD);
#define EBSD_MARCH(PH, F1, O1, D2, F2, O2, END) \
    march_step<C, RAD, PH, SS, TWO, F1, O1, D2, F2, O2, END>(k, tp, a, b, n, y, y0, y1, ss1, ss2, hist)
    if constexpr (TWO) {
        if (top) {
            EBSD_MARCH(NR - 1, true, false, false, false, false, true);
            y++;
            march_for<0, NR>([&](auto ic) {
                constexpr int p = decltype(ic)::value;  // y = p + 1
                EBSD_MARCH(p, false, (p + 1 >= RAD), (p >= RAD), (p == RAD), (p >= 2 * RAD), true);
                y++;
            });
        } else {
            march_for<0, NR>([&](auto ic) {
                constexpr int p = decltype(ic)::value;
                EBSD_MARCH(p, false, (p >= 2 * RAD), false, false, false, true);
                y++;
            });
            march_for<0, NR>([&](auto ic) {
                constexpr int p = decltype(ic)::value;
                EBSD_MARCH(p, false, true, true, false, (p >= 2 * RAD), true);
                y++;
            });
        }
    } else {
        if (top) {
            march_for<RAD, NR>([&](auto ic) {
                constexpr int p = decltype(ic)::value;  // y = p - r
                EBSD_MARCH(p, (p == RAD), (p >= 2 * RAD), false, false, false, true);
                y++;
            });
        } else {
            march_for<0, NR>([&](auto ic) {
                constexpr int p = decltype(ic)::value;
                EBSD_MARCH(p, false, (p >= 2 * RAD), false, false, false, true);
                y++;
            });
        }
    }
    // whole groups of 2r + 1 steps (the sums' registers repeat), without branches
    // until the image's last row comes near; the last group may run past ye, where
    // nothing is stored
    int groups = uniform_int(ye >= y ? (ye - y) / NR + 1 : 0);
    int inside = uniform_int(min(groups, max(0, k.h - 1 - y) / NR));
    y = uniform_int(y);
    groups -= inside;
#pragma unroll 1
    for (; inside > 0; inside--)
        march_for<0, NR>([&](auto ic) {
            constexpr int p = decltype(ic)::value;
            EBSD_MARCH(p, false, true, true, false, true, false);
            y++;
        });
#pragma unroll 1
    for (; groups > 0; groups--)
        march_for<0, NR>([&](auto ic) {
            constexpr int p = decltype(ic)::value;
            EBSD_MARCH(p, false, true, true, false, true, true);
            y++;
        });
#undef EBSD_MARCH
}

// Decisions, buffers and partial sums as in k_demons_rows2.
template <int C, int RAD, bool SS>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(C == 4 ? 1 : (RAD == 4 ? 2 : 3))))
    k_demons_march(const Bucket* __restrict__ bk, int level, int L, Taps tp, float tol, int rows, int nstrips,
                   int nsegs, int cap)
{
    __shared__ double sh_sum;
    __shared__ float hist[SS ? 2 * kMarchHist * 2 * C * 64 : 1];
    const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const int nunits = nstrips * nsegs;
    const int b = lb / nunits, unit = lb - b * nunits;
    const int strip = unit / nsegs, seg = unit - strip * nsegs;
    const PairState st = bk->state[b];
    const int k0 = 2 * L;
    if (st.stop >= 0 && st.stop < k0 - 1) return;  // uniform
    const int h = bk->lh[level], w = bk->lw[level];
    const int64_t npart = (int64_t)bk->nb * bk->max_tiles;
    const int64_t pofs = (int64_t)b * bk->max_tiles;
    bool recompute = false;
    if (SS && L > 0) {
        const double hw = (double)h * (double)w, sc = (double)(1 << level);
        const double ssa = pair_sum(bk->partial + ((k0 - 2) & 3) * npart + pofs, nunits, &sh_sum);
        if (sqrt(ssa / hw) * sc < (double)tol) {
            recompute = true;
        } else {
            const double ssb = pair_sum(bk->partial + ((k0 - 1) & 3) * npart + pofs, nunits, &sh_sum);
            if (sqrt(ssb / hw) * sc < (double)tol) {
                if (unit == 0 && threadIdx.x == 0) {
                    bk->state[b].stop = k0;
                    bk->state[b].convmask = st.convmask | (1u << level);
                }
                return;
            }
        }
        if (recompute && unit == 0 && threadIdx.x == 0) {
            bk->state[b].stop = k0 - 1;
            bk->state[b].convmask = st.convmask | (1u << level);
        }
    }
    if (!recompute && k0 >= cap) return;
    const int64_t slot = (int64_t)b * 2 * bk->H * bk->W;
    const float* R = bk->ref_pyr + (int64_t)bk->ref_slot[b] * bk->pyr_elems + bk->lvl_off[level];
    const float* T = bk->test_pyr + (int64_t)b * bk->pyr_elems + bk->lvl_off[level];
    float* fa = bk->field[(st.base + L) & 1] + slot;
    float* fb = bk->field[(st.base + L + 1) & 1] + slot;

    int sx0, ws, we;
    march_seg(seg, nsegs, w, C, RAD, sx0, ws, we);
    MarchCtx<C> k;
    k.h = uniform_int(h);
    const int uw = uniform_int(w);
    k.uw4 = 4u * (unsigned)uw;
    k.ch1 = (unsigned)k.h * k.uw4;
    k.R = make_rsrc(R, k.ch1);
    k.U = make_rsrc(recompute ? fb : fa, 2u * k.ch1);
    k.UN = make_rsrc(recompute ? fa : fb, 2u * k.ch1);
    k.T = gather_base(T, k.h, uw);
    k.gg = bil_geom(k.h, uw);
    // uniform floats: kept in scalar registers
    const auto sc = [](float v) { return __builtin_bit_cast(float, uniform_int(__builtin_bit_cast(int, v))); };
    k.gg.wm1 = sc(k.gg.wm1);
    k.gg.hm1 = sc(k.gg.hm1);
    k.gg.wm2 = sc(k.gg.wm2);
    k.gg.hm2 = sc(k.gg.hm2);
    k.gg.wf = sc(k.gg.wf);
    const int lane = threadIdx.x, gx = sx0 + C * lane;
    const int xl = min(gx, w - C);
    k.x = (float)xl;
    k.x4 = 4u * (unsigned)xl;
    k.s0 = gx == 0 ? 1.0f : 0.5f;
    k.edge = gx >= w - C;
    k.s1 = k.edge ? 1.0f : 0.5f;
    k.virt = gx >= w;
    k.any_virt = uniform_int(sx0) + 64 * C > uniform_int(w);
    k.last_lane = (uniform_int(w) - C - uniform_int(sx0)) / C;
    k.own = gx >= ws && gx < we;
    const int y0 = uniform_int(strip * rows), y1 = min(y0 + rows, k.h);
    float ss1 = 0.0f, ss2 = 0.0f;
    if (recompute) {
        march_strip<C, RAD, false, false>(k, tp, y0, y1, hist, ss1, ss2);
        return;
    }
    if (k0 + 1 < cap) {
        march_strip<C, RAD, SS, true>(k, tp, y0, y1, hist + lane, ss1, ss2);
        if (SS) {
            ss1 = wave_sum(ss1);
            ss2 = wave_sum(ss2);
            if (lane == 0) {
                bk->partial[(k0 & 3) * npart + pofs + unit] = ss1;
                bk->partial[((k0 + 1) & 3) * npart + pofs + unit] = ss2;
            }
        }
    } else {
        march_strip<C, RAD, SS, false>(k, tp, y0, y1, hist + lane, ss1, ss2);
        if (SS) {
            ss1 = wave_sum(ss1);
            if (lane == 0) bk->partial[(k0 & 3) * npart + pofs + unit] = ss1;
        }
    }
}

template <int C, int RAD>
hipError_t launch_c(const Bucket* d_bk, const Bucket& hb, int level, int L, const Taps& tp, float tol, int cap,
                    int rows, hipStream_t s)
{
    const int h = hb.lh[level], w = hb.lw[level];
    const int nstrips = (h + rows - 1) / rows, nsegs = march_segs(w, C, RAD);
    const dim3 grid((unsigned)((int64_t)hb.nb * nstrips * nsegs));
    if (tol > 0.0f)
        hipLaunchKernelGGL((k_demons_march<C, RAD, true>), grid, dim3(64), 0, s, d_bk, level, L, tp, tol, rows,
                           nstrips, nsegs, cap);
    else
        hipLaunchKernelGGL((k_demons_march<C, RAD, false>), grid, dim3(64), 0, s, d_bk, level, L, tp, tol, rows,
                           nstrips, nsegs, cap);
    return hipGetLastError();
}

}  // namespace

// Columns per lane: 2 up to 128 px, 4 above (multiples of 4, and up to radius 3:
// the sums of more rows do not fit the registers).  The buffer unit's 16-byte
// accesses need the level's rows, channels and pairs at multiples of 16 bytes
// (8 for 2 columns), which a width that is a multiple of the columns gives
// together with an even pattern size.
int march_cols(int h, int w, int radius)
{
    if (radius < 1 || radius > kMaxRadius || h < 2 || w < 4 || (int64_t)h * w > kMaxFp32Pixels) return 0;
    if (w <= 128) return w % 2 == 0 ? 2 : 0;
    return w % 4 == 0 && radius < 4 ? 4 : 0;
}

int march_units(int h, int w, int radius, int rows)
{
    return ((h + rows - 1) / rows) * march_segs(w, march_cols(h, w, radius), radius);
}

hipError_t launch_demons_march(const Bucket* d_bk, const Bucket& hb, int level, int L, const float* taps, int radius,
                               float tol, int cap, int rows, hipStream_t s)
{
    const int c = march_cols(hb.lh[level], hb.lw[level], radius);
    if (hb.nb <= 0 || !c || rows < kMarchMinRows || (c == 4 && (int64_t)hb.H * hb.W % 2)) return hipErrorInvalidValue;
    Taps tp;
    for (int i = 0; i < 2 * kMaxRadius + 1; i++) tp.w[i] = i <= 2 * radius ? taps[i] : 0.0f;
    switch (radius + (c == 4 ? 8 : 0)) {
    case 1: return launch_c<2, 1>(d_bk, hb, level, L, tp, tol, cap, rows, s);
    case 2: return launch_c<2, 2>(d_bk, hb, level, L, tp, tol, cap, rows, s);
    case 3: return launch_c<2, 3>(d_bk, hb, level, L, tp, tol, cap, rows, s);
    case 4: return launch_c<2, 4>(d_bk, hb, level, L, tp, tol, cap, rows, s);
    case 9: return launch_c<4, 1>(d_bk, hb, level, L, tp, tol, cap, rows, s);
    case 10: return launch_c<4, 2>(d_bk, hb, level, L, tp, tol, cap, rows, s);
    case 11: return launch_c<4, 3>(d_bk, hb, level, L, tp, tol, cap, rows, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ebsd
