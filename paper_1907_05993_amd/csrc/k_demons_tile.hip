// Several demons iterations per launch on 2-D tiles (multi-resolution demons,
// section 1, Eq. (1)), for levels whose pixels of the whole batch do not fill
// the device: there a launch of the row-marching kernels lasts as long as its
// chain of row steps (about 0.7 us each, 22 and more per launch), whatever the
// batch.  A workgroup takes an output tile with a halo of K r pixels and runs K
// iterations on it (demons_region.h: state in registers, one barrier per
// iteration), the valid part shrinking by r on every side per iteration.
// Bound: the chain of K iterations (about 1 us each at 32 region rows) and a
// launch's fixed cost (about 5 us); the recomputed halo is idle capacity.
//
// Stops on a tolerance: launch L runs iterations L K .. L K + K - 1 and
// leaves their partial sums (slot: iteration mod 8); the next launch takes the
// decisions in order, and if the pair should have stopped in between, runs
// the iterations up to there again from the previous launch's input, which is
// still in the other buffer.  Counts, status and fields are those of one
// iteration per launch.
#include "demons_region.h"
#include "ebsd_internal.h"

namespace ebsd {

namespace {

constexpr int kTileRPT = 4;  // rows per wavefront

template <int RAD, int K, int NWV>
__global__ void __launch_bounds__(64 * NWV)
    k_demons_tiles(const Bucket* __restrict__ bk, int level, int L, Taps tp, float tol, int ntx, int ntiles, int cap)
{
    constexpr int RPT = kTileRPT, RH = NWV * RPT, HALO = RAD * K;
    constexpr int TX = 64 - 2 * HALO, TY = RH - 2 * HALO;
    static_assert(TX > 0 && TY > 0, "halo covers the region");
    extern __shared__ float2 lds[];  // [2][RH][64] filtered rows
    __shared__ float red[K][NWV];
    __shared__ double sh_sum;
    const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const int b = lb / ntiles, tile = lb - b * ntiles;
    const PairState st = bk->state[b];
    const int k0 = L * K;
    // a stop after more than k0 - K iterations can only have been written by tile 0 of
    // this launch, perhaps between the reads of two wavefronts of this workgroup: all of
    // them take the decision below from the sums
    if (st.stop >= 0 && st.stop <= k0 - K) return;  // uniform
    const int h = bk->lh[level], w = bk->lw[level];
    const int64_t npart = (int64_t)bk->nb * bk->max_tiles;
    const int64_t pofs = (int64_t)b * bk->max_tiles;
    int niter = min(K, cap - k0), again = 0;
    if (tol > 0.0f && L > 0) {
        const double hw = (double)h * (double)w, sc = (double)(1 << level);
        const int last = min(k0, cap);  // iterations run so far
        for (int i = k0 - K; i < last; i++) {
            const double ss = pair_sum(bk->partial + (i & 7) * npart + pofs, ntiles, &sh_sum);
            if (sqrt(ss / hw) * sc < (double)tol) {
                if (tile == 0 && threadIdx.x == 0) {
                    bk->state[b].stop = i + 1;
                    bk->state[b].convmask = st.convmask | (1u << level);
                }
                if (i + 1 == last) return;  // the field is in place
                again = i + 1 - (k0 - K);
                break;
            }
        }
    }
    if (again) niter = again;
    else if (niter <= 0) return;
    const int64_t slot = (int64_t)b * 2 * bk->H * bk->W;
    const float* R = bk->ref_pyr + (int64_t)bk->ref_slot[b] * bk->pyr_elems + bk->lvl_off[level];
    const float* Tg = bk->test_pyr + (int64_t)b * bk->pyr_elems + bk->lvl_off[level];
    // recompute: from the previous launch's input into the buffer its output is in
    const float* u = bk->field[(st.base + L + (again ? 1 : 0)) & 1] + slot;
    float* un = bk->field[(st.base + L + (again ? 0 : 1)) & 1] + slot;

    const int ty = tile / ntx, tx = tile - ty * ntx;
    const int lane = threadIdx.x & 63, wave = uniform_int(threadIdx.x >> 6);
    const int gx0 = tx * TX - HALO, gy0 = ty * TY - HALO;
    const int x = gx0 + lane, r0 = wave * RPT, y0 = gy0 + r0;
    const bool fix = gx0 < 0 || gx0 + 64 > w;  // uniform: some lanes lie outside the image
    const int fix_lane = clampi(x, 0, w - 1) - gx0;
    RegionRows<RPT> s;
    region_load(s, R, u, h, w, x, y0);
    const GatherBase T = gather_base(Tg, h, w);
    const BilGeom g = bil_geom(h, w);
    const float xf = (float)clampi(x, 0, w - 1), yf = (float)y0;
    int off[RPT + 2 * RAD];
#pragma unroll
    for (int j = 0; j < RPT + 2 * RAD; j++)
        off[j] = 64 * clampi(clampi(y0 - RAD + j, 0, h - 1) - gy0, 0, RH - 1) + lane;
    const bool own_x = lane >= HALO && lane < 64 - HALO && x < w;
    unsigned own = 0;
#pragma unroll
    for (int k = 0; k < RPT; k++)
        if (own_x && r0 + k >= HALO && r0 + k < RH - HALO && y0 + k < h) own |= 1u << k;

    for (int i = 0; i < niter; i++) {
        float2* hb = lds + (i & 1) * RH * 64;
        // the rows still needed: inside the image, and in the region shrunk by r per
        // finished iteration (for v), by r more for the field
        const auto needed = [&](int m) { return r0 < min(RH - m, h - gy0) && r0 + RPT > max(m, -gy0); };
        if (needed(RAD * i))
            region_rows<RAD, RPT>(s, T, g, tp, xf, yf, fix, fix_lane, hb + 64 * r0 + lane);
        __syncthreads();
        float ss = 0.0f;
        if (needed(RAD * (i + 1))) ss = region_cols<RAD, RPT>(s, hb, off, tp, own);
        if (tol > 0.0f && !again) {
            ss = wave_sum(ss);
            if (lane == 0) red[i][wave] = ss;
        }
    }
    if (own) {
        EBSD_GLOBAL float* out = gptr(un);
        const int64_t hw = (int64_t)h * w;
#pragma unroll
        for (int k = 0; k < RPT; k++)
            if (own & (1u << k)) {
                const int o = (y0 + k) * w + x;
                out[o] = s.ux[k];
                out[hw + o] = s.uy[k];
            }
    }
    if (tol > 0.0f && !again) {
        __syncthreads();
        if ((int)threadIdx.x < niter) {
            float tot = 0.0f;
#pragma unroll
            for (int i = 0; i < NWV; i++) tot += red[threadIdx.x][i];
            bk->partial[((k0 + threadIdx.x) & 7) * npart + pofs + tile] = tot;
        }
    }
}

// Without smoothing (r = 0) pixels do not interact: one launch runs all `cap`
// iterations of a level, each thread its own pixels, field in registers (the
// field is read and written once per level instead of once per iteration).
// Fixed iteration count only.  The unsmoothed field is irregular, so the lanes'
// gathers fall on different cache lines; from the vector cache (one line per
// clock) 12 patterns of 1244 x 1024 took 1.91 ms for 25 iterations.  A workgroup
// therefore keeps the test pattern around its tile's displaced position in LDS
// (64 columns x 4 PX rows, a margin of 32 px on every side, placed by the
// tile's mean displacement) and gathers there; lanes whose cell lies outside
// the window read memory instead (1.16 ms; a margin of 20 px 1.33, of 44 px
// 1.20).  Bound: vector ALU.  PX = 8 pixels per thread, or 2 where that leaves
// CUs without work (the levels of one or few patterns).
constexpr int kPointThreads = 256, kPointTX = 64, kPointMargin = 32;

template <int PX>
__global__ void __launch_bounds__(kPointThreads)
    k_demons_points(const Bucket* __restrict__ bk, int level, float w0, int ntx, int ntiles, int cap)
{
    constexpr int kPointPx = PX, kPointGroup = PX < 4 ? PX : 4;  // pixels of a thread, and iterated together
    constexpr int kPointTY = PX * kPointThreads / kPointTX;
    constexpr int kPointWW = kPointTX + 2 * kPointMargin, kPointWH = kPointTY + 2 * kPointMargin;
    __shared__ float win[kPointWH * kPointWW];
    __shared__ float red[2][kPointThreads / 64];
    const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const int b = lb / ntiles, tile = lb - b * ntiles;
    const int tx0 = (tile % ntx) * kPointTX, ty0 = (tile / ntx) * kPointTY;
    const int h = bk->lh[level], w = bk->lw[level], n = h * w;
    const int base = bk->state[b].base;
    const int64_t slot = (int64_t)b * 2 * bk->H * bk->W;
    const float* __restrict__ Tg = bk->test_pyr + (int64_t)b * bk->pyr_elems + bk->lvl_off[level];
    const EBSD_GLOBAL float* __restrict__ R =
        gptr(bk->ref_pyr + (int64_t)bk->ref_slot[b] * bk->pyr_elems + bk->lvl_off[level]);
    const GatherBase T = gather_base(Tg, h, w);
    const EBSD_GLOBAL float* __restrict__ u = gptr(bk->field[base & 1] + slot);
    EBSD_GLOBAL float* __restrict__ un = gptr(bk->field[(base + 1) & 1] + slot);
    const BilGeom g = bil_geom(h, w);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int x = min(tx0 + lane, w - 1);
    float ux[kPointPx], uy[kPointPx];
    float mx = 0.0f, my = 0.0f;
#pragma unroll
    for (int k = 0; k < kPointPx; k++) {
        const int y = min(ty0 + wave + k * (kPointThreads / 64), h - 1);
        ux[k] = u[y * w + x];
        uy[k] = u[n + y * w + x];
        mx += ux[k];
        my += uy[k];
    }
    // the window's corner (any value is valid: it only decides which gathers are from LDS)
    mx = wave_sum(mx);
    my = wave_sum(my);
    if (lane == 0) {
        red[0][wave] = mx;
        red[1][wave] = my;
    }
    __syncthreads();
    mx = my = 0.0f;
#pragma unroll
    for (int i = 0; i < kPointThreads / 64; i++) {
        mx += red[0][i];
        my += red[1][i];
    }
    const float sc = 1.0f / (kPointTX * kPointTY);
    const int wx0 = tx0 - kPointMargin + (int)fminf(fmaxf(mx * sc, -(float)w), (float)w);
    const int wy0 = ty0 - kPointMargin + (int)fminf(fmaxf(my * sc, -(float)h), (float)h);
    for (int i = threadIdx.x; i < kPointWH * kPointWW; i += kPointThreads) {
        const int yy = i / kPointWW, xx = i - yy * kPointWW;
        win[i] = Tg[clampi(wy0 + yy, 0, h - 1) * w + clampi(wx0 + xx, 0, w - 1)];
    }
    __syncthreads();
    const float fx0 = (float)wx0, fy0 = (float)wy0;
#pragma unroll
    for (int k0 = 0; k0 < kPointPx; k0 += kPointGroup) {
        float r[kPointGroup], gx[kPointGroup], gy[kPointGroup], py[kPointGroup];
#pragma unroll
        for (int k = 0; k < kPointGroup; k++) {
            const int y = min(ty0 + wave + (k0 + k) * (kPointThreads / 64), h - 1);
            const int xm = max(x - 1, 0), xp = min(x + 1, w - 1);
            const int ym = max(y - 1, 0), yp = min(y + 1, h - 1);
            r[k] = R[y * w + x];
            gx[k] = (R[y * w + xp] - R[y * w + xm]) * ((xp - xm == 2) ? 0.5f : 1.0f);
            gy[k] = (R[yp * w + x] - R[ym * w + x]) * ((yp - ym == 2) ? 0.5f : 1.0f);
            py[k] = (float)y;
        }
        for (int i = 0; i < cap; i++) {
            Bilin t[kPointGroup];
#pragma unroll
            for (int k = 0; k < kPointGroup; k++) {
                const float sx = (float)x + ux[k0 + k], sy = py[k] + uy[k0 + k];
                // bilinear_issue_g's cell and weights
                const float xc = fminf(fmaxf(sx, 0.0f), g.wm1), yc = fminf(fmaxf(sy, 0.0f), g.hm1);
                const float xf = fminf(floorf(xc), g.wm2), yf = fminf(floorf(yc), g.hm2);
                const float dx = xf - fx0, dy = yf - fy0;
                const bool in = dx >= 0.0f && dx <= (float)(kPointWW - 2) && dy >= 0.0f && dy <= (float)(kPointWH - 2);
                const int o = in ? (int)fmaf(dy, (float)kPointWW, dx) : 0;
                t[k].v00 = win[o];
                t[k].v01 = win[o + 1];
                t[k].v10 = win[o + kPointWW];
                t[k].v11 = win[o + kPointWW + 1];
                t[k].fx = xc - xf;
                t[k].fy = yc - yf;
                if (!in) t[k] = bilinear_issue_g(T, g, sx, sy);
            }
#pragma unroll
            for (int k = 0; k < kPointGroup; k++) {
                float vx, vy;
                demons_force(bilinear_blend_g(t[k]), r[k], gx[k], gy[k], ux[k0 + k], uy[k0 + k], vx, vy);
                // the one-tap smoothing, both passes (w0 = 1)
                ux[k0 + k] = fmaf(w0, fmaf(w0, vx, 0.0f), 0.0f);
                uy[k0 + k] = fmaf(w0, fmaf(w0, vy, 0.0f), 0.0f);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kPointPx; k++) {
        const int y = ty0 + wave + k * (kPointThreads / 64);
        if (tx0 + lane < w && y < h) {
            un[y * w + x] = ux[k];
            un[n + y * w + x] = uy[k];
        }
    }
}

template <int RAD, int K, int NWV>
hipError_t launch_tiles(const Bucket* d_bk, const Bucket& hb, int level, int L, const Taps& tp, float tol, int cap,
                        hipStream_t s)
{
    constexpr int RH = NWV * kTileRPT;
    constexpr size_t lds = sizeof(float2) * 2 * RH * 64;
    static std::atomic<uint64_t> attr_done{0};
    const hipError_t e = ensure_dynamic_lds((const void*)k_demons_tiles<RAD, K, NWV>, (int)lds, attr_done);
    if (e != hipSuccess) return e;
    const int tx = 64 - 2 * RAD * K, ty = RH - 2 * RAD * K;
    const int ntx = (hb.lw[level] + tx - 1) / tx, ntiles = ntx * ((hb.lh[level] + ty - 1) / ty);
    hipLaunchKernelGGL((k_demons_tiles<RAD, K, NWV>), dim3((unsigned)((int64_t)hb.nb * ntiles)), dim3(64 * NWV), lds,
                       s, d_bk, level, L, tp, tol, ntx, ntiles, cap);
    return hipGetLastError();
}

}  // namespace

int tile_iters(int radius) { return radius >= 1 && radius <= 3 ? 4 : radius == 4 ? 3 : 0; }

int tile_units(int h, int w, int radius, int rows)
{
    const int halo = 2 * radius * tile_iters(radius);
    const int tx = 64 - halo, ty = rows - halo;
    return ((w + tx - 1) / tx) * ((h + ty - 1) / ty);
}

hipError_t launch_demons_tiles(const Bucket* d_bk, const Bucket& hb, int level, int L, const float* taps, int radius,
                               float tol, int cap, int rows, hipStream_t s)
{
    Taps tp;
    for (int i = 0; i < 2 * kMaxRadius + 1; i++) tp.w[i] = i <= 2 * radius ? taps[i] : 0.0f;
    if (hb.nb <= 0 || hb.lh[level] < 2 || hb.lw[level] < 2 || (rows != 32 && rows != 64)) return hipErrorInvalidValue;
    switch (radius + (rows == 64 ? 8 : 0)) {
    case 1: return launch_tiles<1, 4, 8>(d_bk, hb, level, L, tp, tol, cap, s);
    case 2: return launch_tiles<2, 4, 8>(d_bk, hb, level, L, tp, tol, cap, s);
    case 3: return launch_tiles<3, 4, 8>(d_bk, hb, level, L, tp, tol, cap, s);
    case 4: return launch_tiles<4, 3, 8>(d_bk, hb, level, L, tp, tol, cap, s);
    case 9: return launch_tiles<1, 4, 16>(d_bk, hb, level, L, tp, tol, cap, s);
    case 10: return launch_tiles<2, 4, 16>(d_bk, hb, level, L, tp, tol, cap, s);
    case 11: return launch_tiles<3, 4, 16>(d_bk, hb, level, L, tp, tol, cap, s);
    case 12: return launch_tiles<4, 3, 16>(d_bk, hb, level, L, tp, tol, cap, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_demons_points(const Bucket* d_bk, const Bucket& hb, int level, const float* taps, int cap,
                                hipStream_t s)
{
    if (hb.nb <= 0 || hb.lh[level] < 2 || hb.lw[level] < 2) return hipErrorInvalidValue;
    const int ntx = (hb.lw[level] + kPointTX - 1) / kPointTX;
    const auto tiles = [&](int ty) { return ntx * ((hb.lh[level] + ty - 1) / ty); };
    constexpr int rows = kPointThreads / kPointTX;  // of one pixel per thread
    if ((int64_t)hb.nb * tiles(8 * rows) >= 1024)
        hipLaunchKernelGGL(k_demons_points<8>, dim3((unsigned)((int64_t)hb.nb * tiles(8 * rows))), dim3(kPointThreads),
                           0, s, d_bk, level, taps[0], ntx, tiles(8 * rows), cap);
    else
        hipLaunchKernelGGL(k_demons_points<2>, dim3((unsigned)((int64_t)hb.nb * tiles(2 * rows))), dim3(kPointThreads),
                           0, s, d_bk, level, taps[0], ntx, tiles(2 * rows), cap);
    return hipGetLastError();
}

}  // namespace ebsd
