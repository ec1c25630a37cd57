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

// What a workgroup of launch L has to do.
struct TileWork {
    int b, tile;
    int niter;     // iterations to run
    bool sums;     // leave their partial sums
    const float *R, *T, *u;
    float* un;
};

// The decisions that launch L takes (all threads, uniform); false: nothing to do.
template <int K>
__device__ bool tile_work(const Bucket* __restrict__ bk, int level, int L, float tol, int ntiles, int cap,
                          double* sh_sum, TileWork& t)
{
    const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const int b = lb / ntiles, tile = lb - b * ntiles;
    const PairState st = bk->state[b];
    const int k0 = L * K;
    // a stop after more than k0 - K iterations can only have been written by tile 0 of
    // this launch, perhaps between the reads of two wavefronts of this workgroup: all of
    // them take the decision below from the sums
    if (st.stop >= 0 && st.stop <= k0 - K) return false;
    const int64_t npart = (int64_t)bk->nb * bk->max_tiles;
    const int64_t pofs = (int64_t)b * bk->max_tiles;
    int niter = min(K, cap - k0), again = 0;
    if (tol > 0.0f && L > 0) {
        const double hw = (double)bk->lh[level] * (double)bk->lw[level], sc = (double)(1 << level);
        const int last = min(k0, cap);  // iterations run so far
        for (int i = k0 - K; i < last; i++) {
            const double ss = pair_sum(bk->partial + (i & 7) * npart + pofs, ntiles, sh_sum);
            if (sqrt(ss / hw) * sc < (double)tol) {
                if (tile == 0 && threadIdx.x == 0) {
                    bk->state[b].stop = i + 1;
                    bk->state[b].convmask = st.convmask | (1u << level);
                }
                if (i + 1 == last) return false;  // the field is in place
                again = i + 1 - (k0 - K);
                break;
            }
        }
    }
    if (again) niter = again;
    else if (niter <= 0) return false;
    const int64_t slot = (int64_t)b * 2 * bk->H * bk->W;
    t.b = b;
    t.tile = tile;
    t.niter = niter;
    t.sums = tol > 0.0f && !again;
    t.R = bk->ref_pyr + (int64_t)bk->ref_slot[b] * bk->pyr_elems + bk->lvl_off[level];
    t.T = bk->test_pyr + (int64_t)b * bk->pyr_elems + bk->lvl_off[level];
    // recompute: from the previous launch's input into the buffer its output is in
    t.u = bk->field[(st.base + L + (again ? 1 : 0)) & 1] + slot;
    t.un = bk->field[(st.base + L + (again ? 0 : 1)) & 1] + slot;
    return true;
}

// The tile's partial sums of the launch's iterations from the wavefronts' (all
// threads).
template <int K, int NWV>
__device__ void tile_sums(const Bucket* __restrict__ bk, int L, const TileWork& t, const float (*red)[NWV])
{
    __syncthreads();
    if ((int)threadIdx.x < t.niter) {
        float tot = 0.0f;
#pragma unroll
        for (int i = 0; i < NWV; i++) tot += red[threadIdx.x][i];
        const int64_t npart = (int64_t)bk->nb * bk->max_tiles;
        bk->partial[((L * K + threadIdx.x) & 7) * npart + (int64_t)t.b * bk->max_tiles + t.tile] = tot;
    }
}

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
    TileWork t;
    if (!tile_work<K>(bk, level, L, tol, ntiles, cap, &sh_sum, t)) return;  // uniform
    const int h = bk->lh[level], w = bk->lw[level];
    const int ty = t.tile / ntx, tx = t.tile - ty * ntx;
    const int lane = threadIdx.x & 63, wave = uniform_int(threadIdx.x >> 6);
    const int gx0 = tx * TX - HALO, gy0 = ty * TY - HALO;
    const int x = gx0 + lane, r0 = wave * RPT, y0 = gy0 + r0;
    const bool fix = gx0 < 0 || gx0 + 64 > w;  // uniform: some lanes lie outside the image
    const int fix_lane = clampi(x, 0, w - 1) - gx0;
    RegionRows<RPT> s;
    region_load(s, t.R, t.u, h, w, x, y0);
    const GatherBase T = gather_base(t.T, h, w);
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

    for (int i = 0; i < t.niter; i++) {
        float2* hb = lds + (i & 1) * RH * 64;
        // the rows still needed: inside the image, and in the region shrunk by r per
        // finished iteration (for v), by r more for the field
        const auto needed = [&](int m) { return r0 < min(RH - m, h - gy0) && r0 + RPT > max(m, -gy0); };
        if (needed(RAD * i))
            region_rows<RAD, RPT>(s, T, g, tp, xf, yf, fix, fix_lane, hb + 64 * r0 + lane);
        __syncthreads();
        float ss = 0.0f;
        if (needed(RAD * (i + 1))) ss = region_cols<RAD, RPT>(s, hb, off, tp, own);
        if (t.sums) {
            ss = wave_sum(ss);
            if (lane == 0) red[i][wave] = ss;
        }
    }
    if (own) {
        EBSD_GLOBAL float* out = gptr(t.un);
        const int64_t hw = (int64_t)h * w;
#pragma unroll
        for (int k = 0; k < RPT; k++)
            if (own & (1u << k)) {
                const int o = (y0 + k) * w + x;
                out[o] = s.ux[k];
                out[hw + o] = s.uy[k];
            }
    }
    if (t.sums) tile_sums<K, NWV>(bk, L, t, red);
}

// The same on regions of 128 columns x 80 rows, two columns per lane and five
// rows per wavefront: with the halo of 4 iterations of radius 3 a tile of 104 x
// 56 px (60% of the region; 40 x 40 of 64 x 64 above), and none at the sides of
// levels up to 128 px.  One LDS buffer of filtered rows (80 KiB, one workgroup of
// 16 wavefronts per CU), so two barriers per iteration.  Bound: vector ALU.
// Measured per iteration (against regions of 64 x 64): 64 levels of 128 x 128 px
// 8.3 us (13.1), 16 of 256 x 256 9.2 (11.3), one of 1244 x 1024 9.9 (13.1).
constexpr int kWideRPT = 5, kWideRows = 16 * kWideRPT, kWideCols = 128;

template <int RAD, int K>
__global__ void __launch_bounds__(1024)
    k_demons_wide(const Bucket* __restrict__ bk, int level, int L, Taps tp, float tol, int ntx, int ntiles, int cap)
{
    constexpr int RPT = kWideRPT, RH = kWideRows, HALO = RAD * K, NWV = RH / RPT;
    constexpr int TX = kWideCols - 2 * HALO, TY = RH - 2 * HALO;
    static_assert(TX > 0 && TY > 0 && HALO % 2 == 0, "halo covers the region or splits a lane");
    extern __shared__ float4 wide[];  // [RH][64] filtered rows: (x, y) of a lane's two columns
    __shared__ float red[K][NWV];
    __shared__ double sh_sum;
    TileWork t;
    if (!tile_work<K>(bk, level, L, tol, ntiles, cap, &sh_sum, t)) return;  // uniform
    const int h = bk->lh[level], w = bk->lw[level];
    const int ty = t.tile / ntx, tx = t.tile - ty * ntx;
    const int lane = threadIdx.x & 63, wave = uniform_int(threadIdx.x >> 6);
    const int gx0 = tx == 0 && ntx == 1 ? 0 : tx * TX - HALO, gy0 = ty * TY - HALO;
    const int x = gx0 + 2 * lane, r0 = wave * RPT, y0 = gy0 + r0;
    // columns outside the image (uniform: any) take the border column's v
    const bool fix = gx0 < 0 || gx0 + kWideCols > w;
    const int first = max(-gx0, 0) / 2, last = min(w - 1 - gx0, kWideCols - 1);
    float ux[RPT][2], uy[RPT][2], r[RPT][2], gx[RPT][2], gy[RPT][2], px[2];
    unsigned own = 0;
    {
        const EBSD_GLOBAL float* __restrict__ R = gptr(t.R);
        const EBSD_GLOBAL float* __restrict__ u = gptr(t.u);
        float above[2], here[2], below[2];
        int xc[2];
#pragma unroll
        for (int c = 0; c < 2; c++) {
            xc[c] = clampi(x + c, 0, w - 1);
            px[c] = (float)xc[c];
            above[c] = R[max(clampi(y0, 0, h - 1) - 1, 0) * w + xc[c]];
            here[c] = R[clampi(y0, 0, h - 1) * w + xc[c]];
        }
#pragma unroll
        for (int k = 0; k < RPT; k++) {
            const int yc = clampi(y0 + k, 0, h - 1);
            const int ym = max(yc - 1, 0), yp = min(yc + 1, h - 1);
            const float sy = (yp - ym == 2) ? 0.5f : 1.0f;
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const int xm = max(xc[c] - 1, 0), xp = min(xc[c] + 1, w - 1);
                const int o = yc * w + xc[c];
                below[c] = R[yp * w + xc[c]];
                ux[k][c] = u[o];
                uy[k][c] = u[(int64_t)h * w + o];
                r[k][c] = here[c];
                gx[k][c] = (R[yc * w + xp] - R[yc * w + xm]) * ((xp - xm == 2) ? 0.5f : 1.0f);
                gy[k][c] = (below[c] - above[c]) * sy;
                // the next row: the same one again where the index is clamped
                if (clampi(y0 + k + 1, 0, h - 1) != yc) {
                    above[c] = here[c];
                    here[c] = below[c];
                }
                if (x + c - gx0 >= (ntx == 1 ? 0 : HALO) && x + c - gx0 < kWideCols - (ntx == 1 ? 0 : HALO) &&
                    x + c < w && r0 + k >= HALO && r0 + k < RH - HALO && y0 + k < h)
                    own |= 1u << (2 * k + c);
            }
        }
    }
    const GatherBase T = gather_base(t.T, h, w);
    const BilGeom g = bil_geom(h, w);
    for (int i = 0; i < t.niter; i++) {
        // the rows still needed: inside the image, and in the region shrunk by r per
        // finished iteration (for v), by r more for the field
        const auto needed = [&](int m) { return r0 < min(RH - m, h - gy0) && r0 + RPT > max(m, -gy0); };
        if (needed(RAD * i)) {
#pragma unroll
            for (int k = 0; k < RPT; k++) {
                Bilin b[2];
#pragma unroll
                for (int c = 0; c < 2; c++)
                    b[c] = bilinear_issue_g(T, g, px[c] + ux[k][c], (float)(y0 + k) + uy[k][c]);
                float vx[2], vy[2];
#pragma unroll
                for (int c = 0; c < 2; c++)
                    demons_force(bilinear_blend_g(b[c]), r[k][c], gx[k][c], gy[k][c], ux[k][c], uy[k][c], vx[c], vy[c]);
                if (fix) {
                    const auto lane_of = [](float v, int l) {
                        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
                    };
                    const float lx = lane_of(vx[0], first), ly = lane_of(vy[0], first);
                    const float rx = lane_of(last & 1 ? vx[1] : vx[0], last >> 1);
                    const float ry = lane_of(last & 1 ? vy[1] : vy[0], last >> 1);
#pragma unroll
                    for (int c = 0; c < 2; c++) {
                        vx[c] = x + c < 0 ? lx : (x + c >= w ? rx : vx[c]);
                        vy[c] = x + c < 0 ? ly : (x + c >= w ? ry : vy[c]);
                    }
                }
                lane_taps<2, RAD>(vx, tp);
                lane_taps<2, RAD>(vy, tp);
                wide[(r0 + k) * 64 + lane] = make_float4(vx[0], vy[0], vx[1], vy[1]);
            }
        }
        __syncthreads();
        float ss = 0.0f;
        if (needed(RAD * (i + 1))) {
            float ax[RPT][2], ay[RPT][2];
#pragma unroll
            for (int k = 0; k < RPT; k++)
#pragma unroll
                for (int c = 0; c < 2; c++) ax[k][c] = ay[k][c] = 0.0f;
#pragma unroll
            for (int j = 0; j < RPT + 2 * RAD; j++) {  // a row enters every sum it is a tap of, in tap order
                const int row = clampi(clampi(y0 - RAD + j, 0, h - 1) - gy0, 0, RH - 1);
                const float4 q = wide[row * 64 + lane];
#pragma unroll
                for (int k = 0; k < RPT; k++) {
                    if (j - k < 0 || j - k > 2 * RAD) continue;
                    ax[k][0] = fmaf(tp.w[j - k], q.x, ax[k][0]);
                    ay[k][0] = fmaf(tp.w[j - k], q.y, ay[k][0]);
                    ax[k][1] = fmaf(tp.w[j - k], q.z, ax[k][1]);
                    ay[k][1] = fmaf(tp.w[j - k], q.w, ay[k][1]);
                }
            }
#pragma unroll
            for (int k = 0; k < RPT; k++)
#pragma unroll
                for (int c = 0; c < 2; c++) {
                    if (own & (1u << (2 * k + c))) {
                        const float dx = ax[k][c] - ux[k][c], dy = ay[k][c] - uy[k][c];
                        ss = fmaf(dx, dx, fmaf(dy, dy, ss));
                    }
                    ux[k][c] = ax[k][c];
                    uy[k][c] = ay[k][c];
                }
        }
        if (t.sums) {
            ss = wave_sum(ss);
            if (lane == 0) red[i][wave] = ss;
        }
        __syncthreads();  // the rows are rewritten by the next iteration
    }
    EBSD_GLOBAL float* out = gptr(t.un);
    const int64_t hw = (int64_t)h * w;
#pragma unroll
    for (int k = 0; k < RPT; k++)
#pragma unroll
        for (int c = 0; c < 2; c++)
            if (own & (1u << (2 * k + c))) {
                const int o = (y0 + k) * w + x + c;
                out[o] = ux[k][c];
                out[hw + o] = uy[k][c];
            }
    if (t.sums) tile_sums<K, NWV>(bk, L, t, red);
}

// Without smoothing (r = 0) pixels do not interact: one launch runs all `cap`
// iterations of a level, each thread its own pixels, field in registers (the
// field is read and written once per level instead of once per iteration).
// Fixed iteration count only.  The unsmoothed field is irregular, so the lanes'
// gathers fall on different cache lines; from the vector cache (one line per
// clock) 12 patterns of 1244 x 1024 took 1.91 ms for 25 iterations.  A workgroup
// therefore keeps the test pattern around its tile's displaced position in LDS
// (64 columns x 8 PX rows, a margin of 36 px on every side, placed by the tile's
// mean displacement) and gathers there; lanes whose cell lies outside the window
// read memory instead: 1.13 ms.  (Tiles of 4 PX rows and 32 px 1.18, with 24 px
// 1.23, 16 px 1.33; of 16 PX rows and 48 px 1.23.)  Bound: vector ALU at 45%, and
// the memory reads of a few far lanes that nearly every wavefront has in nearly
// every iteration.  PX = 8 pixels per thread, or 2 where that leaves CUs without
// work (the levels of one or few patterns: 12 of 622 x 512 209 us, 253 with 8).
constexpr int kPointThreads = 512, kPointTX = 64, kPointMargin = 36;

template <int PX, bool LARGE>
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
    const BilGeomOf<LARGE> g = bil_geom<LARGE>(h, w);
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

// Tiles of a level cut from regions of 128 columns (none of the halo across when
// the level fits one) x 80 rows.
int wide_tiles_x(int w, int halo) { return w <= kWideCols ? 1 : (w + kWideCols - 2 * halo - 1) / (kWideCols - 2 * halo); }

template <int RAD, int K>
hipError_t launch_wide(const Bucket* d_bk, const Bucket& hb, int level, int L, const Taps& tp, float tol, int cap,
                       hipStream_t s)
{
    constexpr size_t lds = sizeof(float4) * kWideRows * 64;
    static std::atomic<uint64_t> attr_done{0};
    const hipError_t e = ensure_dynamic_lds((const void*)k_demons_wide<RAD, K>, (int)lds, attr_done);
    if (e != hipSuccess) return e;
    const int ty = kWideRows - 2 * RAD * K;
    const int ntx = wide_tiles_x(hb.lw[level], RAD * K), ntiles = ntx * ((hb.lh[level] + ty - 1) / ty);
    hipLaunchKernelGGL((k_demons_wide<RAD, K>), dim3((unsigned)((int64_t)hb.nb * ntiles)), dim3(1024), lds, s, d_bk,
                       level, L, tp, tol, ntx, ntiles, cap);
    return hipGetLastError();
}

}  // namespace

int tile_iters(int radius, int rows)
{
    if (radius < 1 || radius > 4) return 0;
    return radius < 4 || rows == 80 ? 4 : 3;
}

int tile_units(int h, int w, int radius, int rows)
{
    const int halo = radius * tile_iters(radius, rows), ty = rows - 2 * halo;
    const int nx = rows == kWideRows ? wide_tiles_x(w, halo) : (w + 64 - 2 * halo - 1) / (64 - 2 * halo);
    return nx * ((h + ty - 1) / ty);
}

hipError_t launch_demons_tiles(const Bucket* d_bk, const Bucket& hb, int level, int L, const float* taps, int radius,
                               float tol, int cap, int rows, hipStream_t s)
{
    Taps tp;
    for (int i = 0; i < 2 * kMaxRadius + 1; i++) tp.w[i] = i <= 2 * radius ? taps[i] : 0.0f;
    if (hb.nb <= 0 || hb.lh[level] < 2 || hb.lw[level] < 2 || (rows != 32 && rows != 64 && rows != kWideRows) ||
        (int64_t)hb.lh[level] * hb.lw[level] > kMaxFp32Pixels)
        return hipErrorInvalidValue;
    switch (1000 * radius + rows) {
    case 1032: return launch_tiles<1, 4, 8>(d_bk, hb, level, L, tp, tol, cap, s);
    case 2032: return launch_tiles<2, 4, 8>(d_bk, hb, level, L, tp, tol, cap, s);
    case 3032: return launch_tiles<3, 4, 8>(d_bk, hb, level, L, tp, tol, cap, s);
    case 4032: return launch_tiles<4, 3, 8>(d_bk, hb, level, L, tp, tol, cap, s);
    case 1064: return launch_tiles<1, 4, 16>(d_bk, hb, level, L, tp, tol, cap, s);
    case 2064: return launch_tiles<2, 4, 16>(d_bk, hb, level, L, tp, tol, cap, s);
    case 3064: return launch_tiles<3, 4, 16>(d_bk, hb, level, L, tp, tol, cap, s);
    case 4064: return launch_tiles<4, 3, 16>(d_bk, hb, level, L, tp, tol, cap, s);
    case 1080: return launch_wide<1, 4>(d_bk, hb, level, L, tp, tol, cap, s);
    case 2080: return launch_wide<2, 4>(d_bk, hb, level, L, tp, tol, cap, s);
    case 3080: return launch_wide<3, 4>(d_bk, hb, level, L, tp, tol, cap, s);
    case 4080: return launch_wide<4, 4>(d_bk, hb, level, L, tp, tol, cap, s);
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
    const auto launch = [&](auto kernel, int px) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((int64_t)hb.nb * tiles(px * rows))), dim3(kPointThreads), 0, s, d_bk,
                           level, taps[0], ntx, tiles(px * rows), cap);
    };
    if ((int64_t)hb.lh[level] * hb.lw[level] > kMaxFp32Pixels) launch(k_demons_points<8, true>, 8);
    else if ((int64_t)hb.nb * tiles(8 * rows) >= 1024) launch(k_demons_points<8, false>, 8);
    else launch(k_demons_points<2, false>, 2);
    return hipGetLastError();
}

}  // namespace ebsd
