// Level-resident demons (multi-resolution demons, section 1, Eq. (1)): a level of
// at most 64 x 64 pixels is iterated to its cap or tolerance inside one
// workgroup per pair, so a coarse level costs one launch, and each pair stops
// on its own tolerance.  The iteration is demons_region.h's with the whole level
// as the region: 16 wavefronts of 64 columns, RPT = ceil(h / 16) rows each;
// the test pattern's level sits in LDS for the gathers, the field, the
// reference and its gradient in registers, and one barrier per iteration
// separates the horizontal taps from the vertical ones.
//
// What bounds it: vector ALU (about 75 instructions per pixel and iteration;
// a 64 x 64 level is 1.9 us per iteration at full rate on the pair's one CU;
// measured 2.1 us for up to 256 pairs and 4 rounds of that for 1024.  With the
// field, the gradient's operands and both passes of taps in LDS, eight
// wavefronts and three barriers per iteration, one pair took 6.8 us, and 1024
// pairs ran faster on the two-iteration row kernels (26.8 us per iteration):
// 1024 warm-started pairs of 256 x 256 now 73.4 ms instead of 75.9).
// The update's sum is reduced in another order than the row kernels', which can
// move a stop decision only when the RMS update lies within rounding of the
// tolerance.  A pair's stop is decided one barrier late: the sum of iteration
// k is read behind the barrier of iteration k + 1, before that one changes the
// field.
#include <hip/hip_runtime.h>

#include "demons_region.h"
#include "ebsd_internal.h"
#include "../../include/ebsd.h"

namespace ebsd {

namespace {

constexpr int kResWaves = 16;
constexpr int kResThreads = 64 * kResWaves;

// dynamic LDS: two buffers of filtered rows (16 RPT rows of 64), the test level
template <int RPT>
constexpr size_t res_lds_bytes(int px)
{
    return sizeof(float2) * 2 * 64 * kResWaves * RPT + sizeof(float) * px;
}

template <int RAD, int RPT>
__global__ void __launch_bounds__(kResThreads)
    k_demons_resident(const Bucket* __restrict__ bk, int level, Taps tp, float tol, int cap)
{
    extern __shared__ float2 lds[];
    __shared__ float red[2][kResWaves];
    const int b = blockIdx.x;
    PairState st = bk->state[b];
    const int h = bk->lh[level], w = bk->lw[level], n = h * w;
    float* sT = reinterpret_cast<float*>(lds + 2 * 64 * kResWaves * RPT);
    const float* __restrict__ Rg = bk->ref_pyr + (int64_t)bk->ref_slot[b] * bk->pyr_elems + bk->lvl_off[level];
    const float* __restrict__ Tg = bk->test_pyr + (int64_t)b * bk->pyr_elems + bk->lvl_off[level];
    const int64_t slot = (int64_t)b * 2 * bk->H * bk->W;
    for (int i = threadIdx.x; i < n; i += kResThreads) sT[i] = Tg[i];
    const int x = threadIdx.x & 63, wave = uniform_int(threadIdx.x >> 6);
    const int y0 = wave * RPT;
    const bool rows = y0 < h;  // uniform; wavefronts below the level only take part in the barriers
    RegionRows<RPT> s;
    int off[RPT + 2 * RAD];
    unsigned count = 0;
    if (rows) {
        region_load(s, Rg, bk->field[st.base & 1] + slot, h, w, x, y0);
#pragma unroll
        for (int j = 0; j < RPT + 2 * RAD; j++) off[j] = 64 * clampi(y0 - RAD + j, 0, h - 1) + x;
#pragma unroll
        for (int k = 0; k < RPT; k++)
            if (x < w && y0 + k < h) count |= 1u << k;
    }
    const BilGeom g = bil_geom(h, w);
    const LdsImage T{sT, w};
    const double scale = (double)(1 << level);
    const bool fix = w < 64;
    const int fix_lane = min(x, w - 1);
    __syncthreads();

    auto converged = [&](int slot_) {  // the same value in every thread
        float tot = 0.0f;
#pragma unroll
        for (int i = 0; i < kResWaves; i++) tot += red[slot_][i];
        return sqrt((double)tot / ((double)h * (double)w)) * scale < (double)tol;
    };
    int k = 0;
    bool conv = false;
    while (k < cap) {
        float2* hb = lds + (k & 1) * 64 * kResWaves * RPT;
        if (rows) region_rows<RAD, RPT>(s, T, g, tp, (float)x, (float)y0, fix, fix_lane, hb + 64 * y0 + x);
        __syncthreads();
        if (tol > 0.0f && k > 0 && converged((k - 1) & 1)) {
            conv = true;
            break;
        }
        float ss = 0.0f;
        if (rows) ss = region_cols<RAD, RPT>(s, hb, off, tp, count);
        if (tol > 0.0f) {
            ss = wave_sum(ss);
            if (x == 0) red[k & 1][wave] = ss;
        }
        k++;
    }
    if (tol > 0.0f && !conv && cap > 0) {
        __syncthreads();
        conv = converged((cap - 1) & 1);
    }
    float* __restrict__ out = bk->field[(st.base + k) & 1] + slot;
    if (rows && x < w) {
#pragma unroll
        for (int r = 0; r < RPT; r++)
            if (y0 + r < h) {
                out[(y0 + r) * w + x] = s.ux[r];
                out[n + (y0 + r) * w + x] = s.uy[r];
            }
    }
    if (threadIdx.x == 0) {
        bk->iters[(int64_t)b * bk->L + level] = k;
        st.cur = (st.base + k) & 1;
        st.base = st.cur ^ 1;  // where the next level's field is prolonged to
        st.stop = -1;
        if (conv) st.convmask |= 1u << level;
        bk->state[b] = st;
    }
}

template <int RAD, int RPT>
hipError_t launch_rpt(const Bucket* d_bk, int nb, int h, int w, int level, const Taps& tp, float tol, int cap,
                      hipStream_t s)
{
    static std::atomic<uint64_t> attr_done{0};
    const hipError_t e = ensure_dynamic_lds((const void*)k_demons_resident<RAD, RPT>,
                                            (int)res_lds_bytes<RPT>(64 * 16 * RPT), attr_done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_demons_resident<RAD, RPT>), dim3((unsigned)nb), dim3(kResThreads),
                       res_lds_bytes<RPT>(h * w), s, d_bk, level, tp, tol, cap);
    return hipGetLastError();
}

template <int RAD>
hipError_t launch_rad(const Bucket* d_bk, int nb, int h, int w, int level, const Taps& tp, float tol, int cap,
                      hipStream_t s)
{
    if (h <= 16) return launch_rpt<RAD, 1>(d_bk, nb, h, w, level, tp, tol, cap, s);
    if (h <= 32) return launch_rpt<RAD, 2>(d_bk, nb, h, w, level, tp, tol, cap, s);
    return launch_rpt<RAD, 4>(d_bk, nb, h, w, level, tp, tol, cap, s);
}

}  // namespace

bool demons_resident_ok(int h, int w) { return h >= 2 && w >= 2 && h <= 64 && w <= 64; }

hipError_t launch_demons_resident(const Bucket* d_bk, const Bucket& hb, int level, const float* taps, int radius,
                                  float tol, int cap, hipStream_t s)
{
    const int h = hb.lh[level], w = hb.lw[level];
    if (!demons_resident_ok(h, w) || hb.nb <= 0) return hipErrorInvalidValue;
    Taps tp;
    for (int i = 0; i < 2 * kMaxRadius + 1; i++) tp.w[i] = i <= 2 * radius ? taps[i] : 0.0f;
    switch (radius) {
    case 0: return launch_rad<0>(d_bk, hb.nb, h, w, level, tp, tol, cap, s);
    case 1: return launch_rad<1>(d_bk, hb.nb, h, w, level, tp, tol, cap, s);
    case 2: return launch_rad<2>(d_bk, hb.nb, h, w, level, tp, tol, cap, s);
    case 3: return launch_rad<3>(d_bk, hb.nb, h, w, level, tp, tol, cap, s);
    case 4: return launch_rad<4>(d_bk, hb.nb, h, w, level, tp, tol, cap, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ebsd
