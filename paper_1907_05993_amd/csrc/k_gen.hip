// Synthetic Kikuchi-pattern pairs on the GPU: training and benchmark inputs
// with ground-truth labels for the warm-start network and the registration.
//
// A pattern is the gnomonic view of FCC band profiles plus a linear
// background; the test pattern is rendered by pull-back through F^-1, so its
// exact shift field is the projective model of Eq. (2) of arXiv:1907.05993,
// q(x) = pi(F r(x)) - x.  Each pattern is scaled to a mean count and Poisson
// noise is drawn with a counter-based generator (Philox4x32-10, Salmon et al.
// 2011) and the PTRS transformed-rejection sampler (Hormann 1993), so every
// pixel of every pattern is reproducible on its own, independent of the
// launch shape.  Rendering is FP64; outputs are fp32.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <new>
#include <set>
#include <tuple>
#include <vector>

#include "../../include/ebsd.h"
#include "ebsd_internal.h"

namespace {

constexpr int kMaxBands = 32;
constexpr int kGenThreads = 256;
constexpr int kGenBlocks = 32;  // blocks per pattern

static_assert(kMaxBands <= 32, "band masks of 32 bits");

struct BandTable {
    double n[kMaxBands][3];  // unit plane normals (crystal frame)
    double theta[kMaxBands]; // Bragg half-width (rad)
    double sin_theta[kMaxBands];
    int count;
};

struct GenPair {
    double G[9];     // crystal -> detector
    double Finv[9];  // inverse of the applied deformation gradient
    double F[9];
    double gx, gy, counts;
    uint32_t key0, key1;
    int32_t noise, bands;
};

// ---- Philox4x32-10 ----------------------------------------------------------------
__device__ inline void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1)
{
    for (int r = 0; r < 10; r++) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
        const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
        const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0;
        c[1] = lo1;
        c[2] = n2;
        c[3] = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// Two doubles in [0, 1) with 53 random bits each from the Philox block of
// counter (pixel, attempt, stream, 0).
__device__ inline void uniforms2(uint32_t p, uint32_t attempt, uint32_t stream, uint32_t k0, uint32_t k1,
                                 double& u, double& v)
{
    uint32_t c[4] = {p, attempt, stream, 0u};
    philox4x32_10(c, k0, k1);
    const double s = 1.0 / 9007199254740992.0;  // 2^-53
    u = (double)(((uint64_t)(c[0] >> 5) << 26) | (uint64_t)(c[1] >> 6)) * s;
    v = (double)(((uint64_t)(c[2] >> 5) << 26) | (uint64_t)(c[3] >> 6)) * s;
}

// Poisson(lam): PTRS for lam >= 10, inversion by sequential search below.
// At most kMaxTries proposals (PTRS accepts more than 90% of them; after the
// cap the rounded mean is returned).
constexpr int kMaxTries = 64;

// Constants of PTRS at mean lam >= 10 that its first test needs.
struct Ptrs {
    double a, b, vr;
};
__device__ inline Ptrs ptrs_of(double lam)
{
    Ptrs q;
    q.b = 0.931 + 2.53 * sqrt(lam);
    q.a = -0.059 + 0.02483 * q.b;
    q.vr = 0.9277 - 3.6224 / (q.b - 2.0);
    return q;
}

// Proposal t of the draw.  Quick: inside the squeeze, which takes no logarithms
// (86 % of the proposals at mean 100).
__device__ inline double ptrs_propose(const Ptrs& q, double lam, uint32_t p, uint32_t t, uint32_t stream, uint32_t k0,
                                      uint32_t k1, double& us, double& v, bool& quick)
{
    double u;
    uniforms2(p, t, stream, k0, k1, u, v);
    u -= 0.5;
    us = 0.5 - fabs(u);
    quick = us >= 0.07 && v <= q.vr;
    return floor((2.0 * q.a / us + q.b) * u + lam + 0.43);
}

// log k! of k = 0, 1, ...: the first 16 from a table, then Stirling's series
// (Abramowitz and Stegun 6.1.41; the term left out is below 1e-16 at k = 16).
__device__ inline double log_factorial(double k)
{
    constexpr double kTab[16] = {0.0,
                                 0.0,
                                 0.69314718055994530942,
                                 1.7917594692280550008,
                                 3.1780538303479456197,
                                 4.7874917427820459943,
                                 6.5792512120101009951,
                                 8.5251613610654143002,
                                 10.604602902745250228,
                                 12.801827480081469611,
                                 15.104412573075515295,
                                 17.502307845873885839,
                                 19.987214495661886150,
                                 22.552163853123422886,
                                 25.191221182738681500,
                                 27.899271383840891566};
    if (k < 16.0) return kTab[(int)k];
    const double x = k + 1.0, i = 1.0 / x, i2 = i * i;
    const double c = i * (1.0 / 12 - i2 * (1.0 / 360 - i2 * (1.0 / 1260 - i2 * (1.0 / 1680 - i2 * (1.0 / 1188 -
                          i2 * (691.0 / 360360))))));
    return (x - 0.5) * log(x) - x + 0.91893853320467274178 + c;
}

// The exact test of a proposal outside the squeeze.
__device__ inline bool ptrs_accept(const Ptrs& q, double lam, double k, double us, double v)
{
    if (k < 0.0 || (us < 0.013 && v > us)) return false;
    const double invalpha = 1.1239 + 1.1328 / (q.b - 3.4);
    return log(v) + log(invalpha) - log(q.a / (us * us) + q.b) <= -lam + k * log(lam) - log_factorial(k);
}

// lam < 10
__device__ inline double poisson_search(double lam, uint32_t p, uint32_t stream, uint32_t k0, uint32_t k1)
{
    double u, v;
    uniforms2(p, 0u, stream, k0, k1, u, v);
    double pk = exp(-lam), cdf = pk;
    int k = 0;
    while (u > cdf && k < 1000) {
        k++;
        pk *= lam / (double)k;
        cdf += pk;
    }
    return (double)k;
}

// ---- rendering ----------------------------------------------------------------------

// Tiles of 16 x 16 px per workgroup, 8 x 8 px per wavefront: a compact wavefront
// meets few bands.
constexpr int kGenTile = 16;

// A pattern's bands in the detector frame (LDS).
struct Bands {
    double n[kMaxBands][3];
    double norm[kMaxBands];
};

__device__ void rotate_bands(const BandTable* __restrict__ bt, const double* G, Bands& s)
{
    const int b = threadIdx.x;
    if (b < bt->count) {
        double q = 0.0;
#pragma unroll
        for (int i = 0; i < 3; i++) {
            s.n[b][i] = G[3 * i] * bt->n[b][0] + G[3 * i + 1] * bt->n[b][1] + G[3 * i + 2] * bt->n[b][2];
            q += s.n[b][i] * s.n[b][i];
        }
        s.norm[b] = sqrt(q);
    }
    __syncthreads();
}

__device__ inline void view_ray(const GenPair& g, int which, double x, double y, double xs, double ys, double zs,
                                double& rx, double& ry, double& rz)
{
    rx = x - xs;
    ry = y - ys;
    rz = zs;
    if (which) {
        const double tx = g.Finv[0] * rx + g.Finv[1] * ry + g.Finv[2] * rz;
        const double ty = g.Finv[3] * rx + g.Finv[4] * ry + g.Finv[5] * rz;
        const double tz = g.Finv[6] * rx + g.Finv[7] * ry + g.Finv[8] * rz;
        rx = tx;
        ry = ty;
        rz = tz;
    }
}

// The bands (bit mask, uniform over the wavefront) that a pixel of the wavefront's
// 8 x 8 tile at (x0, y0) can lie in, lane b deciding on band b from the centre ray:
// over the tile the ray moves by at most d, the unit ray by at most 2 d / |r|, and
// the sine by that times |n|.  A band is only left out where this is sure.
__device__ inline uint32_t bands_near(const BandTable* __restrict__ bt, const Bands& s, const GenPair& g, int which,
                                      int x0, int y0, double xs, double ys, double zs)
{
    const int b = threadIdx.x & 63;
    bool keep = false;
    if (b < bt->count) {
        double rx, ry, rz;
        view_ray(g, which, (double)x0 + 3.5, (double)y0 + 3.5, xs, ys, zs, rx, ry, rz);
        double d = 3.5 * 1.4143;
        if (which) {
            const double c0 = sqrt(g.Finv[0] * g.Finv[0] + g.Finv[3] * g.Finv[3] + g.Finv[6] * g.Finv[6]);
            const double c1 = sqrt(g.Finv[1] * g.Finv[1] + g.Finv[4] * g.Finv[4] + g.Finv[7] * g.Finv[7]);
            d = 3.5 * (c0 + c1);
        }
        const double r2 = rx * rx + ry * ry + rz * rz, r = sqrt(r2);
        const double move = 2.0 * d / r;
        const double sine = (s.n[b][0] * rx + s.n[b][1] * ry + s.n[b][2] * rz) / r;
        const double margin = s.norm[b] * (move * (1.0 + 1e-9) + 1e-9);
        // squares far from the limits of the type, here and at every pixel
        const bool sure = r2 > 1e-100 && r2 < 1e100 && move < 1.0 && s.norm[b] < 1e100;
        keep = !(sure && fabs(sine) - margin > bt->sin_theta[b]);
    }
    return (uint32_t)__ballot(keep);
}

__device__ double band_sum(const BandTable* __restrict__ bt, const Bands& s, uint32_t near, double dx, double dy,
                           double dz)
{
    const double inv = 1.0 / sqrt(dx * dx + dy * dy + dz * dz);
    dx *= inv;
    dy *= inv;
    dz *= inv;
    double acc = 0.0;
    for (; near; near &= near - 1) {
        const int b = __builtin_ctz(near);
        const double sine = s.n[b][0] * dx + s.n[b][1] * dy + s.n[b][2] * dz;
        if (fabs(sine) <= bt->sin_theta[b]) acc += 0.5 * (1.0 + cos(M_PI * asin(sine) / bt->theta[b]));
    }
    return acc;
}

// Intensity of the lane's pixel of tile t (0 outside the pattern); all lanes of the
// wavefront call it.  p: the pixel's index, -1 outside.
__device__ inline double tile_intensity(const BandTable* __restrict__ bt, const Bands& s, const GenPair& g, int which,
                                        int t, int tiles_x, int H, int W, double xs, double ys, double zs, int& p)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ty = t / tiles_x, tx = t - ty * tiles_x;
    const int x0 = tx * kGenTile + (wave & 1) * 8, y0 = ty * kGenTile + (wave >> 1) * 8;
    const int x = x0 + (lane & 7), y = y0 + (lane >> 3);
    p = x < W && y < H ? y * W + x : -1;
    const uint32_t near = g.bands ? bands_near(bt, s, g, which, x0, y0, xs, ys, zs) : 0u;
    if (p < 0) return 0.0;
    const double bg =
        1.0 + 0.2 * (g.gx * ((double)x / (double)(W - 1) - 0.5) + g.gy * ((double)y / (double)(H - 1) - 0.5));
    if (!g.bands) return bg;
    double rx, ry, rz;
    view_ray(g, which, (double)x, (double)y, xs, ys, zs, rx, ry, rz);
    return bg + 0.5 * band_sum(bt, s, near, rx, ry, rz);
}

// Pass 1: per-block partial sums of the unscaled intensity (fixed tree order).
// blockIdx.y = 2 * pair + (0 reference, 1 test).  Bound: FP64 vector ALU.
__global__ void __launch_bounds__(kGenThreads)
k_gen_sum(const GenPair* __restrict__ gp, const BandTable* __restrict__ bt, int H, int W, double xs, double ys,
          double zs, int tiles_x, int tiles, double* __restrict__ part)
{
    __shared__ Bands bands;
    __shared__ double sh[kGenThreads];
    const int pat = blockIdx.y;
    const GenPair& g = gp[pat >> 1];
    rotate_bands(bt, g.G, bands);
    double sum = 0.0;
    for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
        int p;
        sum += tile_intensity(bt, bands, g, pat & 1, t, tiles_x, H, W, xs, ys, zs, p);
    }
    sh[threadIdx.x] = sum;
    __syncthreads();
    for (int s = kGenThreads / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[(int64_t)pat * kGenBlocks + blockIdx.x] = sh[0];
}

// Pass 2: scale to the mean count, Poisson noise, fp32 store.  The intensity is
// computed again (less than the 16 B per pixel that keeping it would move, and no
// memory for it).  Draws that are not settled by a first quick proposal wait in LDS
// and are taken 256 at a time, one exact test and one more proposal each, until
// they are settled: drawn in place, a few lanes held every wavefront for several
// proposals.  64 pairs of 256 x 256: k_gen_sum 286 -> 115 us (all 25 bands at each
// pixel before), k_gen_write 746 -> 275 us.
constexpr int kGenQueue = 2 * kGenThreads;  // at most kGenThreads - 1 wait before a tile
static_assert(kMaxTries <= 64, "proposal number in the 7 bits above a pixel index of 24");
__global__ void __launch_bounds__(kGenThreads) __attribute__((amdgpu_waves_per_eu(4)))
k_gen_write(const GenPair* __restrict__ gp, const BandTable* __restrict__ bt, int H, int W, double xs, double ys,
            double zs, int tiles_x, int tiles, const double* __restrict__ part, float* __restrict__ ref,
            float* __restrict__ test)
{
    __shared__ Bands bands;
    __shared__ double wait_v[kGenQueue];
    __shared__ uint32_t wait_p[kGenQueue];  // pixel | proposal << 24
    __shared__ int waiting;
    const int pat = blockIdx.y;
    const uint32_t which = pat & 1;
    const GenPair& g = gp[pat >> 1];
    if (threadIdx.x == 0) waiting = 0;
    rotate_bands(bt, g.G, bands);
    const int64_t np = (int64_t)H * W;
    double tot = 0.0;
    for (int b = 0; b < (int)gridDim.x; b++) tot += part[(int64_t)pat * kGenBlocks + b];
    const double scale = g.counts > 0.0 ? g.counts / (tot / (double)np) : 1.0;
    float* dst = (which ? test : ref) + (int64_t)(pat >> 1) * np;
    const auto push = [&](bool mine, double v, uint32_t p) {
        const uint64_t m = __ballot(mine);
        int at = 0;
        if ((threadIdx.x & 63) == 0 && m) at = atomicAdd(&waiting, (int)__popcll(m));
        at = __builtin_amdgcn_readfirstlane(at) + (int)__popcll(m & ((1ull << (threadIdx.x & 63)) - 1));
        if (mine) {
            wait_v[at] = v;
            wait_p[at] = p;
        }
    };
    for (int t = blockIdx.x; t < tiles; t += gridDim.x) {  // uniform over the workgroup
        int p;
        double v = tile_intensity(bt, bands, g, (int)which, t, tiles_x, H, W, xs, ys, zs, p) * scale;
        bool done = true;
        double k = v;
        if (g.noise && p >= 0) {
            k = 0.0;
            if (v >= 10.0) {
                double us, r;
                k = ptrs_propose(ptrs_of(v), v, (uint32_t)p, 0u, which, g.key0, g.key1, us, r, done);
            } else if (v > 0.0) {
                done = false;
            }
        }
        if (p >= 0 && done) dst[p] = (float)k;
        if (!g.noise) continue;
        push(!done, v, (uint32_t)p);
        __syncthreads();
        const bool last = t + (int)gridDim.x >= tiles;
        for (int n = waiting; n >= kGenThreads || (last && n > 0);) {  // uniform
            const int i = max(n - kGenThreads, 0) + (int)threadIdx.x;
            double lam = 0.0;
            uint32_t e = 0;
            if (i < n) {
                lam = wait_v[i];
                e = wait_p[i];
            }
            __syncthreads();
            if (threadIdx.x == 0) waiting = max(n - kGenThreads, 0);
            __syncthreads();
            bool again = false;
            if (i < n) {
                const uint32_t q = e & 0xffffffu;
                double out;
                if (lam < 10.0) {
                    out = poisson_search(lam, q, which, g.key0, g.key1);
                } else {
                    const Ptrs c = ptrs_of(lam);
                    uint32_t tr = e >> 24;
                    double us, r;
                    bool quick;
                    out = ptrs_propose(c, lam, q, tr, which, g.key0, g.key1, us, r, quick);
                    if (!ptrs_accept(c, lam, out, us, r)) {
                        tr++;
                        e = q | tr << 24;
                        if (tr == (uint32_t)kMaxTries) {
                            out = floor(lam + 0.5);
                        } else {
                            out = ptrs_propose(c, lam, q, tr, which, g.key0, g.key1, us, r, quick);
                            again = !quick;
                        }
                    }
                }
                if (!again) dst[q] = (float)out;
            }
            push(again, lam, e);
            __syncthreads();
            n = waiting;
        }
        __syncthreads();
    }
}

// Labels: q = pi(F r(x)) - x at the coarse grid points x = 4 i + 1.5, [H/4][W/4][2].
__global__ void k_gen_labels(const GenPair* __restrict__ gp, int H, int W, double xs, double ys, double zs,
                             float* __restrict__ label)
{
    const int pair = blockIdx.y;
    const int gh = H / 4, gw = W / 4;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= gh * gw) return;
    const GenPair& g = gp[pair];
    const double x = 4.0 * (double)(i % gw) + 1.5, y = 4.0 * (double)(i / gw) + 1.5;
    const double rx = x - xs, ry = y - ys;
    const double v0 = g.F[0] * rx + g.F[1] * ry + g.F[2] * zs;
    const double v1 = g.F[3] * rx + g.F[4] * ry + g.F[5] * zs;
    const double v2 = g.F[6] * rx + g.F[7] * ry + g.F[8] * zs;
    float* out = label + ((int64_t)pair * gh * gw + i) * 2;
    out[0] = (float)(xs + zs * v0 / v2 - x);
    out[1] = (float)(ys + zs * v1 / v2 - y);
}

// The 25 distinct plane normals of the FCC families {111}, {200}, {220},
// {311}; half-width asin((lambda / 2a) |hkl|) with lambda / a = 0.02438
// (20 kV electrons on nickel).
BandTable fcc_bands()
{
    BandTable bt{};
    const int fam[4][3] = {{1, 1, 1}, {2, 0, 0}, {2, 2, 0}, {3, 1, 1}};
    int nb = 0;
    for (auto& f : fam) {
        std::set<std::tuple<int, int, int>> seen;
        int perm[3] = {f[0], f[1], f[2]};
        std::sort(perm, perm + 3);
        do {
            for (int sg = 0; sg < 8; sg++) {
                int v[3];
                for (int j = 0; j < 3; j++) v[j] = (sg >> j & 1) ? -perm[j] : perm[j];
                int first = v[0] != 0 ? v[0] : (v[1] != 0 ? v[1] : v[2]);
                if (first < 0)
                    for (int& c : v) c = -c;
                seen.insert(std::make_tuple(v[0], v[1], v[2]));
            }
        } while (std::next_permutation(perm, perm + 3));
        for (auto& t : seen) {
            const double h = std::get<0>(t), k = std::get<1>(t), l = std::get<2>(t);
            const double gl = std::sqrt(h * h + k * k + l * l);
            bt.n[nb][0] = h / gl;
            bt.n[nb][1] = k / gl;
            bt.n[nb][2] = l / gl;
            bt.theta[nb] = std::asin(0.02438 / 2.0 * gl);
            bt.sin_theta[nb] = std::sin(bt.theta[nb]);
            nb++;
        }
    }
    bt.count = nb;
    return bt;
}

bool inv3(const double* A, double* B)
{
    const double c00 = A[4] * A[8] - A[5] * A[7], c01 = A[5] * A[6] - A[3] * A[8], c02 = A[3] * A[7] - A[4] * A[6];
    const double det = A[0] * c00 + A[1] * c01 + A[2] * c02;
    if (!(std::fabs(det) > 0.0) || !std::isfinite(det)) return false;
    const double id = 1.0 / det;
    B[0] = c00 * id;
    B[1] = (A[2] * A[7] - A[1] * A[8]) * id;
    B[2] = (A[1] * A[5] - A[2] * A[4]) * id;
    B[3] = c01 * id;
    B[4] = (A[0] * A[8] - A[2] * A[6]) * id;
    B[5] = (A[2] * A[3] - A[0] * A[5]) * id;
    B[6] = c02 * id;
    B[7] = (A[1] * A[6] - A[0] * A[7]) * id;
    B[8] = (A[0] * A[4] - A[1] * A[3]) * id;
    return true;
}

struct DevMem {
    void* p = nullptr;
    ~DevMem()
    {
        if (p) (void)hipFree(p);
    }
};

}  // namespace

extern "C" int ebsd_gen_pairs(const ebsd_gen_spec* specs, int32_t n, int32_t H, int32_t W, double pc_x,
                              double pc_y, double pc_z, float* ref, float* test, float* label, void* stream)
{
    if (n < 0 || (n > 0 && (!specs || !ref || !test))) return EBSD_EINVAL;
    if (H < 8 || W < 8 || H > 4096 || W > 4096 || (label && (H % 4 || W % 4))) return EBSD_ESHAPE;
    if (!(pc_z > 0.0) || !std::isfinite(pc_x) || !std::isfinite(pc_y) || !std::isfinite(pc_z)) return EBSD_EINVAL;
    if (n == 0) return EBSD_OK;
    std::vector<char> up;
    try {
        up.resize(sizeof(BandTable) + sizeof(GenPair) * (size_t)n);
        *reinterpret_cast<BandTable*>(up.data()) = fcc_bands();
    } catch (const std::bad_alloc&) {
        return EBSD_ENOMEM;
    }
    for (int i = 0; i < n; i++) {
        const ebsd_gen_spec& s = specs[i];
        GenPair& g = reinterpret_cast<GenPair*>(up.data() + sizeof(BandTable))[i];
        for (int j = 0; j < 9; j++) {
            if (!std::isfinite(s.G[j]) || !std::isfinite(s.F[j])) return EBSD_EINVAL;
            g.G[j] = s.G[j];
            g.F[j] = s.F[j];
        }
        if (!inv3(g.F, g.Finv)) return EBSD_EINVAL;
        if (!std::isfinite(s.gx) || !std::isfinite(s.gy) || !std::isfinite(s.counts)) return EBSD_EINVAL;
        g.gx = s.gx;
        g.gy = s.gy;
        g.counts = s.counts;
        g.key0 = s.key[0];
        g.key1 = s.key[1];
        g.noise = s.noise != 0;
        g.bands = s.bands != 0;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    ebsd::DeviceWideLock lk(ebsd::capture_mutex());  // the buffers' frees wait for the device
    // one allocation and one upload: band table, pairs, partial sums
    const size_t up_bytes = sizeof(BandTable) + sizeof(GenPair) * (size_t)n;
    DevMem mem;
    if (hipMalloc(&mem.p, up_bytes + sizeof(double) * 2 * (size_t)n * kGenBlocks) != hipSuccess) {
        (void)hipGetLastError();
        return EBSD_ENOMEM;
    }
    if (hipMemcpyAsync(mem.p, up.data(), up_bytes, hipMemcpyHostToDevice, st) != hipSuccess) return EBSD_EDEVICE;
    const double xs = pc_x * W - 0.5, ys = pc_y * H - 0.5, zs = pc_z * W;
    const BandTable* btp = static_cast<const BandTable*>(mem.p);
    const GenPair* gp = reinterpret_cast<const GenPair*>(btp + 1);
    double* part = reinterpret_cast<double*>(static_cast<char*>(mem.p) + up_bytes);
    const int tiles_x = (W + kGenTile - 1) / kGenTile, tiles = tiles_x * ((H + kGenTile - 1) / kGenTile);
    for (int c0 = 0; c0 < n; c0 += 16384) {  // 2 patterns per pair on grid.y (<= 65535)
        const int cnt = std::min(16384, n - c0);
        const dim3 grid(std::min(kGenBlocks, tiles), 2 * cnt);
        hipLaunchKernelGGL(k_gen_sum, grid, dim3(kGenThreads), 0, st, gp + c0, btp, H, W, xs, ys, zs,
                           tiles_x, tiles, part + (size_t)2 * c0 * kGenBlocks);
        hipLaunchKernelGGL(k_gen_write, grid, dim3(kGenThreads), 0, st, gp + c0, btp, H, W, xs, ys, zs,
                           tiles_x, tiles, part + (size_t)2 * c0 * kGenBlocks, ref + (int64_t)c0 * H * W, test + (int64_t)c0 * H * W);
        if (label) {
            const int ng = (H / 4) * (W / 4);
            hipLaunchKernelGGL(k_gen_labels, dim3((ng + 255) / 256, cnt), dim3(256), 0, st, gp + c0, H, W, xs, ys, zs,
                               label + (int64_t)c0 * ng * 2);
        }
    }
    if (hipGetLastError() != hipSuccess) return EBSD_EDEVICE;
    // the temporaries are freed on return: wait for the kernels that read them
    return hipStreamSynchronize(st) == hipSuccess ? EBSD_OK : EBSD_EDEVICE;
}
