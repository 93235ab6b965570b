// Reconstruction-loop kernels (Sec. III-B: gradient descent on the
// Gaussians with densification and pruning after Sec. II-B) and evaluation
// metrics (Sec. III-B, "Evaluation Metrics"). Contracts in
// include/sdgr_train.h.
//
// All of it is memory- or launch-bound elementwise work except the
// nearest-neighbour search (exhaustive) and the SSIM windows (separable, in
// FP64).
#include "common.hpp"
#include "sdgr_train.h"

#include <math.h>

#include <algorithm>
#include <cmath>
#include <string>

namespace sdgr {
namespace {

inline unsigned blocks_for(int64_t n, int b, unsigned cap = 1u << 20)
{
    const int64_t g = (n + b - 1) / b;
    return (unsigned)(g < 1 ? 1 : (g > cap ? cap : g));
}

// ------------------------------------------------------------------ Adam

struct AdamGroupDev {
    float* p;
    const float* g;
    float* m;
    float* v;
    int64_t start, count;
    float lr;
    int32_t log_space;
    float lo, hi;
    int32_t clamp;
};

struct AdamArgs {
    AdamGroupDev grp[SDGR_ADAM_MAX_GROUPS];
    int32_t ngroups;
    float b1, b2, eps;
    float bc1, bc2;   // 1 / (1 - b1^t), 1 / (1 - b2^t)
};

__global__ void __launch_bounds__(256) k_adam(AdamArgs a, int64_t total)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        int k = 0;
        while (k + 1 < a.ngroups && e >= a.grp[k + 1].start) ++k;
        const AdamGroupDev& G = a.grp[k];
        const int64_t i = e - G.start;
        float x = G.p[i];
        float g = G.g[i];
        if (G.log_space) g *= x;   // d/d(log x) = x d/dx
        const float m = a.b1 * G.m[i] + (1.0f - a.b1) * g;
        const float v = a.b2 * G.v[i] + (1.0f - a.b2) * g * g;
        const float step = G.lr * (m * a.bc1) / (sqrtf(v * a.bc2) + a.eps);
        x = G.log_space ? x * expf(-step) : x - step;
        if (G.clamp) x = fminf(fmaxf(x, G.lo), G.hi);
        G.p[i] = x;
        G.m[i] = m;
        G.v[i] = v;
    }
}

// ------------------------------------------------------ densify statistics

__global__ void __launch_bounds__(256)
k_densify_stats(const float* __restrict__ dmu, int64_t n, float* __restrict__ acc,
                float* __restrict__ cnt, float* __restrict__ dir)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float g0 = dmu[3 * i], g1 = dmu[3 * i + 1], g2 = dmu[3 * i + 2];
    const float nn = sqrtf(g0 * g0 + g1 * g1 + g2 * g2);
    if (!(nn > 0.0f)) return;
    acc[i] += nn;
    cnt[i] += 1.0f;
    dir[3 * i] += g0;
    dir[3 * i + 1] += g1;
    dir[3 * i + 2] += g2;
}

// ---------------------------------------------------- densify and prune

constexpr uint8_t ACT_KEEP = 0, ACT_PRUNE = 1, ACT_CLONE = 2, ACT_SPLIT = 3;

struct DensifyArgs {
    sdgr_gaussian_set in, out;
    sdgr_densify_config cfg;
    int64_t n;
};

__device__ __forceinline__ uint32_t outputs_of(uint8_t a)
{
    return a == ACT_PRUNE ? 0u : (a == ACT_KEEP ? 1u : 2u);
}

__device__ __forceinline__ float max3(const float* s)
{
    return fmaxf(s[0], fmaxf(s[1], s[2]));
}

// Action of each Gaussian (FP32 decisions) and the output count of each
// block of 256.
__global__ void __launch_bounds__(256)
k_densify_count(DensifyArgs a, const float* __restrict__ acc, const float* __restrict__ cnt,
                uint8_t* __restrict__ act, uint32_t* __restrict__ bsum)
{
    __shared__ uint32_t s_w[4];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t nout = 0u;
    if (i < a.n) {
        const float smax = max3(a.in.scales + 3 * i);
        uint8_t c = ACT_KEEP;
        if (a.in.ext[i] < a.cfg.kappa_min || 3.0f * smax > a.cfg.max_radius)
            c = ACT_PRUNE;
        else if (cnt[i] > 0.0f && __fdiv_rn(acc[i], cnt[i]) >= a.cfg.grad_threshold)
            c = smax > a.cfg.split_scale ? ACT_SPLIT : ACT_CLONE;
        act[i] = c;
        nout = outputs_of(c);
    }
    uint32_t total;
    block_excl_scan_256(nout, s_w, total);
    if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

// Exclusive scan of the block counts (one workgroup: each thread sums a
// contiguous run, the runs' sums are scanned in LDS) and the total.
__global__ void __launch_bounds__(1024)
k_densify_scan(const uint32_t* __restrict__ bsum, int64_t nb, uint32_t* __restrict__ boff,
               int64_t* __restrict__ n_out)
{
    __shared__ uint32_t s[1024];
    const int64_t per = (nb + 1023) / 1024;
    const int64_t b0 = threadIdx.x * per, b1 = min(nb, b0 + per);
    uint32_t run = 0u;
    for (int64_t b = b0; b < b1; ++b) run += bsum[b];
    s[threadIdx.x] = run;
    __syncthreads();
    // Hillis-Steele inclusive scan of the 1024 run sums
    for (int d = 1; d < 1024; d <<= 1) {
        const uint32_t t = threadIdx.x >= (unsigned)d ? s[threadIdx.x - d] : 0u;
        __syncthreads();
        s[threadIdx.x] += t;
        __syncthreads();
    }
    uint32_t off = s[threadIdx.x] - run;
    for (int64_t b = b0; b < b1; ++b) {
        boff[b] = off;
        off += bsum[b];
    }
    if (threadIdx.x == 1023) *n_out = (int64_t)s[1023];
}

__device__ __forceinline__ void copy_row(const float* src, float* dst, int64_t from, int64_t to,
                                         int width)
{
    if (!src) return;
    for (int k = 0; k < width; ++k) dst[to * width + k] = src[from * width + k];
}

__device__ __forceinline__ void zero_row(float* dst, int64_t to, int width)
{
    if (!dst) return;
    for (int k = 0; k < width; ++k) dst[to * width + k] = 0.0f;
}

// Write Gaussian i's outputs at slot o (and o + 1): the parameters, with
// the means and scales of copies and children changed, and the moments
// (copied for the original, zero for new Gaussians).
__device__ void emit(const DensifyArgs& a, int64_t i, int64_t o, const float* mu,
                     const float* sc, bool fresh)
{
    const sdgr_gaussian_set& I = a.in;
    const sdgr_gaussian_set& O = a.out;
    for (int k = 0; k < 3; ++k) {
        O.means[3 * o + k] = mu[k];
        O.scales[3 * o + k] = sc[k];
    }
    copy_row(I.quats, O.quats, i, o, 4);
    copy_row(I.amp, O.amp, i, o, 1);
    copy_row(I.ext, O.ext, i, o, 1);
    copy_row(I.sh, O.sh, i, o, I.sh_coeffs);
    struct M { const float* im; const float* iv; float* om; float* ov; int w; };
    const M ms[6] = {{I.m_means, I.v_means, O.m_means, O.v_means, 3},
                     {I.m_scales, I.v_scales, O.m_scales, O.v_scales, 3},
                     {I.m_quats, I.v_quats, O.m_quats, O.v_quats, 4},
                     {I.m_amp, I.v_amp, O.m_amp, O.v_amp, 1},
                     {I.m_ext, I.v_ext, O.m_ext, O.v_ext, 1},
                     {I.m_sh, I.v_sh, O.m_sh, O.v_sh, I.sh_coeffs}};
    for (int g = 0; g < 6; ++g) {
        if (!ms[g].om) continue;
        if (fresh) {
            zero_row(ms[g].om, o, ms[g].w);
            zero_row(ms[g].ov, o, ms[g].w);
        } else {
            copy_row(ms[g].im, ms[g].om, i, o, ms[g].w);
            copy_row(ms[g].iv, ms[g].ov, i, o, ms[g].w);
        }
    }
}

__global__ void __launch_bounds__(256)
k_densify_apply(DensifyArgs a, const uint8_t* __restrict__ act,
                const uint32_t* __restrict__ boff, const float* __restrict__ dir)
{
    __shared__ uint32_t s_w[4];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint8_t c = i < a.n ? act[i] : ACT_PRUNE;
    uint32_t total;
    const uint32_t ex = block_excl_scan_256(outputs_of(c), s_w, total);
    if (i >= a.n || c == ACT_PRUNE) return;
    const int64_t o = (int64_t)boff[blockIdx.x] + ex;
    const float* mu = a.in.means + 3 * i;
    const float* sc = a.in.scales + 3 * i;
    if (c != ACT_SPLIT) emit(a, i, o, mu, sc, false);   // the original stays
    if (c == ACT_KEEP) return;
    // unit accumulated gradient (zero if there is none)
    const float d0 = dir[3 * i], d1 = dir[3 * i + 1], d2 = dir[3 * i + 2];
    const float dn = sqrtf(d0 * d0 + d1 * d1 + d2 * d2);
    const float inv = dn > 0.0f ? 1.0f / dn : 0.0f;
    const float gh[3] = {d0 * inv, d1 * inv, d2 * inv};
    const float smax = max3(sc);
    if (c == ACT_CLONE) {
        const float m2[3] = {mu[0] - smax * gh[0], mu[1] - smax * gh[1], mu[2] - smax * gh[2]};
        emit(a, i, o + 1, m2, sc, true);
        return;
    }
    // split: the largest axis is the column of the rotation for the largest scale
    const float* q = a.in.quats + 4 * i;
    const float qn = rsqrtf(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    const float w = q[0] * qn, x = q[1] * qn, y = q[2] * qn, z = q[3] * qn;
    const int ax = (sc[0] >= sc[1] && sc[0] >= sc[2]) ? 0 : (sc[1] >= sc[2] ? 1 : 2);
    float e[3];
    if (ax == 0) {
        e[0] = 1.f - 2.f * (y * y + z * z); e[1] = 2.f * (x * y + w * z); e[2] = 2.f * (x * z - w * y);
    } else if (ax == 1) {
        e[0] = 2.f * (x * y - w * z); e[1] = 1.f - 2.f * (x * x + z * z); e[2] = 2.f * (y * z + w * x);
    } else {
        e[0] = 2.f * (x * z + w * y); e[1] = 2.f * (y * z - w * x); e[2] = 1.f - 2.f * (x * x + y * y);
    }
    const float f = 1.0f / a.cfg.split_factor;
    const float cs[3] = {sc[0] * f, sc[1] * f, sc[2] * f};
    const float cmax = max3(cs);
    for (int side = 0; side < 2; ++side) {
        const float sg = side == 0 ? 1.0f : -1.0f;
        float m2[3];
        for (int k = 0; k < 3; ++k) m2[k] = mu[k] + sg * smax * e[k] - cmax * gh[k];
        emit(a, i, o + side, m2, cs, true);
    }
}

// ----------------------------------------------------------------- metrics

// Exhaustive nearest neighbours, a query per lane; the reference points are
// the same for the whole wave, so they come as scalar loads and cost the VALU
// nothing. Bound by the VALU: 6.6 instructions a pair (three differences, a
// product, two multiply-adds, half a three-operand minimum), at 7.2 * 10^12
// pairs/s for 31k by 20k points and 9.3 * 10^12 for 4M by 10k, of the 11.9 *
// 10^12 that the card's 157 TFLOP/s (128 lanes to a CU and cycle) allow.
// The references are split over grid y until there are NN_WAVES waves, the
// parts' minima meeting in d2 (distances are never negative, so their bits
// order as unsigned; d2 starts at infinity then). Many short waves also leave
// no long last round: in 4096 waves, 4 to a SIMD, 150k by 100k points took 3235
// us, where every third SIMD had a wave more than the others, in 32768 1621;
// 31k by 20k 107 and 87, 200k by 100k 3650 and 2175, 600k by 50k 3954 and 3318
// (65536: 1565, 89, 2118, 3182). A block of 256 per 256 queries with the
// references staged in LDS took 2613, 369, 3479 and 3985. A search over points
// sorted into cells, skipping boxes further than the minima found, gave the
// same results in 424 us at 31k by 20k.
constexpr int NN_PART = 128;       // fewest references of a part: 16 of the loop's batches
constexpr unsigned NN_WAVES = 32768;   // (also bounds grid y, which takes 65535)

__global__ void __launch_bounds__(WAVE)
k_nearest_sq(const float* __restrict__ q, int64_t nq, const float* __restrict__ ref, int64_t nr,
             int64_t per, float* __restrict__ d2)
{
    const int64_t i = (int64_t)blockIdx.x * WAVE + threadIdx.x;
    const int64_t j = min(i, nq - 1);
    const float qx = q[3 * j], qy = q[3 * j + 1], qz = q[3 * j + 2];
    const int64_t t0 = (int64_t)blockIdx.y * per, t1 = min(nr, t0 + per);
    float best = INFINITY;
#pragma unroll 8
    for (int64_t t = t0; t < t1; ++t) {
        const float dx = qx - ref[3 * t], dy = qy - ref[3 * t + 1], dz = qz - ref[3 * t + 2];
        best = fminf(best, dx * dx + dy * dy + dz * dz);
    }
    if (i >= nq) return;
    if (gridDim.y == 1) d2[i] = best;
    else atomicMin(reinterpret_cast<unsigned int*>(d2) + i, __float_as_uint(best));
}

__global__ void __launch_bounds__(256) k_fill_f32(float* p, float v, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// --------------------------------------------------------- image metrics

constexpr int SSIM_WIN = 11;
// A workgroup takes SSIM_TX x SSIM_TY window positions: the pixels under them
// in LDS, the window's sums of x, y, x^2, y^2 and x y along the rows, then
// along the columns, all in FP64 (where the moments' differences need no
// second pass over the 121 taps). A workgroup per image, a thread per position
// over all taps twice in FP32: the call took 140 us for 24 images of 64 x 64
// (24 workgroups, four host synchronisations), now 47 (168 workgroups and one,
// the read of the results).
constexpr int SSIM_TX = 32, SSIM_TY = 8;
constexpr int SSIM_PX = SSIM_TX + SSIM_WIN - 1, SSIM_PY = SSIM_TY + SSIM_WIN - 1;

// A workgroup's part of an image's metrics.
struct MetricsPart {
    double ssim, err;
    float max;
    float pad;
};

// Largest value, NaN if there is one (as torch's max).
__device__ __forceinline__ float max_or_nan(float a, float b)
{
    return a != a ? a : (b != b ? b : fmaxf(a, b));
}

constexpr int RANGE_PARTS = 256;

__global__ void __launch_bounds__(256)
k_max_parts(const float* __restrict__ a, int64_t n, float* __restrict__ parts)
{
    __shared__ float s_m[4];
    float m = -INFINITY;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        m = max_or_nan(m, a[i]);
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) m = max_or_nan(m, __shfl_xor(m, d, WAVE));
    if (lane_id() == 0) s_m[threadIdx.x / WAVE] = m;
    __syncthreads();
    if (threadIdx.x == 0)
        parts[blockIdx.x] = max_or_nan(max_or_nan(s_m[0], s_m[1]), max_or_nan(s_m[2], s_m[3]));
}

struct MetricsShared {
    float x[SSIM_PY][SSIM_PX], y[SSIM_PY][SSIM_PX];
    double row[5][SSIM_PY][SSIM_TX];
    double win[SSIM_WIN];
    double a[4], b[4];
    float m[4];
};

// The part of window positions (tx, ty) in units of the tile, and the error
// and maximum of the pixels it owns (the last tiles own the rest of a row or
// column); the whole workgroup calls, thread 0 gets the result.
__device__ MetricsPart metrics_tile(MetricsShared& S, const float* __restrict__ X,
                                    const float* __restrict__ Y, int h, int w, int tx, int ty,
                                    double c1, double c2)
{
    const int vw = w - SSIM_WIN + 1, vh = h - SSIM_WIN + 1;
    const int c0 = tx * SSIM_TX, r0 = ty * SSIM_TY;
    const int own_c = (tx + 1) * SSIM_TX >= vw ? w - c0 : SSIM_TX;
    const int own_r = (ty + 1) * SSIM_TY >= vh ? h - r0 : SSIM_TY;
    double err = 0.0, acc = 0.0;
    float mx = -INFINITY;
    __syncthreads();   // the tile before is done with S
    for (int k = threadIdx.x; k < SSIM_PX * SSIM_PY; k += blockDim.x) {
        const int r = k / SSIM_PX, c = k % SSIM_PX;
        const bool in = r0 + r < h && c0 + c < w;
        const float x = in ? X[(int64_t)(r0 + r) * w + c0 + c] : 0.0f;
        const float y = in ? Y[(int64_t)(r0 + r) * w + c0 + c] : 0.0f;
        S.x[r][c] = x;
        S.y[r][c] = y;
        if (r < own_r && c < own_c) {
            const float d = x - y;
            err += (double)d * d;
            mx = fmaxf(mx, y);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < SSIM_PY * SSIM_TX; k += blockDim.x) {
        const int r = k / SSIM_TX, c = k % SSIM_TX;
        double sx = 0.0, sy = 0.0, xx = 0.0, yy = 0.0, xy = 0.0;
#pragma unroll
        for (int t = 0; t < SSIM_WIN; ++t) {
            const double x = S.x[r][c + t], y = S.y[r][c + t];
            const double wx = S.win[t] * x, wy = S.win[t] * y;
            sx += wx;
            sy += wy;
            xx += wx * x;
            yy += wy * y;
            xy += wx * y;
        }
        S.row[0][r][c] = sx;
        S.row[1][r][c] = sy;
        S.row[2][r][c] = xx;
        S.row[3][r][c] = yy;
        S.row[4][r][c] = xy;
    }
    __syncthreads();
    for (int k = threadIdx.x; k < SSIM_TX * SSIM_TY; k += blockDim.x) {
        const int r = k / SSIM_TX, c = k % SSIM_TX;
        if (r0 + r >= vh || c0 + c >= vw) continue;
        double s[5] = {};
#pragma unroll
        for (int t = 0; t < SSIM_WIN; ++t)
#pragma unroll
            for (int q = 0; q < 5; ++q) s[q] += S.win[t] * S.row[q][r + t][c];
        const double ma = s[0], mb = s[1];
        const double va = s[2] - ma * ma, vb = s[3] - mb * mb, cv = s[4] - ma * mb;
        acc += ((2.0 * ma * mb + c1) * (2.0 * cv + c2)) /
               ((ma * ma + mb * mb + c1) * (va + vb + c2));
    }
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        acc += __shfl_xor(acc, d, WAVE);
        err += __shfl_xor(err, d, WAVE);
        mx = fmaxf(mx, __shfl_xor(mx, d, WAVE));
    }
    const int wv = threadIdx.x / WAVE;
    if (lane_id() == 0) {
        S.a[wv] = acc;
        S.b[wv] = err;
        S.m[wv] = mx;
    }
    __syncthreads();
    return MetricsPart{(S.a[0] + S.a[1]) + (S.a[2] + S.a[3]),
                       (S.b[0] + S.b[1]) + (S.b[2] + S.b[3]),
                       fmaxf(fmaxf(S.m[0], S.m[1]), fmaxf(S.m[2], S.m[3])), 0.0f};
}

// One workgroup per tile of positions, its part into parts[image][tile]; or
// (parts null) one per image over all its tiles, the metrics themselves out.
// range_parts: the data range is the largest of them instead of `range`.
// Sums run in a fixed order, so the result does not depend on timing.
__global__ void __launch_bounds__(256)
k_image_metrics(const float* __restrict__ x, const float* __restrict__ ref, int h, int w,
                float range, const float* __restrict__ range_parts, int nrange, int ntx, int nty,
                MetricsPart* __restrict__ parts, float* __restrict__ ssim,
                float* __restrict__ mse, float* __restrict__ rmax)
{
    __shared__ MetricsShared S;
    if (threadIdx.x < SSIM_WIN) {
        double sum = 0.0, mine = 0.0;
        for (int t = 0; t < SSIM_WIN; ++t) {
            const double d = t - SSIM_WIN / 2, e = exp(-d * d / (2.0 * 1.5 * 1.5));
            sum += e;
            if (t == (int)threadIdx.x) mine = e;
        }
        S.win[threadIdx.x] = mine / sum;
    }
    float L = range;
    if (range_parts) {
        L = -INFINITY;
        for (int k = 0; k < nrange; ++k) L = max_or_nan(L, range_parts[k]);
    }
    const double c1 = (0.01 * L) * (0.01 * L), c2 = (0.03 * L) * (0.03 * L);
    const int64_t img = blockIdx.x;
    const float* X = x + img * (int64_t)h * w;
    const float* Y = ref + img * (int64_t)h * w;
    if (parts) {
        const int tile = blockIdx.y;
        const MetricsPart p = metrics_tile(S, X, Y, h, w, tile % ntx, tile / ntx, c1, c2);
        if (threadIdx.x == 0) parts[img * gridDim.y + tile] = p;
        return;
    }
    MetricsPart all{0.0, 0.0, -INFINITY, 0.0f};
    for (int tile = 0; tile < ntx * nty; ++tile) {
        const MetricsPart p = metrics_tile(S, X, Y, h, w, tile % ntx, tile / ntx, c1, c2);
        all.ssim += p.ssim;
        all.err += p.err;
        all.max = fmaxf(all.max, p.max);
    }
    if (threadIdx.x == 0) {
        ssim[img] = (float)(all.ssim / ((double)(h - SSIM_WIN + 1) * (w - SSIM_WIN + 1)));
        mse[img] = (float)(all.err / ((double)h * w));
        rmax[img] = all.max;
    }
}

// The images' metrics from their tiles' parts, a wave per image.
__global__ void __launch_bounds__(WAVE)
k_metrics_sum(const MetricsPart* __restrict__ parts, int tiles, int h, int w,
              const float* __restrict__ range_parts, int nrange, float* __restrict__ ssim,
              float* __restrict__ mse, float* __restrict__ rmax, float* __restrict__ range_out)
{
    const int64_t img = blockIdx.x;
    double a = 0.0, b = 0.0;
    float m = -INFINITY;
    for (int t = threadIdx.x; t < tiles; t += WAVE) {
        const MetricsPart p = parts[img * tiles + t];
        a += p.ssim;
        b += p.err;
        m = fmaxf(m, p.max);
    }
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        a += __shfl_xor(a, d, WAVE);
        b += __shfl_xor(b, d, WAVE);
        m = fmaxf(m, __shfl_xor(m, d, WAVE));
    }
    if (threadIdx.x == 0) {
        ssim[img] = (float)(a / ((double)(h - SSIM_WIN + 1) * (w - SSIM_WIN + 1)));
        mse[img] = (float)(b / ((double)h * w));
        rmax[img] = m;
        if (img == 0 && range_out) {
            float L = -INFINITY;
            for (int k = 0; k < nrange; ++k) L = max_or_nan(L, range_parts[k]);
            *range_out = L;
        }
    }
}

int einval(const char* msg) { return report_error(SDGR_EINVAL, msg); }

#define TRAIN_HIP(expr)                                                              \
    do {                                                                             \
        hipError_t e_ = (expr);                                                      \
        if (e_ != hipSuccess)                                                        \
            return report_error(SDGR_EHIP, (std::string(#expr) + ": " +             \
                                            hipGetErrorString(e_)).c_str());         \
    } while (0)

constexpr size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

bool set_arrays_ok(const sdgr_gaussian_set& s)
{
    if (!s.means || !s.scales || !s.quats || !s.ext) return false;
    if (!s.m_means || !s.v_means || !s.m_scales || !s.v_scales || !s.m_quats || !s.v_quats ||
        !s.m_ext || !s.v_ext)
        return false;
    if (s.amp && (!s.m_amp || !s.v_amp)) return false;
    if (s.sh && (!s.m_sh || !s.v_sh)) return false;
    return true;
}

}  // namespace
}  // namespace sdgr

using namespace sdgr;

extern "C" {

int sdgr_adam_step(const sdgr_param_group* groups, int32_t ngroups, int64_t t,
                   const sdgr_adam_config* cfg, void* stream)
{
    clear_error();
    if (!cfg || cfg->reserved != 0) return einval("adam config null or reserved not 0");
    if (!(cfg->beta1 >= 0.f && cfg->beta1 < 1.f) || !(cfg->beta2 >= 0.f && cfg->beta2 < 1.f) ||
        !(cfg->eps > 0.f))
        return einval("adam betas outside [0, 1) or eps not positive");
    if (t < 1) return einval("adam step t must be >= 1");
    if (ngroups < 0 || ngroups > SDGR_ADAM_MAX_GROUPS || (ngroups > 0 && !groups))
        return einval("adam group count outside 0..SDGR_ADAM_MAX_GROUPS");
    AdamArgs a{};
    int64_t total = 0;
    for (int k = 0; k < ngroups; ++k) {
        const sdgr_param_group& G = groups[k];
        if (G.count < 0) return einval("adam group with negative count");
        if (G.count == 0) continue;
        if (!G.param || !G.grad || !G.m || !G.v) return einval("adam group with a null array");
        if (!std::isfinite(G.lr)) return einval("adam learning rate not finite");
        if (G.reserved != 0) return einval("adam group reserved field not 0");
        if (std::isnan(G.lo) || std::isnan(G.hi)) return einval("adam clamp bound is NaN");
        AdamGroupDev& D = a.grp[a.ngroups++];
        D.p = G.param; D.g = G.grad; D.m = G.m; D.v = G.v;
        D.start = total; D.count = G.count; D.lr = G.lr; D.log_space = G.log_space != 0;
        D.lo = G.lo; D.hi = G.hi; D.clamp = G.lo < G.hi;
        total += G.count;
    }
    if (total == 0) return SDGR_OK;
    a.b1 = cfg->beta1; a.b2 = cfg->beta2; a.eps = cfg->eps;
    a.bc1 = (float)(1.0 / (1.0 - pow((double)cfg->beta1, (double)t)));
    a.bc2 = (float)(1.0 / (1.0 - pow((double)cfg->beta2, (double)t)));
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(total, 256, 8192)), dim3(256), 0,
                       (hipStream_t)stream, a, total);
    TRAIN_HIP(hipGetLastError());
    return SDGR_OK;
}

int sdgr_densify_stats(const float* d_means, int64_t n, float* grad_acc, float* grad_cnt,
                       float* grad_dir, void* stream)
{
    clear_error();
    if (n < 0) return einval("negative count");
    if (n == 0) return SDGR_OK;
    if (!d_means || !grad_acc || !grad_cnt || !grad_dir) return einval("null array");
    hipLaunchKernelGGL(k_densify_stats, dim3(blocks_for(n, 256)), dim3(256), 0,
                       (hipStream_t)stream, d_means, n, grad_acc, grad_cnt, grad_dir);
    TRAIN_HIP(hipGetLastError());
    return SDGR_OK;
}

size_t sdgr_densify_workspace_bytes(int64_t n)
{
    if (n < 0) return 0;
    const size_t nb = (size_t)((n + 255) / 256) + 1;
    return align256((size_t)n + 1) + 2 * align256(4 * nb);
}

int sdgr_densify(const sdgr_gaussian_set* in, int64_t n, const float* grad_acc,
                 const float* grad_cnt, const float* grad_dir, const sdgr_densify_config* cfg,
                 sdgr_gaussian_set* out, int64_t capacity, int64_t* n_out, void* workspace,
                 size_t workspace_bytes, void* stream)
{
    clear_error();
    if (!in || !out || !cfg || !n_out) return einval("null argument");
    if (cfg->reserved != 0 || in->reserved != 0 || out->reserved != 0)
        return einval("reserved fields must be 0");
    if (n < 0 || n > (int64_t)1 << 30) return einval("count outside [0, 2^30]");
    if (capacity < 2 * n) return einval("output capacity below twice the input count");
    if (!(cfg->split_factor > 1.0f) || !std::isfinite(cfg->split_factor))
        return einval("split_factor must be > 1");
    if (in->sh_coeffs < 0 || in->sh_coeffs > 16 || out->sh_coeffs != in->sh_coeffs)
        return einval("sh_coeffs outside 0..16 or different between in and out");
    if (!set_arrays_ok(*in) || !set_arrays_ok(*out))
        return einval("null parameter or moment array");
    if ((in->amp != nullptr) != (out->amp != nullptr) ||
        (in->sh != nullptr) != (out->sh != nullptr))
        return einval("in and out differ in which optional arrays they have");
    if (n > 0 && (!grad_acc || !grad_cnt || !grad_dir)) return einval("null statistics");
    if (workspace_bytes < sdgr_densify_workspace_bytes(n) || (n > 0 && !workspace))
        return report_error(SDGR_EWORKSPACE, "workspace smaller than sdgr_densify_workspace_bytes");
    if ((uintptr_t)workspace & 255) return einval("workspace not 256-byte aligned");
    hipStream_t s = (hipStream_t)stream;
    if (n == 0) {
        hipLaunchKernelGGL(k_densify_scan, dim3(1), dim3(1024), 0, s, (const uint32_t*)nullptr,
                           (int64_t)0, (uint32_t*)nullptr, n_out);
        TRAIN_HIP(hipGetLastError());
        return SDGR_OK;
    }
    const int64_t nb = (n + 255) / 256;
    char* w = (char*)workspace;
    uint8_t* act = (uint8_t*)w;
    uint32_t* bsum = (uint32_t*)(w + align256((size_t)n + 1));
    uint32_t* boff = (uint32_t*)(w + align256((size_t)n + 1) + align256(4 * (size_t)(nb + 1)));
    DensifyArgs a{*in, *out, *cfg, n};
    hipLaunchKernelGGL(k_densify_count, dim3((unsigned)nb), dim3(256), 0, s, a, grad_acc,
                       grad_cnt, act, bsum);
    hipLaunchKernelGGL(k_densify_scan, dim3(1), dim3(1024), 0, s, bsum, nb, boff, n_out);
    hipLaunchKernelGGL(k_densify_apply, dim3((unsigned)nb), dim3(256), 0, s, a, act, boff,
                       grad_dir);
    TRAIN_HIP(hipGetLastError());
    return SDGR_OK;
}

int sdgr_nearest_sq(const float* query, int64_t nq, const float* ref, int64_t nr, float* d2,
                    void* stream)
{
    clear_error();
    if (nq < 0 || nr < 0) return einval("negative point count");
    if (nq == 0) return SDGR_OK;
    if (!query || !d2 || (nr > 0 && !ref)) return einval("null array");
    if (nq > (int64_t)1 << 31) return einval("more than 2^31 query points");
    hipStream_t s = (hipStream_t)stream;
    const unsigned waves = blocks_for(nq, WAVE, 1u << 31);
    // few queries: parts of at least NN_PART references, up to NN_WAVES waves
    const int64_t most = std::min<int64_t>(NN_WAVES / waves, (nr + NN_PART - 1) / NN_PART);
    const int64_t parts = std::max<int64_t>(most, 1);
    if (parts > 1) {
        hipLaunchKernelGGL(k_fill_f32, dim3(blocks_for(nq, 256)), dim3(256), 0, s, d2, INFINITY,
                           nq);
        TRAIN_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(k_nearest_sq, dim3(waves, (unsigned)parts), dim3(WAVE), 0, s, query, nq,
                       ref, nr, (nr + parts - 1) / parts, d2);
    TRAIN_HIP(hipGetLastError());
    return SDGR_OK;
}

static int check_metrics(const float* x, const float* ref, int32_t nimg, int32_t h, int32_t w,
                         const float* ssim, const float* mse, const float* ref_max)
{
    if (nimg < 0) return einval("negative image count");
    if (h < SSIM_WIN || w < SSIM_WIN) return einval("images smaller than the 11 x 11 window");
    if (nimg > 0 && (!x || !ref || !ssim || !mse || !ref_max)) return einval("null array");
    return SDGR_OK;
}

static int metrics_tiles(int h, int w, int* ntx, int* nty)
{
    *ntx = (w - SSIM_WIN + SSIM_TX) / SSIM_TX;
    *nty = (h - SSIM_WIN + SSIM_TY) / SSIM_TY;
    return *ntx * *nty;
}

int sdgr_image_metrics(const float* x, const float* ref, int32_t nimg, int32_t h, int32_t w,
                       float data_range, float* ssim, float* mse, float* ref_max, void* stream)
{
    clear_error();
    if (const int rc = check_metrics(x, ref, nimg, h, w, ssim, mse, ref_max)) return rc;
    if (!(data_range > 0.0f) || !std::isfinite(data_range)) return einval("data_range must be > 0");
    if (nimg == 0) return SDGR_OK;
    int ntx, nty;
    metrics_tiles(h, w, &ntx, &nty);
    hipLaunchKernelGGL(k_image_metrics, dim3((unsigned)nimg), dim3(256), 0, (hipStream_t)stream,
                       x, ref, h, w, data_range, (const float*)nullptr, 0, ntx, nty,
                       (MetricsPart*)nullptr, ssim, mse, ref_max);
    TRAIN_HIP(hipGetLastError());
    return SDGR_OK;
}

size_t sdgr_image_metrics_workspace_bytes(int32_t nimg, int32_t h, int32_t w)
{
    if (nimg <= 0 || h < SSIM_WIN || w < SSIM_WIN) return 0;
    int ntx, nty;
    const int64_t tiles = (int64_t)metrics_tiles(h, w, &ntx, &nty);
    return align256(RANGE_PARTS * sizeof(float)) +
           align256((size_t)nimg * (size_t)tiles * sizeof(MetricsPart));
}

int sdgr_image_metrics_tiled(const float* x, const float* ref, int32_t nimg, int32_t h,
                             int32_t w, float data_range, float* ssim, float* mse,
                             float* ref_max, float* range, void* workspace,
                             size_t workspace_bytes, void* stream)
{
    clear_error();
    if (const int rc = check_metrics(x, ref, nimg, h, w, ssim, mse, ref_max)) return rc;
    if (!range && (!(data_range > 0.0f) || !std::isfinite(data_range)))
        return einval("data_range must be > 0");
    if (nimg == 0) return SDGR_OK;
    if (!workspace || workspace_bytes < sdgr_image_metrics_workspace_bytes(nimg, h, w))
        return report_error(SDGR_EWORKSPACE, "workspace too small for the image metrics");
    if ((uintptr_t)workspace & 255) return einval("workspace not 256-byte aligned");
    int ntx, nty;
    const int tiles = metrics_tiles(h, w, &ntx, &nty);
    if (tiles > 65535)   // grid y: one workgroup per image covers any size
        return report_error(SDGR_EUNSUPPORTED, "images too large for the tiled metrics");
    hipStream_t s = (hipStream_t)stream;
    float* rp = (float*)workspace;
    MetricsPart* parts = (MetricsPart*)((char*)workspace + align256(RANGE_PARTS * sizeof(float)));
    const int64_t px = (int64_t)nimg * h * w;
    const int nrange = range ? (int)blocks_for(px, 4096, RANGE_PARTS) : 0;
    if (range)
        hipLaunchKernelGGL(k_max_parts, dim3((unsigned)nrange), dim3(256), 0, s, ref, px, rp);
    hipLaunchKernelGGL(k_image_metrics, dim3((unsigned)nimg, (unsigned)tiles), dim3(256), 0, s, x,
                       ref, h, w, data_range, range ? rp : (const float*)nullptr, nrange, ntx,
                       nty, parts, ssim, mse, ref_max);
    hipLaunchKernelGGL(k_metrics_sum, dim3((unsigned)nimg), dim3(WAVE), 0, s, parts, tiles, h, w,
                       rp, nrange, ssim, mse, ref_max, range);
    TRAIN_HIP(hipGetLastError());
    return SDGR_OK;
}

}  // extern "C"
