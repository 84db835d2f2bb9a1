// mds_lpd.hip -- log pointwise predictive density of held-out pairs (the
// model-selection part of Section 2): for each held-out pair, the log of the
// average over posterior draws of its truncated-normal density, summed over
// the pairs.
//
// The held-out pairs are first compacted into a list (row i, column j < i,
// y) in row-major order -- a count pass, an exclusive scan over the rows and
// a fill pass -- so that each draw costs O(pairs), not O(N^2).  Each draw
// then updates, per pair, a running log-sum-exp (largest term, sum of
// exp(l - largest)), and a last pass adds ln(average) over the pairs in a
// fixed order.
#include "mds_internal.h"
#include "mds_math.h"

namespace mds {
namespace {

constexpr int kRowThreads = 256;
constexpr int kScanThreads = 1024;
constexpr int kPartThreads = 256;

// The compaction passes walk a row in rounds of four columns per thread: one
// word of held-out bytes and one of mask bytes, loaded together, then y of the
// columns they keep.  (One byte per lane and load made them bound by vector
// memory instructions.)  They read the lower triangles of both masks and most
// lines of y's.  N = 5392, FP64, 10% held out, a mask: count 58 -> 46 us (it
// runs beside the write-back of the prepared Y), fill 61 -> 30 us.
// bytes j .. j+3 of a row as a word, byte 0 lowest; columns at or past `end`
// read as 0.  `wide`: the row starts at a multiple of four bytes (and then a
// word inside its n columns is one load).
__device__ __forceinline__ uint32_t row_word(const uint8_t* row, int j, int end, int n, bool wide)
{
    if (wide && j + 3 < n) {
        const uint32_t v = *reinterpret_cast<const uint32_t*>(row + j);
        const int left = end - j;
        return left >= 4 ? v : (left <= 0 ? 0u : v & (0xffffffffu >> (32 - 8 * left)));
    }
    uint32_t v = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b)
        if (j + b < end) v |= (uint32_t)row[j + b] << (8 * b);
    return v;
}

struct HeldoutRows {
    const uint8_t* missing;  // NULL: no mask
    int64_t ld_m;
    const uint8_t* heldout;
    int64_t ld_h;
    int n;
    bool wide_m, wide_h;  // every row starts at a multiple of four bytes
};

// keep[b]: whether pair (i, j0 + b) is held out, j0 + b below i; yv[b]: its y
template <typename S>
__device__ __forceinline__ void heldout_pairs(const S* __restrict__ yrow, const HeldoutRows& r,
                                              int i, int j0, bool (&keep)[4], S (&yv)[4])
{
    const uint32_t h = row_word(r.heldout + i * r.ld_h, j0, i, r.n, r.wide_h);
    const uint32_t m =
        r.missing ? row_word(r.missing + i * r.ld_m, j0, i, r.n, r.wide_m) : 0u;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        keep[b] = ((h >> (8 * b)) & 0xffu) != 0 && ((m >> (8 * b)) & 0xffu) == 0;
        yv[b] = keep[b] ? yrow[j0 + b] : (S)0;
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) keep[b] = keep[b] && !isnan(yv[b]);
}

// held-out pairs of row i (j < i)
template <typename S>
__global__ void __launch_bounds__(kRowThreads)
    heldout_count_kernel(const S* __restrict__ y, int64_t ld_y, HeldoutRows r,
                         int64_t* __restrict__ row_count)
{
    const int i = blockIdx.x;
    int c = 0;
    for (int j0 = 4 * threadIdx.x; j0 < i; j0 += 4 * kRowThreads) {
        bool keep[4];
        S yv[4];
        heldout_pairs(y + i * ld_y, r, i, j0, keep, yv);
#pragma unroll
        for (int b = 0; b < 4; ++b) c += keep[b] ? 1 : 0;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) c += __shfl_xor(c, m, kWave);
    __shared__ int wsum[kRowThreads / kWave];
    if ((threadIdx.x & (kWave - 1)) == 0) wsum[threadIdx.x / kWave] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int q = 0; q < kRowThreads / kWave; ++q) t += wsum[q];
        row_count[i] = t;
    }
}

// in place: row_count -> exclusive row offsets; row n holds the total.  Each
// thread sums its chunk of rows, the chunk sums are scanned by lane shifts
// within waves and then over the waves
__global__ void __launch_bounds__(kScanThreads)
    row_scan_kernel(int64_t n, int64_t* __restrict__ rows, int64_t* __restrict__ total)
{
    __shared__ int64_t wsum[kScanThreads / kWave];
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    const int64_t chunk = (n + kScanThreads - 1) / kScanThreads;
    const int64_t r0 = min(n, (int64_t)t * chunk), r1 = min(n, r0 + chunk);
    int64_t s = 0;
#pragma unroll 8
    for (int64_t r = r0; r < r1; ++r) s += rows[r];
    int64_t inc = s;
    for (int o = 1; o < kWave; o <<= 1) {
        const int64_t v = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += v;
    }
    if (lane == kWave - 1) wsum[w] = inc;
    __syncthreads();
    int64_t run = inc - s, all = 0;
    for (int q = 0; q < kScanThreads / kWave; ++q) {
        run += q < w ? wsum[q] : 0;
        all += wsum[q];
    }
    if (t == 0) {
        rows[n] = all;
        *total = all;
    }
    for (int64_t r = r0; r < r1; ++r) {
        const int64_t v = rows[r];
        rows[r] = run;
        run += v;
    }
}

// writes the held-out pairs of row i at its offset, in column order: the
// columns of a round are ordered by (wave, lane, byte)
template <typename S>
__global__ void __launch_bounds__(kRowThreads)
    heldout_fill_kernel(const S* __restrict__ y, int64_t ld_y, HeldoutRows r,
                        const int64_t* __restrict__ row_off, int64_t capacity,
                        int32_t* __restrict__ pi, int32_t* __restrict__ pj, double* __restrict__ py)
{
    constexpr int W = kRowThreads / kWave;
    const int i = blockIdx.x, t = threadIdx.x;
    const int lane = t & (kWave - 1), w = t / kWave;
    const uint64_t below = (1ull << lane) - 1ull;
    __shared__ int wcount[W];
    int64_t base = row_off[i];
    for (int r0 = 0; r0 < i; r0 += 4 * kRowThreads) {
        const int j0 = r0 + 4 * t;
        bool keep[4];
        S yv[4];
        heldout_pairs(y + i * ld_y, r, i, j0, keep, yv);
        int all = 0, before = 0;  // kept pairs of the wave, and of its lanes below this one
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const uint64_t mask = __builtin_amdgcn_ballot_w64(keep[b]);
            all += __builtin_popcountll(mask);
            before += __builtin_popcountll(mask & below);
        }
        if (lane == 0) wcount[w] = all;
        __syncthreads();
        int mine = 0, run = 0;
#pragma unroll
        for (int q = 0; q < W; ++q) {
            mine = q == w ? run : mine;
            run += wcount[q];
        }
        int64_t k = base + mine + before;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            if (keep[b] && k < capacity) {
                pi[k] = i;
                pj[k] = j0 + b;
                py[k] = (double)yv[b];
            }
            k += keep[b] ? 1 : 0;
        }
        base += run;
        __syncthreads();
    }
}

// per pair: l = ln p(y | delta, sigma) of the truncated normal for each of
// n_draws draws (draw s: x at xs + s * xstride, sigma = sigmas[s]), folded
// in draw order into the running log-sum-exp (acc[2k] = largest term,
// acc[2k+1] = sum of exp(l - largest)); `first` starts the sums with the
// first draw.  The state stays in registers across the draws, so a call with
// S draws reads and writes it once instead of S times.  Each thread takes
// kLpdPairs pairs (one block covers 128 consecutive pairs, lane-strided so every load is
// coalesced); ln sigma and 1/sigma of a chunk of
// draws are formed once per block, in LDS.  A pair with delta/sigma >= 9 takes
// ln Phi = 0 (|ln Phi(t)| < 2.3e-19 there, far below the rounding of l), and a
// wavefront skips the terms when every pair does.  The arithmetic of a draw
// does not depend on how the draws are grouped into calls: S calls of one draw
// and one call of S draws give the same bits.
//
// Several draws per pass are bound by vector instructions (135 per pair
// and draw with the short forms of mds_math.h; the library's exp, log and sqrt
// and the full-range ln Phi took 190), one draw per pass by the pair list and
// the state it streams.  1.45 M pairs, D = 2, ten draws and the finalize: 100 ->
// 86 us.
//
// Two pairs per thread (the special functions take two at a time) and blocks of
// one wave: the most work-groups, so that small lists fill the chip (2800
// locations, 0.39 M pairs, ten draws: 38.8 -> 32.0 us against blocks of 256
// threads with four pairs) and large ones end evenly (1.45 M pairs: 86.6 -> 85.3
// us; six dimensions, twelve draws, 2.9 M pairs: 215 -> 200 us).
// One draw per pass: blocks of four waves start sooner (0.39 M pairs, D = 2: 6.6 ->
// 6.1 us, D = 6: 7.3 -> 6.8; 1.45 M, D = 2: 13.9 -> 13.5), except for lists that
// leave the chip empty (12 000 pairs: 4.6 us, 4.8 with four waves) and, from D = 5
// on, long ones, which one-wave blocks end sooner (1.45 M pairs, D = 6: 16.7 with
// four, 15.6).  From D = 5 on each thread forms the constants itself, without a
// barrier (D = 6, 0.39 M pairs: 6.84 -> 6.79).
constexpr int kLpdThreads = kWave;           // several draws
constexpr int kLpdOneThreads = 4 * kWave;    // one draw, at most
inline int lpd_threads(bool one, int d, int64_t m)
{
    const bool four = m >= (1 << 17) && (d <= 4 || m < (1 << 20));
    return one && four ? kLpdOneThreads : kLpdThreads;
}
constexpr int kLpdPairs = 2;
constexpr int kLpdDrawChunk = 64;  // draws whose constants a block holds at a time

struct DrawConst {
    double inv_sigma;
    double c0;  // -ln(sqrt(2 pi) sigma)
};

// sqrt(s2): s2 / sqrt(s2) and one correction by its own residual, which leaves
// the final rounding (z = (y - delta)/sigma magnifies an error of delta); the
// rare values out of its range (0, squares so small that the residual
// underflows, infinite, NaN) go through the library's
__device__ __forceinline__ double lpd_distance(double s2)
{
    constexpr uint32_t kLow = (1023u - 900u) << 20, kHigh = (1023u + 1000u) << 20;
    const double rs = rsqrt_f64(s2);
    double delta = s2 * rs;
    delta = fma(fma(-delta, delta, s2), 0.5 * rs, delta);
    // 2^-900 <= s2 < 2^1000, from the word that holds sign and exponent
    const bool ok = (uint32_t)__double2hiint(s2) - kLow < kHigh - kLow;
    if (__builtin_amdgcn_ballot_w64(!ok)) delta = ok ? delta : sqrt(s2);
    return delta;
}

template <int D, bool ONE>
__global__ void __launch_bounds__(ONE ? kLpdOneThreads : kLpdThreads)
    lpd_accumulate_kernel(int64_t m, const int32_t* __restrict__ pi, const int32_t* __restrict__ pj,
                          const double* __restrict__ py, const double* __restrict__ xs,
                          int64_t ldx, int64_t xstride, const double* __restrict__ sigmas,
                          int32_t n_draws, double* __restrict__ acc, int first)
{
    constexpr double kLnSqrt2Pi = 0.91893853320467274178;
    constexpr int P = kLpdPairs;
    static_assert(P % 2 == 0 && kLpdThreads >= kLpdDrawChunk, "pairs and threads");
    const int T = ONE ? (int)blockDim.x : kLpdThreads;
    constexpr bool OWN = ONE && D > 4;
    __shared__ DrawConst dc[ONE ? 1 : kLpdDrawChunk];
    const int64_t base = (int64_t)blockIdx.x * (T * P) + threadIdx.x;
    int64_t ii[P], jj[P];
    double yv[P], mx[P], sm[P];
#pragma unroll
    for (int u = 0; u < P; ++u) {
        const int64_t k = base + (int64_t)u * T;
        // a lane past the end works on the last pair and stores nothing
        const int64_t kk = k < m ? k : m - 1;
        ii[u] = pi[kk] * ldx;
        jj[u] = pj[kk] * ldx;
        yv[u] = py[kk];
        mx[u] = first ? 0.0 : acc[2 * kk];
        sm[u] = first ? 0.0 : acc[2 * kk + 1];
    }
    // ONE: a single draw, with the loops known to run once (same arithmetic)
    const int32_t draws = ONE ? 1 : n_draws;
    const tab64_ptr tb = tab64();
    for (int s0 = 0; s0 < draws; s0 += kLpdDrawChunk) {
        const int chunk = ONE ? 1 : min(draws - s0, kLpdDrawChunk);
        auto constants = [&](int k) {
            const double sigma = sigmas[s0 + k];
            return DrawConst{1.0 / sigma, -kLnSqrt2Pi - log(sigma)};
        };
        if constexpr (!OWN) {
            __syncthreads();
            if ((int)threadIdx.x < chunk) dc[threadIdx.x] = constants(threadIdx.x);
            __syncthreads();
        }
        for (int sc = 0; sc < chunk; ++sc) {
            const DrawConst c = OWN ? constants(0) : dc[sc];
            const double* x = xs + (int64_t)(s0 + sc) * xstride;
            const bool start = first && s0 + sc == 0;
            double s2[P];
#pragma unroll
            for (int u = 0; u < P; ++u) {
                s2[u] = 0.0;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    const double diff = x[ii[u] + d] - x[jj[u] + d];
                    s2[u] = fma(diff, diff, s2[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < P; u += 2) {
                const double da = lpd_distance(s2[u]), db = lpd_distance(s2[u + 1]);
                const double ta = da * c.inv_sigma, tb2 = db * c.inv_sigma;
                const bool na = ta < 9.0, nb = tb2 < 9.0;
                double l[2] = {0.0, 0.0};
                if (__builtin_amdgcn_ballot_w64(na) | __builtin_amdgcn_ballot_w64(nb))
                    neg_ln_phi2_f64(ta, tb2, na, nb, tb, l[0], l[1]);
                const double za = (yv[u] - da) * c.inv_sigma;
                const double zb = (yv[u + 1] - db) * c.inv_sigma;
                l[0] += fma(-0.5 * za, za, c.c0);
                l[1] += fma(-0.5 * zb, zb, c.c0);
                if (start) {
                    mx[u] = l[0];
                    mx[u + 1] = l[1];
                    sm[u] = sm[u + 1] = 1.0;
                    continue;
                }
                // running log-sum-exp: one exp of -|l - largest| serves both
                // cases; arguments out of the short form's range (and NaN) go
                // through the library's
                const double dl[2] = {l[0] - mx[u], l[1] - mx[u + 1]};
                double e[2];
                exp2_neg_f64(-fabs(dl[0]), -fabs(dl[1]), tb, e[0], e[1]);
                if (__builtin_amdgcn_ballot_w64(!(fabs(dl[0]) < 700.0)) |
                    __builtin_amdgcn_ballot_w64(!(fabs(dl[1]) < 700.0))) {
                    e[0] = fabs(dl[0]) < 700.0 ? e[0] : exp(-fabs(dl[0]));
                    e[1] = fabs(dl[1]) < 700.0 ? e[1] : exp(-fabs(dl[1]));
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const bool up = dl[h] > 0.0;
                    sm[u + h] = fma(up ? sm[u + h] : 1.0, e[h], up ? 1.0 : sm[u + h]);
                    mx[u + h] = up ? l[h] : mx[u + h];
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < P; ++u) {
        const int64_t k = base + (int64_t)u * T;
        if (k < m) {
            acc[2 * k] = mx[u];
            acc[2 * k + 1] = sm[u];
        }
    }
}

// lpd = sum_k [acc_max + ln(acc_sum) - ln S], in two passes of fixed
// order: block b sums its contiguous share of the pairs (compensated
// per-thread sums, then a tree) into part[b]; one block adds the parts
__global__ void __launch_bounds__(kPartThreads)
    lpd_partial_kernel(int64_t m, const double* __restrict__ acc, double log_draws,
                       double* __restrict__ part)
{
    __shared__ double ps[kPartThreads];
    const int t = threadIdx.x;
    const int64_t chunk = (m + gridDim.x - 1) / gridDim.x;
    const int64_t k0 = (int64_t)blockIdx.x * chunk, k1 = min(m, k0 + chunk);
    double s = 0.0, c = 0.0;
    for (int64_t k = k0 + t; k < k1; k += kPartThreads) {
        const double v = acc[2 * k] + log(acc[2 * k + 1]) - log_draws;
        const double u = s + v;
        c += (fabs(s) >= fabs(v)) ? (s - u) + v : (v - u) + s;
        s = u;
    }
    ps[t] = s + c;
    __syncthreads();
    for (int h = kPartThreads / 2; h > 0; h >>= 1) {
        if (t < h) ps[t] += ps[t + h];
        __syncthreads();
    }
    if (t == 0) part[blockIdx.x] = ps[0];
}

__global__ void __launch_bounds__(kLpdMaxParts)
    lpd_sum_parts_kernel(int parts, const double* __restrict__ part, double* __restrict__ out)
{
    __shared__ double ps[kLpdMaxParts];
    const int t = threadIdx.x;
    ps[t] = t < parts ? part[t] : 0.0;
    __syncthreads();
    for (int h = kLpdMaxParts / 2; h > 0; h >>= 1) {
        if (t < h) ps[t] += ps[t + h];
        __syncthreads();
    }
    if (t == 0) *out = ps[0];
}

}  // namespace

namespace {
HeldoutRows heldout_rows(const uint8_t* missing, int64_t ld_m, const uint8_t* heldout,
                         int64_t ld_h, int64_t n)
{
    auto wide = [](const uint8_t* p, int64_t ld) { return ((uintptr_t)p | (uintptr_t)ld) % 4 == 0; };
    return {missing, ld_m, heldout, ld_h, (int)n, wide(missing, ld_m), wide(heldout, ld_h)};
}
}  // namespace

hipError_t launch_heldout_count(const void* y, int dt, int64_t ld_y, const uint8_t* missing,
                                int64_t ld_m, const uint8_t* heldout, int64_t ld_h, int64_t n,
                                int64_t* rows, int64_t* total, hipStream_t s)
{
    if (n > 0) {
        const HeldoutRows r = heldout_rows(missing, ld_m, heldout, ld_h, n);
        if (dt == 0)
            hipLaunchKernelGGL((heldout_count_kernel<double>), dim3((unsigned)n), dim3(kRowThreads),
                               0, s, (const double*)y, ld_y, r, rows);
        else
            hipLaunchKernelGGL((heldout_count_kernel<float>), dim3((unsigned)n), dim3(kRowThreads),
                               0, s, (const float*)y, ld_y, r, rows);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(row_scan_kernel, dim3(1), dim3(kScanThreads), 0, s, n, rows, total);
    return hipGetLastError();
}

hipError_t launch_heldout_fill(const void* y, int dt, int64_t ld_y, const uint8_t* missing,
                               int64_t ld_m, const uint8_t* heldout, int64_t ld_h, int64_t n,
                               const int64_t* rows, int64_t capacity, int32_t* pi, int32_t* pj,
                               double* py, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    const HeldoutRows r = heldout_rows(missing, ld_m, heldout, ld_h, n);
    if (dt == 0)
        hipLaunchKernelGGL((heldout_fill_kernel<double>), dim3((unsigned)n), dim3(kRowThreads), 0,
                           s, (const double*)y, ld_y, r, rows, capacity, pi, pj, py);
    else
        hipLaunchKernelGGL((heldout_fill_kernel<float>), dim3((unsigned)n), dim3(kRowThreads), 0,
                           s, (const float*)y, ld_y, r, rows, capacity, pi, pj, py);
    return hipGetLastError();
}

hipError_t launch_lpd_accumulate(int64_t m, const int32_t* pi, const int32_t* pj,
                                 const double* py, int d, const double* xs, int64_t ldx,
                                 int64_t xstride, const double* sigmas, int32_t n_draws,
                                 double* acc, int first, hipStream_t s)
{
    if (m == 0 || n_draws == 0) return hipSuccess;
    const int threads = lpd_threads(n_draws == 1, d, m);
    const int64_t per_block = threads * kLpdPairs;
    const dim3 grid((unsigned)((m + per_block - 1) / per_block)), block(threads);
#define MDS_LPD_CASE(DD)                                                                     \
    case DD:                                                                                 \
        if (n_draws == 1)                                                                    \
            hipLaunchKernelGGL((lpd_accumulate_kernel<DD, true>), grid, block, 0, s, m, pi, pj,   \
                               py, xs, ldx, xstride, sigmas, n_draws, acc, first);           \
        else                                                                                 \
            hipLaunchKernelGGL((lpd_accumulate_kernel<DD, false>), grid, block, 0, s, m, pi, pj,  \
                               py, xs, ldx, xstride, sigmas, n_draws, acc, first);           \
        break;
    switch (d) {
        MDS_LPD_CASE(1)
        MDS_LPD_CASE(2)
        MDS_LPD_CASE(3)
        MDS_LPD_CASE(4)
        MDS_LPD_CASE(5)
        MDS_LPD_CASE(6)
        MDS_LPD_CASE(7)
        MDS_LPD_CASE(8)
        default:
            return hipErrorInvalidValue;
    }
#undef MDS_LPD_CASE
    return hipGetLastError();
}

static int lpd_parts(int64_t m)
{
    const int64_t p = (m + 8 * kPartThreads - 1) / (8 * kPartThreads);
    return (int)max((int64_t)1, min((int64_t)kLpdMaxParts, p));
}

hipError_t launch_lpd_finalize(int64_t m, const double* acc, int64_t n_draws, double* part,
                               double* out, hipStream_t s)
{
    const int parts = lpd_parts(m);
    hipLaunchKernelGGL(lpd_partial_kernel, dim3(parts), dim3(kPartThreads), 0, s, m, acc,
                       log((double)n_draws), part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(lpd_sum_parts_kernel, dim3(1), dim3(kLpdMaxParts), 0, s, parts, part, out);
    return hipGetLastError();
}

}  // namespace mds
