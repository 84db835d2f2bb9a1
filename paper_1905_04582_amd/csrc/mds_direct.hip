// mds_direct.hip -- the small-problem form of the FP64 evaluation: one launch
// that computes whole gradient rows, with the leapfrog update of those rows.
//
// A problem of about a thousand locations is bound by the latency of its
// launches, not by its arithmetic: the tiled sweep leaves partial sums that a
// second kernel collects (N = 1000: 7 + 4 us per evaluation, of which each
// launch and its chain of first loads take 3).  Here a work-group owns
// kDirectRows rows and evaluates them against every column, so each pair is
// evaluated twice (from either row), the sums of a row close inside the
// work-group, and the kick and drift of the row follow in the same launch.
// The drifted positions go to another buffer than the ones the launch reads
// (other work-groups still need them).  Pairs evaluated twice cost what the
// tiled sweep's small tiles cost in prologues and row reductions.  One gradient
// of a captured sequence, D = 2, against the best tiling of the sweep: N = 60, 2.8
// and 7.5 us; N = 257, 3.3 and 8.1; N = 1000, 5.8 and 9.7; N = 1280, 10.4 and 10.0.
// (Four rows: with two or eight, or 16 waves, N = 1000 takes longer; the segments
// below the diagonal and the number of work-groups pull in opposite directions.)
//
// Lane l of a wave holds row i0 + l % 4 and column c0 + l / 4 of a block of 16
// columns; y comes from the strict lower triangle on either side of the
// diagonal, as segments of four rows' or sixteen columns' length.  Waves take
// blocks w, w + W, ... in two interleaved chains.  The sums L, dL/dsigma need
// run over the ordered pairs too and are halved (each pair adds the same two
// values).  Every order is fixed: the result is reproducible.
#include <hip/hip_ext.h>

#include "mds_internal.h"
#include "mds_math.h"
#include "mds_wave.h"

namespace mds {
namespace {

constexpr int kDirectCols = kWave / kDirectRows;  // columns of one block
constexpr int kDirectWaves = 8;
constexpr int kGroups = kWave / 16;  // rows of 16 lanes: partial sums per wave and row
constexpr double kSkipT = 9.0;  // the FP64 sweep's skip point
constexpr int kDppRowRor4 = 0x124, kDppRowRor8 = 0x128;  // rotate within 16 lanes

template <int D, bool SCAL>
__global__ void __launch_bounds__(kWave * kDirectWaves) direct_kernel(DirectArgs a)
{
    __shared__ double part[kDirectWaves * kGroups][kDirectRows * D];
    __shared__ double scal[3][kDirectWaves];
    const int lane = threadIdx.x & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int n = a.n;
    const int ii = lane % kDirectRows, jj = lane / kDirectRows;
    const int i0 = blockIdx.x * kDirectRows, i = i0 + ii;
    const int ic = min(i, n - 1);
    const double* __restrict__ X = a.x;
    const int ldx = a.ldx, ldy = a.ldy;

    // the next two blocks' columns: y of the pair (from the lower triangle) and
    // x of the column; a lane past the matrix repeats the last column
    const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<double*>(a.y), (short)0, 0x7fffffff, 0x00020000);
    struct Column {
        double y, x[D];
    };
    auto load = [&](int c0) {
        Column c;
        const int j = min(c0 + jj, n - 1);
        const uint32_t off = (uint32_t)(max(ic, j) * ldy + min(ic, j)) * 8u;
        c.y = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(yres, off, 0, 0));
#pragma unroll
        for (int d = 0; d < D; ++d) c.x[d] = X[j * ldx + d];
        return c;
    };

    const double sig = *(const_f64_ptr)a.sigma;
    double xi[D], g[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        xi[d] = X[ic * ldx + d];
        g[d] = 0.0;
    }
    constexpr int kStride = kDirectWaves * kDirectCols;
    int ca = w * kDirectCols;
    Column na = load(ca), nb = load(ca + kStride);

    const double inv_s = 1.0 / sig, inv_s2 = inv_s * inv_s;
    const NearConst64 nc = near_const(sig, inv_s);
    const double thr2 = a.truncated ? (kSkipT * sig) * (kSkipT * sig) : -1.0;
    const tab64_ptr ctab = tab64();
    double sA = 0.0, sM = 0.0, sE = 0.0;
    int cnt = 0, near_steps = 0;

    for (; ca < n; ca += 2 * kStride) {
        const Column pa = na, pb = nb;
        if (ca + 2 * kStride < n) {
            na = load(ca + 2 * kStride);
            nb = load(ca + 3 * kStride);
        }
        const int ja = ca + jj, jb = ja + kStride;
        double da[D], db[D], s2a = 0.0, s2b = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            da[d] = xi[d] - pa.x[d];
            db[d] = xi[d] - pb.x[d];
            s2a = fma(da[d], da[d], s2a);
            s2b = fma(db[d], db[d], s2b);
        }
        const uint64_t ma = __builtin_amdgcn_ballot_w64(ja < n && ja != i && i < n && !isnan(pa.y));
        const uint64_t mb = __builtin_amdgcn_ballot_w64(jb < n && jb != i && i < n && !isnan(pb.y));
        const uint64_t ta = __builtin_amdgcn_ballot_w64(s2a < thr2) & ma;
        const uint64_t tb = __builtin_amdgcn_ballot_w64(s2b < thr2) & mb;
        const double rsa = rsqrt_f64(fmax(s2a, 2.2250738585072014e-308));
        const double rsb = rsqrt_f64(fmax(s2b, 2.2250738585072014e-308));
        double wa = __builtin_amdgcn_inverse_ballot_w64(ma) ? fma(s2a, rsa, -pa.y) : 0.0;
        double wb = __builtin_amdgcn_inverse_ballot_w64(mb) ? fma(s2b, rsb, -pb.y) : 0.0;
        if constexpr (SCAL) {
            sA = fma(wa, wa, sA);
            sA = fma(wb, wb, sA);
            // each pair once: the columns below the row
            cnt += __builtin_popcountll(ma & __builtin_amdgcn_ballot_w64(ja < i)) +
                   __builtin_popcountll(mb & __builtin_amdgcn_ballot_w64(jb < i));
        }
        if (ta | tb) {
            const double dla = s2a * rsa, dlb = s2b * rsb;
            double ua, ub, mla, mlb;
            near_terms2_f64(s2a, s2b, dla, dlb, __builtin_amdgcn_inverse_ballot_w64(ta),
                            __builtin_amdgcn_inverse_ballot_w64(tb), nc, ctab, ua, ub, mla, mlb);
            if constexpr (SCAL) {
                near_steps = 1;
                sE = extend_product(sE, ua, ub);
                sM = fma(dla, mla, sM);
                sM = fma(dlb, mlb, sM);
            }
            wa += mla;
            wb += mlb;
        }
        const double cfa = wa * rsa, cfb = wb * rsb;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            g[d] = fma(cfa, da[d], g[d]);
            g[d] = fma(cfb, db[d], g[d]);
        }
    }

    // lanes of one row within 16 by rotations, the rest through LDS
#pragma unroll
    for (int d = 0; d < D; ++d) {
        double v = g[d];
        v += dpp<kDppRowRor8>(v);
        v += dpp<kDppRowRor4>(v);
        if ((lane & 15) < kDirectRows) part[w * kGroups + lane / 16][ii * D + d] = v;
    }
    if constexpr (SCAL) {
        const double lnphi = near_steps ? -log1p_product(sE, ctab) : 0.0;
        const double r = wave_sum(fma(sA, 0.5 * inv_s2, lnphi));
        const double s = wave_sum(((sA + sM) * inv_s2) * inv_s);
        if (lane == 0) {
            scal[0][w] = 0.5 * r;
            scal[1][w] = 0.5 * s;
            scal[2][w] = (double)cnt;
        }
    }
    __syncthreads();
    if constexpr (SCAL) {
        if (threadIdx.x == kWave * kDirectWaves - 1) {
            double r = 0.0, s = 0.0, m = 0.0;
            for (int q = 0; q < kDirectWaves; ++q) {
                r += scal[0][q];
                s += scal[1][q];
                m += scal[2][q];
            }
            a.tscal[2 * blockIdx.x + 0] = r;
            a.tscal[2 * blockIdx.x + 1] = s;
            a.tcount[blockIdx.x] = (uint32_t)m;
        }
    }
    const int t = threadIdx.x;
    if (t >= kDirectRows * D) return;
    const int k = i0 + t / D, d = t % D;
    if (k >= n) return;
    double sum = 0.0;
#pragma unroll
    for (int q = 0; q < kDirectWaves * kGroups; ++q) sum += part[q][t];
    double gr = -(sum * inv_s2);
    if (a.scale) gr *= *a.scale;
    const double x = X[k * ldx + d];
    if (a.prior) gr -= (*a.prior) * x;
    a.grad[(int64_t)k * a.ldg + d] = gr;
    double xn = x;
    if (a.p) {
        const double eps = *a.step;
        double* pp = a.p + (int64_t)k * a.ldp + d;
        const double pn = *pp + a.kick_mult * eps * gr;
        *pp = pn;
        if (a.drift) xn += eps * (a.inv_mass ? a.inv_mass[k * D + d] : 1.0) * pn;
    }
    if (a.x_out) a.x_out[(int64_t)k * a.ldxo + d] = xn;
}

}  // namespace

hipError_t launch_direct(int d, bool scal, const DirectArgs& a, hipStream_t s, hipEvent_t start,
                         hipEvent_t stop)
{
    if (a.n == 0) return hipSuccess;
    const dim3 grid((unsigned)direct_blocks(a.n)), block(kWave * kDirectWaves);
#define MDS_DIRECT_LAUNCH(DD, S)                                                              \
    if (start || stop)                                                                        \
        hipExtLaunchKernelGGL((direct_kernel<DD, S>), grid, block, 0, s, start, stop, 0, a);  \
    else                                                                                      \
        hipLaunchKernelGGL((direct_kernel<DD, S>), grid, block, 0, s, a);
#define MDS_DIRECT_CASE(DD)                \
    case DD:                               \
        if (scal) {                        \
            MDS_DIRECT_LAUNCH(DD, true)    \
        } else {                           \
            MDS_DIRECT_LAUNCH(DD, false)   \
        }                                  \
        break;
    switch (d) {
        MDS_DIRECT_CASE(1)
        MDS_DIRECT_CASE(2)
        MDS_DIRECT_CASE(3)
        MDS_DIRECT_CASE(4)
        MDS_DIRECT_CASE(5)
        MDS_DIRECT_CASE(6)
        MDS_DIRECT_CASE(7)
        MDS_DIRECT_CASE(8)
        default:
            return hipErrorInvalidValue;
    }
#undef MDS_DIRECT_LAUNCH
#undef MDS_DIRECT_CASE
    return hipGetLastError();
}

}  // namespace mds
