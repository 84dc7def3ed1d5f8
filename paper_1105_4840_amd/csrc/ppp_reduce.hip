// Reductions, estimators and work distributions of libppp (all fp64, fixed
// merge order, so results do not depend on scheduling).
//
//   replica records --(per window, jackknife block)--> block records
//   block records   --(per window)--> window totals
//   window totals   --> Eq. 12 (JE, factorised over the independent windows),
//                       Eq. 14 and Eq. 13 with the actual increments
//                       lambda_{i+1} - lambda_i, combined estimate and its
//                       uncertainty (Sec. IV B, IV D), reverse JE, gamma_i^2,
//                       jackknife standard errors, Kish effective size,
//                       overlap of adjacent histograms, the Sec. IV B criterion
//   histograms      --> App. C work distributions Omega_j, dF^JE from them and
//                       the variance formula of Sec. IV A.
#include <hip/hip_runtime.h>

#include "ppp.h"
#include "ppp_device.hpp"
#include "ppp_launch.hpp"

namespace ppp {

__device__ __forceinline__ double *dptr(char *ws, int64_t off) { return reinterpret_cast<double *>(ws + off); }

// ---------------------------------------------------------------------------
__global__ void k_init(const DevProblem *__restrict__ probs, char *__restrict__ ws, int *tickets, int n_tickets) {
    const DevProblem &P = probs[blockIdx.y];
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    unsigned long long *hist = reinterpret_cast<unsigned long long *>(ws + P.off_hist);
    const int64_t nh = (int64_t)P.n_sim_windows * P.xi_nbins;
    for (int64_t i = tid; i < nh; i += stride) hist[i] = 0ull;
    if (P.w_half_bins > 0) {
        double *om = dptr(ws, P.off_omega);
        const int64_t nb = 2 * (int64_t)P.w_half_bins + 1;
        const int64_t no = (int64_t)P.n_windows * nb;
        for (int64_t i = tid; i < kAppcChains * no; i += stride)     // every chain; Omega_1: W = 0
            om[i] = (i % no == P.w_half_bins) ? 1.0 : 0.0;
    }
    if (blockIdx.y == 0 && tid < n_tickets) tickets[tid] = 0;
}

hipError_t launch_init(const DevProblem *d_probs, int n_probs, char *ws, int max_windows, int max_k, int max_m,
                       int *d_tickets, int n_tickets, hipStream_t stream) {
    int64_t work = (int64_t)max_windows * max_k;
    const int64_t wo = kAppcChains * (int64_t)max_windows * (2 * (int64_t)max_m + 1);
    if (wo > work) work = wo;
    int nb = (int)((work + 255) / 256);
    if (nb < 1) nb = 1;
    if (nb > 2048) nb = 2048;
    hipLaunchKernelGGL(k_init, dim3(nb, n_probs), dim3(256), 0, stream, d_probs, ws, d_tickets, n_tickets);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// One wave per (window, block): lanes merge strided replicas in order, then a
// fixed butterfly-free tree (lane l takes lane l + off) down to lane 0.
__global__ __launch_bounds__(64) void k_reduce_blocks(const DevProblem *__restrict__ probs, char *__restrict__ ws) {
    const DevProblem &P = probs[blockIdx.y];
    const int B = P.n_blocks, R = P.n_replicas;
    const int wb = blockIdx.x;
    if (wb >= P.n_sim_windows * B) return;
    const int w = wb / B, b = wb % B;
    const int lo = (int)(((int64_t)b * R + B - 1) / B);
    const int hi = (int)(((int64_t)(b + 1) * R + B - 1) / B);
    const double *rec = dptr(ws, P.off_acc) + ((int64_t)w * R) * A_NFIELDS;
    double a[A_NFIELDS];
    acc_empty(a);
    const int l = threadIdx.x;
    for (int r = lo + l; r < hi; r += 64) acc_merge(a, rec + (int64_t)r * A_NFIELDS);
    for (int off = 32; off >= 1; off >>= 1) {
        double o[A_NFIELDS];
        for (int f = 0; f < A_NFIELDS; ++f) o[f] = pull_f(l + off < 64 ? l + off : l, a[f]);
        if (l < off) acc_merge(a, o);
    }
    if (l == 0) {
        double *dst = dptr(ws, P.off_blk) + (int64_t)wb * A_NFIELDS;
        for (int f = 0; f < A_NFIELDS; ++f) dst[f] = a[f];
    }
}

hipError_t launch_reduce(const DevProblem *d_probs, int n_probs, char *ws, int max_windows, int max_blocks,
                         hipStream_t stream) {
    hipLaunchKernelGGL(k_reduce_blocks, dim3(max_windows * max_blocks, n_probs), dim3(64), 0, stream, d_probs, ws);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
struct WinStat {
    double n, mean, var, lse_f, lse_r;
};
__device__ __forceinline__ WinStat win_stat(const double *a, double lam) {
    WinStat s;
    s.n = a[A_N];
    const double m1 = a[A_S1] / a[A_N];
    s.mean = lam + m1;
    s.var = (a[A_S2] - a[A_N] * m1 * m1) / (a[A_N] - 1.0);
    s.lse_f = lse_value(a[A_MF], a[A_SF]);
    s.lse_r = lse_value(a[A_MR], a[A_SR]);
    return s;
}

// contributions of the step i -> i+1 to JE, fluct, gauss
__device__ __forceinline__ void step_terms(const DevProblem &P, const WinStat &st, double li, double lj, double &je,
                                           double &fl, double &ga) {
    const double dl = lj - li;
    je = -P.kT * (st.lse_f - log(st.n));
    fl = P.k * dl * (li - st.mean);
    const double gamma2 = P.k * st.var / P.kT;
    ga = fl + 0.5 * P.k * dl * dl * (1.0 - gamma2);
}

__device__ double block_sum(double v, double *sh) {
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = blockDim.x / 2; off >= 1; off >>= 1) {
        if (t < off) sh[t] += sh[t + off];
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

// Sum and extrema over a wavefront, in every lane.  The butterfly adds the lanes
// 32, 16, 8, 4, 2, 1 apart; from 8 on the values repeat with that period, so a
// rotation inside a row of 16 (a DPP move) brings the same partner as an
// exchange through LDS would, six times sooner.
template <int OFF> __device__ __forceinline__ double row_ror(double v) {
    I2 w = __builtin_bit_cast(I2, v);
    w.lo = __builtin_amdgcn_update_dpp(w.lo, w.lo, 0x120 + OFF, 0xf, 0xf, false);
    w.hi = __builtin_amdgcn_update_dpp(w.hi, w.hi, 0x120 + OFF, 0xf, 0xf, false);
    return __builtin_bit_cast(double, w);
}
template <typename Op> __device__ __forceinline__ double wave_all(double v, Op op) {
    v = op(v, __shfl_xor(v, 32));
    v = op(v, __shfl_xor(v, 16));
    v = op(v, row_ror<8>(v));
    v = op(v, row_ror<4>(v));
    v = op(v, row_ror<2>(v));
    return op(v, row_ror<1>(v));
}
__device__ __forceinline__ double wave_sum(double v) { return wave_all(v, [](double a, double b) { return a + b; }); }
__device__ __forceinline__ double wave_max(double v) { return wave_all(v, [](double a, double b) { return fmax(a, b); }); }

// Sums of a workgroup of up to four wavefronts, in every thread.
template <int NV>
__device__ __forceinline__ void block_sum_vec(double (&v)[NV], double *sh) {
    for (int q = 0; q < NV; ++q) v[q] = wave_sum(v[q]);
    const int wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
        for (int q = 0; q < NV; ++q) sh[q * 4 + wave] = v[q];
    __syncthreads();
    for (int q = 0; q < NV; ++q) {
        double t = 0;
        for (int u = 0; u < n_waves; ++u) t += sh[q * 4 + u];
        v[q] = t;
    }
}

// ---------------------------------------------------------------------------
// Window totals and leave-one-out records of one window, by one wavefront.
//
// Lane l holds blocks [l c, (l + 1) c), c = ceil(B / 64).  A log-sum-exp without
// block b is taken against the largest maximum among the others: the overall
// maximum M, or for the block that holds it the next one; its sum is the sum of
// the blocks before plus that of the blocks after, so nothing cancels in it.  Every
// block then costs c exponentials a direction (one up to 64 blocks; its lane's
// others are added again) instead of the B - 1 merges that each leave-one-out record
// took when it was built by itself.  Counts (exact) and moments are the total less the
// block: a moment is then off by rounding of the total, which matters only where one
// block outweighs the others, and there the standard error is as large as that total.
// 21 windows, 300 blocks: 0.8 ms for all estimators, 11.1 with merges; 4096: 3.0, 1890.
// ---------------------------------------------------------------------------
struct LseLoo {
    double m, s, s2;          // all blocks: maximum, scaled sum, scaled sum of squares (of 2a)
    double before, after;     // scaled sums of the blocks of the lanes before and after
    double m_next, s_next;    // all blocks but the holder of the maximum
    int holder;
};

__device__ __forceinline__ LseLoo lse_totals(const double *blk, int B, int b0, int b1, int fm) {
    LseLoo r;
    double mx = -INFINITY;
    for (int b = b0; b < b1; ++b) mx = fmax(mx, blk[(int64_t)b * A_NFIELDS + fm]);
    r.m = wave_max(mx);
    int h = B;
    for (int b = b1 - 1; b >= b0; --b)
        if (blk[(int64_t)b * A_NFIELDS + fm] == r.m) h = b;
    for (int off = 32; off >= 1; off >>= 1) h = min(h, __shfl_xor(h, off));
    r.holder = h;
    mx = -INFINITY;
    for (int b = b0; b < b1; ++b)
        if (b != h) mx = fmax(mx, blk[(int64_t)b * A_NFIELDS + fm]);
    r.m_next = wave_max(mx);
    double s = 0, s2 = 0, sn = 0;
    for (int b = b0; b < b1; ++b) {
        const double *a = blk + (int64_t)b * A_NFIELDS;
        if (a[fm + 1] == 0.0) continue;                  // no sample in it
        const double t = exp(a[fm] - r.m);
        s += a[fm + 1] * t;
        s2 += a[fm + 3] * (t * t);
        if (b != h) sn += a[fm + 1] * exp(a[fm] - r.m_next);
    }
    double up = s, dn = s;                               // inclusive sums over the lanes
    const int l = (int)threadIdx.x & 63;
    for (int off = 1; off < 64; off <<= 1) {
        const double u = __shfl_up(up, off), d = __shfl_down(dn, off);
        if (l >= off) up += u;
        if (l + off < 64) dn += d;
    }
    const double b_in = __shfl_up(up, 1), a_in = __shfl_down(dn, 1);
    r.before = l > 0 ? b_in : 0.0;
    r.after = l < 63 ? a_in : 0.0;
    r.s = wave_sum(s);
    r.s2 = wave_sum(s2);
    r.s_next = wave_sum(sn);
    return r;
}

// ln sum exp over every block but b, which is one of this lane's [b0, b1).
__device__ __forceinline__ double lse_without(const LseLoo &r, const double *blk, int b0, int b1, int fm, int b) {
    if (b == r.holder) return lse_value(r.m_next, r.s_next);
    double s = r.before;
    for (int c = b0; c < b1; ++c) {
        const double *a = blk + (int64_t)c * A_NFIELDS;
        if (c != b && a[fm + 1] != 0.0) s += a[fm + 1] * exp(a[fm] - r.m);
    }
    return lse_value(r.m, s + r.after);
}

// Statistics of one window (everything that needs only its own record and its
// neighbour's histogram), its terms of every profile and of every leave-one-out
// profile, and its least-squares Gaussian; k_profiles sums the terms over the
// windows.  One workgroup per window.
//
// The paper's sigma_i (Sec. IV A: gamma_i^2 = k sigma_i^2 / kT with sigma_i by
// least-squares fitting of the x_i distribution): the Gaussian A exp(-(x -
// mu)^2 / (2 sigma^2)) closest in least squares to the histogram density
// count_b / (n dxi) at the bin centres, by Levenberg-Marquardt from the sample
// moments.
//
// Bound: the fp64 exponentials of the fit, on one CU a window.  A step's
// exponentials serve its cost and, once it is accepted, the next step's
// Jacobian (16 bins a thread are kept in registers); a rejected step leaves the
// normal equations as they are; a trial equal to the one just rejected is not
// evaluated again (damping far below 1 does not move it); and bins that are
// empty and more than 13 sigma from the mean (a square below 1e-73 of the peak's)
// are left out.
constexpr int kFitKeep = 16;

__global__ __launch_bounds__(256) void k_windows(const DevProblem *__restrict__ probs, char *__restrict__ ws) {
    const DevProblem &P = probs[blockIdx.y];
    const int s = P.n_windows, S = P.n_sim_windows, B = P.n_blocks, K = P.xi_nbins;
    const int w = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
    if (w >= S) return;
    __shared__ double sh[10 * 4];
    __shared__ double s_tot[A_NFIELDS];
    __shared__ double s_n_next;
    __shared__ int s_range[2];
    const double *lam = dptr(ws, P.off_lambda);
    const double *blk = dptr(ws, P.off_blk) + (int64_t)w * B * A_NFIELDS;
    double *out = dptr(ws, P.off_out);
    double *jack = dptr(ws, P.off_jack);
    const unsigned long long *hist = reinterpret_cast<const unsigned long long *>(ws + P.off_hist) + (int64_t)w * K;
#define OUT(f, i) out[(int64_t)(f) * s + (i)]
    if (t == 0) { s_range[0] = K; s_range[1] = -1; }
    __syncthreads();

    if (wave == 0) {
        const int chunk = (B + 63) / 64;
        const int b0 = min(B, lane * chunk), b1 = min(B, b0 + chunk);
        double n = 0, s1 = 0, s2 = 0, lo = INFINITY, hi = -INFINITY, un = 0, ov = 0, bl = 0;
        for (int b = b0; b < b1; ++b) {
            const double *a = blk + (int64_t)b * A_NFIELDS;
            n += a[A_N]; s1 += a[A_S1]; s2 += a[A_S2];
            lo = fmin(lo, a[A_XMIN]); hi = fmax(hi, a[A_XMAX]);
            un += a[A_UNDER]; ov += a[A_OVER]; bl += a[A_BLOWN];
        }
        double a[A_NFIELDS];
        a[A_N] = wave_sum(n); a[A_S1] = wave_sum(s1); a[A_S2] = wave_sum(s2);
        a[A_XMIN] = -wave_max(-lo); a[A_XMAX] = wave_max(hi);
        a[A_UNDER] = wave_sum(un); a[A_OVER] = wave_sum(ov); a[A_BLOWN] = wave_sum(bl);
        const LseLoo F = lse_totals(blk, B, b0, b1, A_MF), R = lse_totals(blk, B, b0, b1, A_MR);
        a[A_MF] = F.m; a[A_SF] = F.s; a[A_MF2] = 2.0 * F.m; a[A_SF2] = F.s2;
        a[A_MR] = R.m; a[A_SR] = R.s; a[A_MR2] = 2.0 * R.m; a[A_SR2] = R.s2;
        if (lane == 0) {
            double *tot = dptr(ws, P.off_tot) + (int64_t)w * A_NFIELDS;
            for (int f = 0; f < A_NFIELDS; ++f) { tot[f] = a[f]; s_tot[f] = a[f]; }
        }
        if (lane == 0 && w < s) {
            const WinStat st = win_stat(a, lam[w]);
            OUT(O_XI_MEAN, w) = st.mean;
            OUT(O_XI_STD, w) = sqrt(st.var);
            OUT(O_GAMMA2, w) = P.k * st.var / P.kT;
            OUT(O_XI_MINS, w) = a[A_XMIN];
            OUT(O_XI_MAXS, w) = a[A_XMAX];
            OUT(O_LSE_FWD, w) = w + 1 < s ? st.lse_f : NAN;
            OUT(O_LSE_REV, w) = w > 0 ? st.lse_r : NAN;
            OUT(O_N_SAMPLES, w) = a[A_N];
            OUT(O_N_BLOWN, w) = a[A_BLOWN];
            OUT(O_UNDER, w) = a[A_UNDER];
            OUT(O_OVER, w) = a[A_OVER];
            // this window's term of the reverse profile at w and of the others at w + 1
            OUT(O_DF_REV, w) = w > 0 ? P.kT * (st.lse_r - log(st.n)) : 0.0;
            if (w + 1 < s) {
                const double dl = lam[w + 1] - lam[w];
                OUT(O_KISH, w) = exp(2.0 * st.lse_f - lse_value(a[A_MF2], a[A_SF2])) / st.n;
                OUT(O_DL_SIGMA, w) = fabs(dl) / sqrt(st.var);
                const double reach = dl > 0 ? a[A_XMAX] - st.mean : st.mean - a[A_XMIN];
                OUT(O_DL_REACH, w) = fabs(dl) / reach;
                OUT(O_CRIT, w) = fabs(dl) <= reach ? 1.0 : 0.0;
                double dje, dfl, dga;
                step_terms(P, st, lam[w], lam[w + 1], dje, dfl, dga);
                OUT(O_DF_JE, w + 1) = dje; OUT(O_DF_FLUCT, w + 1) = dfl; OUT(O_DF_GAUSS, w + 1) = dga;
                OUT(O_DF_FLUCT_LIT, w + 1) = lam[w] - st.mean;
                OUT(O_DF_GAUSS_LIT, w + 1) = 1.0 - P.k * st.var / P.kT;
            } else {
                OUT(O_KISH, w) = NAN; OUT(O_DL_SIGMA, w) = NAN; OUT(O_DL_REACH, w) = NAN; OUT(O_CRIT, w) = NAN;
                OUT(O_OVL, w) = NAN;
            }
        }
        // block b removed from every window: this window's terms without it
        if (B > 1)
            for (int b = b0; b < b1; ++b) {
                const double *c = blk + (int64_t)b * A_NFIELDS;
                const double ln = log(a[A_N] - c[A_N]);
                if (w + 1 < s) {
                    double q[A_NFIELDS];
                    q[A_N] = a[A_N] - c[A_N]; q[A_S1] = a[A_S1] - c[A_S1]; q[A_S2] = a[A_S2] - c[A_S2];
                    WinStat st;
                    const double m1 = q[A_S1] / q[A_N];
                    st.n = q[A_N];
                    st.mean = lam[w] + m1;
                    st.var = (q[A_S2] - q[A_N] * m1 * m1) / (q[A_N] - 1.0);
                    st.lse_f = lse_without(F, blk, b0, b1, A_MF, b);
                    double dje, dfl, dga;
                    step_terms(P, st, lam[w], lam[w + 1], dje, dfl, dga);
                    double *jb = jack + (int64_t)b * JK_FIELDS * s;
                    jb[0 * s + w + 1] = dje; jb[1 * s + w + 1] = dfl; jb[2 * s + w + 1] = dga;
                }
                if (P.free_ens) {
                    // Eq. 5 from the ends, Eq. 6 from the free ensemble
                    double *jt = dptr(ws, P.off_jack_turn) + (int64_t)b * JK_TURN;
                    if (w == 0) jt[0] = P.kT * (lse_without(R, blk, b0, b1, A_MR, b) - ln);
                    if (w == s - 1) jt[2] = P.kT * (lse_without(F, blk, b0, b1, A_MF, b) - ln);
                    if (w == s) {
                        jt[1] = -P.kT * (lse_without(F, blk, b0, b1, A_MF, b) - ln);
                        jt[3] = -P.kT * (lse_without(R, blk, b0, b1, A_MR, b) - ln);
                    }
                }
            }
    } else {
        // meanwhile the other wavefronts find the range of non-empty bins, and
        // wavefront 1 the sample count of the next window
        int lo = K, hi = -1;
        for (int b = t - 64; b < K; b += 192)
            if (hist[b]) { lo = min(lo, b); hi = b; }
        for (int off = 32; off >= 1; off >>= 1) {
            lo = min(lo, __shfl_xor(lo, off));
            hi = max(hi, __shfl_xor(hi, off));
        }
        if (lane == 0 && hi >= 0) { atomicMin(&s_range[0], lo); atomicMax(&s_range[1], hi); }
        if (wave == 1 && w + 1 < s) {
            double nn = 0;
            for (int b = lane; b < B; b += 64) nn += blk[(int64_t)(B + b) * A_NFIELDS + A_N];
            nn = wave_sum(nn);
            if (lane == 0) s_n_next = nn;
        }
    }
    __syncthreads();
    if (w >= s) return;
    const double n = s_tot[A_N];
    const int e_lo = s_range[0], e_hi = s_range[1];
    // overlap of adjacent histograms: sum_b min(rho_i(b), rho_{i+1}(b))
    if (w + 1 < s) {
        double part[1] = {0.0};
        // (a window without samples gives 0 / 0 in every bin, and fmin then takes the neighbour's)
        for (int b = (n > 0.0 ? e_lo : 0) + t; b <= (n > 0.0 ? e_hi : K - 1); b += 256)
            part[0] += fmin((double)hist[b] / n, (double)hist[K + b] / s_n_next);
        block_sum_vec<1>(part, sh);
        if (t == 0) OUT(O_OVL, w) = part[0];
    }

    const double m1 = s_tot[A_S1] / n;
    const double var = (s_tot[A_S2] - n * m1 * m1) / (n - 1.0);
    double nz[1] = {0.0};                             // non-empty bins
    for (int b = e_lo + t; b <= e_hi; b += 256) nz[0] += hist[b] ? 1.0 : 0.0;
    block_sum_vec<1>(nz, sh);
    if (!(n > 2.0) || !(var > 0.0) || nz[0] < 3.0) {   // three parameters need three points
        if (t == 0) { OUT(O_SIGMA_LSQ, w) = NAN; OUT(O_GAMMA2_LSQ, w) = NAN; }
        return;
    }
    const double norm = 1.0 / (n * P.xi_bin);
    const double x0 = P.xi_min, xb = P.xi_bin;
    // parameters, damping, squared residual and normal equations (J^T J, J^T r) of the accepted point
    double A = 1.0 / (sqrt(var) * 2.5066282746310002), mu = lam[w] + m1, sg = sqrt(var);
    double lm = 1e-3, c0 = 0.0;
    double v[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    double ke[kFitKeep];
    int first = 0, last = 0;                           // this point's bins, from a multiple of 256
    auto bins_of = [&](double pm, double ps) {
        const double a = floor((pm - 13.0 * ps - x0) / xb), z = ceil((pm + 13.0 * ps - x0) / xb);
        const int ia = a > (double)e_lo ? e_lo : (a < 0.0 ? 0 : (int)a);
        const int iz = z < (double)e_hi ? e_hi : (z > (double)(K - 1) ? K - 1 : (int)z);
        // (a NaN keeps every bin)
        first = a == a ? ia & ~255 : 0;
        last = z == z ? iz : K - 1;
    };
    // squared residual of (pA, pm, ps); the exponentials of the thread's first bins stay in ke
    auto cost = [&](double pA, double pm, double ps) {
        bins_of(pm, ps);
        double c[1] = {0.0};
        const double i2 = 1.0 / (2.0 * ps * ps);
        auto bin = [&](int b) {
            const double d = x0 + ((double)b + 0.5) * xb - pm;
            const double e = exp(-d * d * i2);
            const double r = (double)hist[b] * norm - pA * e;
            c[0] += r * r;
            return e;
        };
#pragma unroll
        for (int i = 0; i < kFitKeep; ++i) {
            const int b = first + t + 256 * i;
            if (b <= last) ke[i] = bin(b);
        }
        for (int b = first + t + 256 * kFitKeep; b <= last; b += 256) bin(b);
        block_sum_vec<1>(c, sh);
        return c[0];
    };
    auto normal_equations = [&]() {
        for (int q = 0; q < 9; ++q) v[q] = 0.0;
        const double i2 = 1.0 / (2.0 * sg * sg), is2 = 1.0 / (sg * sg);
        auto bin = [&](int b, double e, double d) {
            const double f = A * e;
            const double r = (double)hist[b] * norm - f;
            const double jA = e, jm = f * d * is2, js = f * d * d * is2 / sg;
            v[0] += jA * jA; v[1] += jA * jm; v[2] += jA * js;
            v[3] += jm * jm; v[4] += jm * js; v[5] += js * js;
            v[6] += jA * r; v[7] += jm * r; v[8] += js * r;
        };
#pragma unroll
        for (int i = 0; i < kFitKeep; ++i) {
            const int b = first + t + 256 * i;
            if (b <= last) bin(b, ke[i], x0 + ((double)b + 0.5) * xb - mu);
        }
        for (int b = first + t + 256 * kFitKeep; b <= last; b += 256) {
            const double d = x0 + ((double)b + 0.5) * xb - mu;
            bin(b, exp(-d * d * i2), d);
        }
        block_sum_vec<9>(v, sh);
    };
    c0 = cost(A, mu, sg);
    normal_equations();
    double tA = NAN, tm = NAN, ts = NAN;               // the trial rejected last
    for (int it = 0; it < 200; ++it) {
        // (J^T J + lm diag) delta = J^T r, by Cramer's rule on the 3x3 system (in every thread)
        const double a00 = v[0] * (1 + lm), a11 = v[3] * (1 + lm), a22 = v[5] * (1 + lm);
        const double a01 = v[1], a02 = v[2], a12 = v[4];
        const double det = a00 * (a11 * a22 - a12 * a12) - a01 * (a01 * a22 - a12 * a02) + a02 * (a01 * a12 - a11 * a02);
        const double g0 = v[6], g1 = v[7], g2 = v[8];
        const double d0 = (g0 * (a11 * a22 - a12 * a12) - a01 * (g1 * a22 - a12 * g2) + a02 * (g1 * a12 - a11 * g2)) / det;
        const double d1 = (a00 * (g1 * a22 - a12 * g2) - g0 * (a01 * a22 - a12 * a02) + a02 * (a01 * g2 - g1 * a02)) / det;
        const double d2 = (a00 * (a11 * g2 - g1 * a12) - a01 * (a01 * g2 - g1 * a02) + g0 * (a01 * a12 - a11 * a02)) / det;
        const double nA = A + d0, nm = mu + d1, ns = fabs(sg + d2);
        const bool done = fabs(d0) <= 1e-14 * fabs(A) && fabs(d1) <= 1e-14 * (fabs(mu) + sg) && fabs(d2) <= 1e-14 * sg;
        if (nA == tA && nm == tm && ns == ts) {
            lm *= 10.0;
        } else {
            const double c1 = cost(nA, nm, ns);
            if (c1 <= c0) {
                A = nA; mu = nm; sg = ns; c0 = c1; lm = fmax(lm * 0.1, 1e-15);
                tA = NAN;
                if (!done && lm <= 1e12) normal_equations();
            } else {
                lm *= 10.0;
                tA = nA; tm = nm; ts = ns;
            }
        }
        if (done || lm > 1e12) break;
    }
    if (t == 0) {
        OUT(O_SIGMA_LSQ, w) = sg;
        OUT(O_GAMMA2_LSQ, w) = P.k * sg * sg / P.kT;
    }
#undef OUT
}

// Running sums of a row of s terms in place, eight loads at a time.
__device__ __forceinline__ void prefix_row(double *row, int s) {
    double acc = 0.0;
    row[0] = 0.0;
    for (int j0 = 1; j0 < s; j0 += 8) {
        double v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = j0 + i < s ? row[j0 + i] : 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            acc += v[i];
            if (j0 + i < s) row[j0 + i] = acc;
        }
    }
}

// Jackknife standard error of value(b) over the B blocks.
template <typename Fn> __device__ __forceinline__ double jack_se(int B, Fn &&value) {
    if (B <= 1) return NAN;
    double m = 0;
#pragma unroll 8
    for (int b = 0; b < B; ++b) m += value(b);
    m /= B;
    double ss = 0;
#pragma unroll 8
    for (int b = 0; b < B; ++b) {
        const double d = value(b) - m;
        ss += d * d;
    }
    return sqrt((B - 1.0) / B * ss);
}

// Profiles: the windows' terms summed along lambda, their leave-one-out twins and
// standard errors, and the turn-on free energies.  One workgroup per problem.
__global__ __launch_bounds__(256) void k_profiles(const DevProblem *__restrict__ probs, char *__restrict__ ws) {
    const DevProblem &P = probs[blockIdx.x];
    const int s = P.n_windows, B = P.n_blocks, t = threadIdx.x;
    const double *lam = dptr(ws, P.off_lambda);
    const double *tot = dptr(ws, P.off_tot);
    double *out = dptr(ws, P.off_out);
    double *jack = dptr(ws, P.off_jack);
    double *turn = dptr(ws, P.off_turn);
    double *jt = dptr(ws, P.off_jack_turn);
    __shared__ double s_eq5_first;
#define OUT(f, i) out[(int64_t)(f) * s + (i)]
    // one thread per row of terms; the least-squares Gaussians' row of Eq. 13 is formed first
    for (int j = t; j < s; j += 256) {
        double g = 0.0;
        if (j > 0) {
            // Eq. 13 with gamma_i^2 from the fitted sigma_i, <x_i> the sample mean
            const double dl = lam[j] - lam[j - 1];
            const double mean = OUT(O_XI_MEAN, j - 1), g2 = OUT(O_GAMMA2_LSQ, j - 1);
            g = P.k * dl * (lam[j - 1] - mean) + 0.5 * P.k * dl * dl * (1.0 - g2);
        }
        OUT(O_DF_GAUSS_LSQ, j) = g;
    }
    __syncthreads();
    const int rows[7] = {O_DF_JE, O_DF_FLUCT, O_DF_GAUSS, O_DF_REV, O_DF_FLUCT_LIT, O_DF_GAUSS_LIT, O_DF_GAUSS_LSQ};
    for (int q = t; q < 7 + (B > 1 ? 3 * B : 0); q += 256) {
        if (q < 7) prefix_row(&OUT(rows[q], 0), s);
        else prefix_row(jack + ((int64_t)((q - 7) / 3) * JK_FIELDS + (q - 7) % 3) * s, s);
    }
    __syncthreads();
    // Turn-on free energies from the records of window 1 (a1), window s (as) and the
    // unrestrained ensemble (a0).
    // Eq. 5: DF = kT ln <exp(+beta k/2 (x - lambda)^2)> over the restrained window
    // Eq. 6: DF = -kT ln <exp(-beta k/2 (x_0 - lambda)^2)> over the free ensemble
    // Eq. 10 factorised over x_0, x_1 .. x_s: the turn-on at lambda_1 from x_0, the
    // steps, and the turn-off at lambda_s from x_s
    if (t == 0) {
        if (P.free_ens) {
            const double *a1 = tot, *as = tot + (int64_t)(s - 1) * A_NFIELDS, *a0 = tot + (int64_t)s * A_NFIELDS;
            const double eq5_first = P.kT * (lse_value(a1[A_MR], a1[A_SR]) - log(a1[A_N]));
            const double eq5_last = P.kT * (lse_value(as[A_MF], as[A_SF]) - log(as[A_N]));
            const double eq6_first = -P.kT * (lse_value(a0[A_MF], a0[A_SF]) - log(a0[A_N]));
            const double eq6_last = -P.kT * (lse_value(a0[A_MR], a0[A_SR]) - log(a0[A_N]));
            turn[PPP_ON_EQ5_FIRST] = eq5_first;
            turn[PPP_ON_EQ6_FIRST] = eq6_first;
            turn[PPP_ON_EQ5_LAST] = eq5_last;
            turn[PPP_ON_EQ6_LAST] = eq6_last;
            turn[PPP_ON_EQ10_LOG] = -P.beta * (eq6_first + OUT(O_DF_JE, s - 1) - eq5_last);
            // Eq. 7: <k/2 (x - lambda)^2> over the restrained window and over x_0
            const double dls = lam[s - 1] - lam[0];
            turn[PPP_ON_LOWER_FIRST] = 0.5 * P.k * a1[A_S2] / a1[A_N];
            turn[PPP_ON_UPPER_FIRST] = 0.5 * P.k * a0[A_S2] / a0[A_N];
            turn[PPP_ON_LOWER_LAST] = 0.5 * P.k * as[A_S2] / as[A_N];
            turn[PPP_ON_UPPER_LAST] = 0.5 * P.k * (a0[A_S2] - 2.0 * dls * a0[A_S1] + a0[A_N] * dls * dls) / a0[A_N];
            const WinStat f0 = win_stat(a0, lam[0]);
            turn[PPP_ON_FREE_N] = a0[A_N];
            turn[PPP_ON_FREE_BLOWN] = a0[A_BLOWN];
            turn[PPP_ON_FREE_MEAN] = f0.mean;
            turn[PPP_ON_FREE_STD] = sqrt(f0.var);
            turn[PPP_ON_FREE_UNDER] = a0[A_UNDER];
            turn[PPP_ON_FREE_OVER] = a0[A_OVER];
            s_eq5_first = eq5_first;
        } else {
            for (int f = 0; f < PPP_ON_NFIELDS; ++f) turn[f] = NAN;
            s_eq5_first = NAN;
        }
    }
    if (P.free_ens && B > 1)
        for (int b = t; b < B; b += 256)
            jt[b * JK_TURN + 4] = -P.beta * (jt[b * JK_TURN + 1] + jack[(int64_t)b * JK_FIELDS * s + s - 1] - jt[b * JK_TURN + 2]);
    __syncthreads();
    for (int j = t; j < s; j += 256) {
        const double je = OUT(O_DF_JE, j), fl = OUT(O_DF_FLUCT, j);
        OUT(O_DF_COM, j) = 0.5 * (je + fl);
        OUT(O_DF_UNC, j) = 0.5 * (je - fl);
        OUT(O_G, j) = je - s_eq5_first;                // Eq. 15; NaN without the free ensemble
        if (j > 0) {
            // Eqs. 14 and 13 as printed, lambda_j taken as the end point of j + 1 windows
            const double span = lam[j] - lam[0], npts = (double)(j + 1);
            const double fl_lit = P.k * span * OUT(O_DF_FLUCT_LIT, j) / npts;
            OUT(O_DF_GAUSS_LIT, j) = P.k * span * span / (2.0 * npts) * OUT(O_DF_GAUSS_LIT, j) / npts + fl_lit;
            OUT(O_DF_FLUCT_LIT, j) = fl_lit;
        }
    }
    const int se[JK_FIELDS] = {O_DF_JE_SE, O_DF_FLUCT_SE, O_DF_GAUSS_SE, O_DF_COM_SE, O_G_SE};
    for (int q = t; q < JK_FIELDS * s + (P.free_ens ? JK_TURN : 0); q += 256) {
        if (q >= JK_FIELDS * s) {
            const int f = q - JK_FIELDS * s;
            const int fields[JK_TURN] = {PPP_ON_EQ5_FIRST_SE, PPP_ON_EQ6_FIRST_SE, PPP_ON_EQ5_LAST_SE,
                                         PPP_ON_EQ6_LAST_SE, PPP_ON_EQ10_LOG_SE};
            turn[fields[f]] = jack_se(B, [&](int b) { return jt[b * JK_TURN + f]; });
            continue;
        }
        const int f = q / s, j = q % s;
        const double *row = jack + j;
        const int64_t step = (int64_t)JK_FIELDS * s;
        double e;
        if (f < 3) e = jack_se(B, [&](int b) { return row[b * step + (int64_t)f * s]; });
        else if (f == 3) e = jack_se(B, [&](int b) { return 0.5 * (row[b * step] + row[b * step + s]); });
        else e = P.free_ens ? jack_se(B, [&](int b) { return row[b * step] - jt[b * JK_TURN]; }) : NAN;
        OUT(se[f], j) = e;
    }
#undef OUT
}

hipError_t launch_estimators(const DevProblem *d_probs, int n_probs, char *ws, int max_windows, hipStream_t stream) {
    hipLaunchKernelGGL(k_windows, dim3(max_windows, n_probs), dim3(256), 0, stream, d_probs, ws);
    hipLaunchKernelGGL(k_profiles, dim3(n_probs), dim3(256), 0, stream, d_probs, ws);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// App. C.  For the step i -> i+1, every non-empty x bin b of rho_i moves the work
// by a whole number of bins and carries probability rho_i(b); consecutive
// non-empty bins with the same move are merged into one (shift, probability)
// pair (the move is monotone in b).  Chain 0: x at the bin centre, move
// floor(dW_i(x) / dW).  Chain 1, the listing as printed: x at the bin's upper
// edge and truncation toward zero of W = w dW + dW_i(x), i.e. the move is
// floor(f) for w + f >= 0 and ceil(f) below, f = dW_i(x) / dW; its pairs keep
// both and merge only where both agree.  Chain 2, the reverse path: the bins of
// rho_{i+1} with the work of moving the centre back, dW^rev_i(x) = k/2
// [(x - lambda_i)^2 - (x - lambda_{i+1})^2], x at the bin centre, move floor.
//
// One 256-thread block per (window step, problem, chain), bound by the block scans' barriers:
// some 2 us for 256 bins, so the bins outside the window's samples are left out (50000
// bins, most of them empty: 390 -> 22 us).  The bins are taken 256 at a time: the non-empty ones are compacted in order, run heads are marked, and
// each head sums its run left to right, the first run of a chunk continuing the
// last one of the previous chunk where the shifts agree, so every probability is
// the same left-to-right sum as in a sequential pass.
__device__ __forceinline__ int block_excl_scan(int v, int *sh, int &total) {
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const int a = t >= off ? sh[t - off] : 0;
        __syncthreads();
        sh[t] += a;
        __syncthreads();
    }
    total = sh[255];
    const int r = sh[t] - v;
    __syncthreads();
    return r;
}

__device__ __forceinline__ int clamp_shift(double f) {
    return f > 2.0e9 ? 2000000000 : (f < -2.0e9 ? -2000000000 : (int)f);
}

__global__ __launch_bounds__(256) void k_appc_pairs(const DevProblem *__restrict__ probs, char *__restrict__ ws) {
#pragma clang fp contract(off)
    const DevProblem &P = probs[blockIdx.y];
    const int i = blockIdx.x, chain = blockIdx.z, t = threadIdx.x;
    if (P.w_half_bins <= 0 || i + 1 >= P.n_windows) return;
    const int K = P.xi_nbins;
    const int64_t sK = (int64_t)P.n_windows * K;
    const double *lam = dptr(ws, P.off_lambda);
    const double *tot = dptr(ws, P.off_tot);
    const int src = chain == 2 ? i + 1 : i;         // window whose x distribution is folded in
    const unsigned long long *hist = reinterpret_cast<const unsigned long long *>(ws + P.off_hist) + (int64_t)src * K;
    int *key0 = reinterpret_cast<int *>(ws + P.off_pairs_shift) + chain * sK + (int64_t)i * K;
    int *key1 = reinterpret_cast<int *>(ws + P.off_pairs_ceil) + (int64_t)i * K;   // chain 1 only
    double *prob = dptr(ws, P.off_pairs_prob) + chain * sK + (int64_t)i * K;
    const double n = tot[(int64_t)src * A_NFIELDS + A_N];
    const double li = lam[i], lj = lam[i + 1];
    __shared__ int s_scan[256];
    __shared__ int s_k0[256], s_k1[256], s_head[256];
    __shared__ double s_pb[256];
    // the bins between the window's smallest and largest sample, and one on either side
    const double *rec = tot + (int64_t)src * A_NFIELDS;
    const double d_lo = floor((rec[A_XMIN] - P.xi_min) / P.xi_bin) - 1.0;
    const double d_hi = floor((rec[A_XMAX] - P.xi_min) / P.xi_bin) + 1.0;
    const int b_lo = d_lo < 0.0 ? 0 : (d_lo < (double)K ? (int)d_lo : K);
    const int b_hi = d_hi < 0.0 ? -1 : (d_hi < (double)K ? (int)d_hi : K - 1);
    int np = 0, last0 = 0, last1 = 0;
    for (int c0 = b_lo; c0 <= b_hi; c0 += 256) {
        const int b = c0 + t;
        const unsigned long long c = b <= b_hi ? hist[b] : 0ull;
        int k0 = 0, k1 = 0;
        double pb = 0.0;
        if (c != 0ull) {
            pb = (double)c / n;
            if (chain != 1) {
                const double xb = P.xi_min + ((double)b + 0.5) * P.xi_bin;
                const double la = chain == 0 ? li : lj, lb = chain == 0 ? lj : li;   // from la to lb
                const double dW = 0.5 * P.k * ((xb - lb) * (xb - lb) - (xb - la) * (xb - la));
                k0 = k1 = clamp_shift(floor(dW / P.w_bin));
            } else {
                const double xb = P.xi_min + ((double)b + 1.0) * P.xi_bin;
                const double f = 0.5 * P.k * ((xb - lj) * (xb - lj) - (xb - li) * (xb - li)) / P.w_bin;
                k0 = clamp_shift(floor(f));
                k1 = clamp_shift(ceil(f));
            }
        }
        int nnz;
        const int pos = block_excl_scan(c != 0ull ? 1 : 0, s_scan, nnz);
        if (c != 0ull) { s_k0[pos] = k0; s_k1[pos] = k1; s_pb[pos] = pb; }
        __syncthreads();
        int head = 0;
        if (t < nnz) {
            const int p0 = t ? s_k0[t - 1] : last0, p1 = t ? s_k1[t - 1] : last1;
            head = (t == 0 && np == 0) || s_k0[t] != p0 || s_k1[t] != p1;
            s_head[t] = head;
        }
        int nheads;
        const int rid = block_excl_scan(head, s_scan, nheads);
        if (head) {
            double p = s_pb[t];
            for (int m = t + 1; m < nnz && !s_head[m]; ++m) p += s_pb[m];
            key0[np + rid] = s_k0[t];
            if (chain == 1) key1[np + rid] = s_k1[t];
            prob[np + rid] = p;
        } else if (t == 0 && nnz > 0) {
            // the chunk opens inside the previous chunk's last run
            double p = prob[np - 1];
            for (int m = 0; m < nnz && !s_head[m]; ++m) p += s_pb[m];
            prob[np - 1] = p;
        }
        if (nnz > 0) { last0 = s_k0[nnz - 1]; last1 = s_k1[nnz - 1]; }
        np += nheads;
        __syncthreads();
    }
    if (t == 0) reinterpret_cast<int *>(ws + P.off_npairs)[chain * P.n_windows + i] = np;
}

// Omega_j(w) = sum_t prob_t Omega_{j-1}(w - shift_t), the folding step of App. C,
// for the three chains (blockIdx.z; chain 2, the reverse path, folds like chain 0).
// Chain 1 folds as printed: target w > 0 takes source w - floor(f),
// w < 0 takes w - ceil(f); at w = 0 the printed step keeps the mean of the
// results at w = -1 and w = +1 instead, which are exactly what the targets -1 and
// +1 compute, so the bin is left unsmoothed here and every reader of Omega_j
// (j >= 1) of chain 1 takes the mean of its neighbours there (omega_at).
//
// A block owns 256 consecutive target bins.  Pairs are taken 256 at a time; for
// each, the sources that the block's targets read lie in 259 consecutive bins
// (one spare on either side), which are staged in LDS together with those of
// the other pairs of the chunk, so the inner loop is one LDS read and one FMA per
// pair.  Pairs whose sources cannot all share one staging window of kAppcStage
// bins are taken in further windows; pairs whose sources lie wholly outside the
// histogram get weight 0.  With one window the sums run in pair order.
constexpr int kAppcStage = 4096;
constexpr int kAppcSpan = 259;                  // sources of one pair for one block

__device__ __forceinline__ double omega_at(const double *om, int64_t b, int M, bool smooth) {
    return (smooth && b == M) ? 0.5 * (om[M - 1] + om[M + 1]) : om[b];
}

__device__ __forceinline__ int64_t block_min_max(int64_t v, bool is_min, int64_t *sh) {
    for (int off = 32; off >= 1; off >>= 1) {
        const int64_t o = __shfl_xor(v, off);
        v = is_min ? (o < v ? o : v) : (o > v ? o : v);
    }
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    int64_t r = sh[0];
    for (int q = 1; q < 4; ++q) r = is_min ? (sh[q] < r ? sh[q] : r) : (sh[q] > r ? sh[q] : r);
    __syncthreads();
    return r;
}

__global__ __launch_bounds__(256) void k_appc_step(const DevProblem *__restrict__ probs, char *__restrict__ ws, int j) {
    const DevProblem &P = probs[blockIdx.y];
    if (P.w_half_bins <= 0 || j >= P.n_windows) return;
    const int chain = blockIdx.z;
    const int M = P.w_half_bins;
    const int64_t nb = 2 * (int64_t)M + 1;
    const int64_t w0 = (int64_t)blockIdx.x * 256;
    if (w0 >= nb) return;
    const int64_t sK = (int64_t)P.n_windows * P.xi_nbins;
    const int64_t w = w0 + threadIdx.x;
    const int np = reinterpret_cast<const int *>(ws + P.off_npairs)[chain * P.n_windows + j - 1];
    const int *shift = reinterpret_cast<const int *>(ws + P.off_pairs_shift) + chain * sK + (int64_t)(j - 1) * P.xi_nbins;
    const int *ceil_s = reinterpret_cast<const int *>(ws + P.off_pairs_ceil) + (int64_t)(j - 1) * P.xi_nbins;
    const double *prob = dptr(ws, P.off_pairs_prob) + chain * sK + (int64_t)(j - 1) * P.xi_nbins;
    const double *prev = dptr(ws, P.off_omega) + chain * (int64_t)P.n_windows * nb + (int64_t)(j - 1) * nb;
    double *cur = dptr(ws, P.off_omega) + chain * (int64_t)P.n_windows * nb + (int64_t)j * nb;
    const bool smooth_prev = chain == 1 && j >= 2;
    __shared__ int s_sf[256], s_sc[256], s_win[256];
    __shared__ double s_prob[256];
    __shared__ int64_t s_red[4];
    __shared__ double s_src[kAppcStage];
    // chain 1 below W = 0 reads through ceil(f), everything else through floor(f)
    const int *sel = (chain == 1 && w < M) ? s_sc : s_sf;
    constexpr int64_t kNone = INT64_MAX;
    constexpr int64_t step = kAppcStage - kAppcSpan;
    double acc = 0.0;
    for (int t0 = 0; t0 < np; t0 += 256) {
        const int cnt = np - t0 < 256 ? np - t0 : 256;
        const int t = threadIdx.x;
        int sf = 0, sc = 0;
        double pt = 0.0;
        int64_t first = kNone;
        if (t < cnt) {
            sf = shift[t0 + t];
            sc = chain == 1 ? ceil_s[t0 + t] : sf;
            pt = prob[t0 + t];
            first = w0 - 1 - (int64_t)(sc > sf ? sc : sf);
            if (first + kAppcSpan <= 0 || first >= nb) first = kNone;    // reads nothing in range
        }
        const int64_t base = block_min_max(first, true, s_red);
        if (base == kNone) continue;                                      // uniform
        const int64_t top = block_min_max(first == kNone ? INT64_MIN : first, false, s_red);
        if (t < cnt) {
            if (first == kNone) {          // weight 0, reading a staged bin of the first window
                sf = sc = (int)(w0 - 1 - base);
                pt = 0.0;
                first = base;
            }
            s_sf[t] = sf;
            s_sc[t] = sc;
            s_prob[t] = pt;
            s_win[t] = (int)((first - base) / step);
        }
        const int n_win = (int)((top - base) / step) + 1;
        for (int win = 0; win < n_win; ++win) {
            const int64_t start = base + (int64_t)win * step;
            const int64_t len = top - start + kAppcSpan < kAppcStage ? top - start + kAppcSpan : kAppcStage;
            for (int q = threadIdx.x; q < len; q += 256) {
                const int64_t src = start + q;
                s_src[q] = (src >= 0 && src < nb) ? omega_at(prev, src, M, smooth_prev) : 0.0;
            }
            __syncthreads();
            if (w < nb) {
                const int off = (int)(w - start);   // s_src[off - s] = Omega_{j-1}(w - s)
                if (n_win == 1) {
#pragma unroll 8
                    for (int u = 0; u < cnt; ++u) acc += s_prob[u] * s_src[off - sel[u]];
                } else {
                    for (int u = 0; u < cnt; ++u)
                        if (s_win[u] == win) acc += s_prob[u] * s_src[off - sel[u]];
                }
            }
            __syncthreads();
        }
    }
    if (w < nb) cur[w] = acc;
}

// Statistics of Omega_j: normalised exponential average (App. B.5), spread and
// the number of non-empty bins, the JE variance formula of Sec. IV A.  One block per
// (window, problem, chain), bound by the latency of its passes over the bins, so a thread
// has eight loads in flight; it adds in bin order all the same (1 - the sum is an output
// of rounding size).  One load at a time: 131 us over 30001 bins, 297 over 90001; so:
// 71 and 135 us.
constexpr int kAppcAhead = 8;
__global__ __launch_bounds__(256) void k_appc_stats(const DevProblem *__restrict__ probs, char *__restrict__ ws) {
    const DevProblem &P = probs[blockIdx.y];
    const int j = blockIdx.x;
    const int chain = blockIdx.z;
    __shared__ double sh[256];
    const int s = P.n_windows;
    if (P.w_half_bins <= 0 || j >= s) return;
    const int M = P.w_half_bins;
    const int64_t nb = 2 * (int64_t)M + 1;
    const double *om = dptr(ws, P.off_omega) + chain * (int64_t)s * nb + (int64_t)j * nb;
    double *out = dptr(ws, P.off_out);
    const double beta = P.beta, dWb = P.w_bin;
    const double shift_mid = 0.5 * (double)j * dWb;
    double tot = 0, q = 0, mw = 0, emax = -INFINITY;
    const bool smooth = chain == 1 && j >= 1;   // chain 1 keeps W = 0 unsmoothed in memory
    auto bins = [&](auto &&use) {               // use(b, Omega_j(b)) for the thread's non-empty bins, in order
        for (int64_t b0 = threadIdx.x; b0 < nb; b0 += 256 * kAppcAhead) {
            double o[kAppcAhead];
#pragma unroll
            for (int r = 0; r < kAppcAhead; ++r) o[r] = b0 + 256 * r < nb ? om[b0 + 256 * r] : 0.0;
#pragma unroll
            for (int r = 0; r < kAppcAhead; ++r) {
                const int64_t b = b0 + 256 * r;
                if (smooth && b == M) o[r] = omega_at(om, M, M, true);
                if (o[r] != 0.0) use(b, o[r]);
            }
        }
    };
    bins([&](int64_t b, double o) {
        const double W = (double)(b - M) * dWb;
        tot += o; q += 1.0; mw += o * W;
        emax = fmax(emax, -beta * W);
    });
    tot = block_sum(tot, sh);
    q = block_sum(q, sh);
    mw = block_sum(mw, sh);
    // block max
    sh[threadIdx.x] = emax;
    __syncthreads();
    for (int off = 128; off >= 1; off >>= 1) {
        if ((int)threadIdx.x < off) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + off]);
        __syncthreads();
    }
    emax = sh[0];
    __syncthreads();
    const double mean = mw / tot;
    double sl = 0, sm = 0, vv = 0;
    bins([&](int64_t b, double o) {
        const double W = (double)(b - M) * dWb;
        sl += o * exp(-beta * W - emax);
        sm += o * exp(-beta * (W + shift_mid) - emax);
        vv += o * (W - mean) * (W - mean);
    });
    sl = block_sum(sl, sh);
    sm = block_sum(sm, sh);
    vv = block_sum(vv, sh);
    if (chain == 2) {
        // reverse JE over the path lambda_j -> lambda_1: <exp(-beta W_rev)> = exp(+beta dF_j)
        if (threadIdx.x == 0) out[(int64_t)O_DF_REV_HIST * s + j] = tot > 0 ? P.kT * (emax + log(sl / tot)) : NAN;
        // Crooks and Kofke: the forward distribution against the mirrored reverse one.
        // After j folds a forward bin w holds work in [w, w + j) dW and a reverse bin v
        // in [v, v + j) dW, so -W_rev matches forward bin w at v = -w - j.
        const double *of = dptr(ws, P.off_omega) + (int64_t)j * nb;      // chain 0
        double ovl = 0, wm = 0, wf = 0;
        for (int64_t b0 = threadIdx.x; b0 < nb; b0 += 256 * kAppcAhead) {
            double f[kAppcAhead], r[kAppcAhead];
#pragma unroll
            for (int q8 = 0; q8 < kAppcAhead; ++q8) {
                const int64_t b = b0 + 256 * q8, v = 2 * (int64_t)M - b - j;      // index of bin -w - j
                const bool in = b < nb && v >= 0 && v < nb;
                f[q8] = in ? of[b] : 0.0;
                r[q8] = in ? om[v] : 0.0;
            }
#pragma unroll
            for (int q8 = 0; q8 < kAppcAhead; ++q8) {
                const double m = fmin(f[q8], r[q8]);
                ovl += m;
                if (f[q8] > 0.0 && r[q8] > 0.0) {
                    // P_f(W) / P_r(-W) = exp(beta (W - dF)): each common bin gives W - kT ln(P_f / P_r)
                    wm += m;
                    wf += m * (((double)(b0 + 256 * q8 - M) + 0.5 * j) * dWb - P.kT * log(f[q8] / r[q8]));
                }
            }
        }
        ovl = block_sum(ovl, sh);
        wm = block_sum(wm, sh);
        wf = block_sum(wf, sh);
        if (threadIdx.x == 0) {
            out[(int64_t)O_CROOKS_OVL * s + j] = ovl;
            out[(int64_t)O_DF_CROOKS * s + j] = wm > 0 ? wf / wm : NAN;
        }
    } else if (threadIdx.x == 0 && chain == 1) {
        out[(int64_t)O_DF_JE_HIST_LIT * s + j] = tot > 0 ? -P.kT * (emax + log(sl / tot)) : NAN;
    } else if (threadIdx.x == 0) {
        const double kT = P.kT;
        const double sig = sqrt(fmax(vv / tot, 0.0));
        out[(int64_t)O_DF_JE_HIST * s + j] = tot > 0 ? -kT * (emax + log(sl / tot)) : NAN;
        out[(int64_t)O_DF_JE_HIST_MID * s + j] = tot > 0 ? -kT * (emax + log(sm / tot)) : NAN;
        out[(int64_t)O_SIGMA_W * s + j] = sig;
        out[(int64_t)O_Q_BINS * s + j] = q;
        out[(int64_t)O_WORK_LOST * s + j] = 1.0 - tot;
        double var = 0.0;
        if (j > 0 && q > 1.0) var = sig * sig / q + beta * beta * sig * sig * sig * sig / (2.0 * (q - 1.0));
        out[(int64_t)O_VAR_PAPER * s + j] = var;
    }
}

hipError_t launch_appc(const DevProblem *d_probs, int n_probs, char *ws, int max_windows, int max_m,
                       hipStream_t stream) {
    if (max_m <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_appc_pairs, dim3(max_windows, n_probs, kAppcChains), dim3(256), 0, stream, d_probs, ws);
    const int64_t nb = 2 * (int64_t)max_m + 1;
    const int grid = (int)((nb + 255) / 256);
    for (int j = 1; j < max_windows; ++j)
        hipLaunchKernelGGL(k_appc_step, dim3(grid, n_probs, kAppcChains), dim3(256), 0, stream, d_probs, ws, j);
    hipLaunchKernelGGL(k_appc_stats, dim3(max_windows, n_probs, kAppcChains), dim3(256), 0, stream, d_probs, ws);
    return hipGetLastError();
}

}  // namespace ppp
