// Simulation kernels (device code, included by the shape translation units) of the parallel pulling protocol (Sec. III(ii)): many
// independent restrained Langevin replicas per window lambda_i, all started
// from the shared state x_o, each recording xi every sample_every steps after
// n_equil and folding it straight into fp64 accumulators:
//   n, sum(xi - lambda_i), sum(xi - lambda_i)^2, min, max, the histogram rho_i,
//   and running log-sum-exp pairs of a = -beta dW_i (Eq. 9 summand) for the
//   forward step and of the reverse step, each also for 2a (Kish size).
//
// Two kernels:
//   * sim_1d: L lanes per replica, overdamped dynamics of one coordinate.
//   * sim_chain<T, G, B>: G consecutive lanes of a wavefront per replica (any G
//     up to 64; 64 / G groups per wavefront, the remaining lanes idle), B beads
//     per lane in registers (lane g owns beads gB .. gB+B-1).  The
//     Lennard-Jones sum uses each unique pair once (Newton's third law): the
//     j-beads rotate one lane per round through the group together with an
//     accumulator of their reaction forces, which finally is pushed back to
//     the owning lane (for even G the last round, which meets the opposite
//     lane, is done from both sides instead).  Each bond and angle is
//     computed once, by the lane owning its first or central bead, from a
//     one-bead halo read from the neighbouring lanes, which read back the
//     forces on their halo beads.  Inside the step loop nothing leaves
//     registers except each sample's accumulator update and histogram count
//     (LDS).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "ppp_device.hpp"
#include "ppp_launch.hpp"
#include "ppp_chain_force.hpp"

namespace ppp {

__device__ __forceinline__ double centre_at(const DevProblem &P, double lam, int64_t n) {
    if (P.n_pull <= 0 || n >= P.n_pull) return lam;
    return P.xi_start + (lam - P.xi_start) * ((double)n / (double)P.n_pull);
}

// Sequential protocol: every replica runs the windows one after another,
// n_steps each, with steps counted from the start of window 1.  A launch never
// crosses a window boundary, so its window is that of its first step.  The
// parallel protocol is the case of window 0 for every launch.
__device__ __forceinline__ int64_t seq_window(const DevProblem &P, int64_t step_begin) {
    return P.sequential ? step_begin / P.n_steps : 0;
}

// First step after `after` at which xi is sampled (steps n > n_equil with
// n - n_equil a multiple of sample_every); the loops then count up to it
// instead of taking a 64-bit remainder every step.
__device__ __forceinline__ int64_t next_sample_after(const DevProblem &P, int64_t after) {
    if (after < P.n_equil) return P.n_equil + P.sample_every;
    return P.n_equil + ((after - P.n_equil) / P.sample_every + 1) * P.sample_every;
}

// Per-replica constants of the sampling step: the forward and reverse exponents
// a = -beta dW of one sample, evaluated exactly as written below but with the
// window's lambda values read once per replica instead of once per sample.
// kind 1: a step to the neighbouring window, a = cf (d - h) with cf = beta k dl,
// h = dl/2, dl the centre's move, d = xi - lambda_w; kind 2: switching the
// restraint on or off, a = q e e with e = xi - ref.
struct SampleCoef {
    double lam_w;
    int kind_f, kind_r;
    double cf, hf, cr, hr;
    double qf, qr, ref_f, ref_r;
};

__device__ __forceinline__ SampleCoef sample_coef(const DevProblem &P, const double *lam, int w) {
    const int s = P.n_windows;
    SampleCoef c;
    c.lam_w = lam[w];
    c.kind_f = c.kind_r = 0;
    c.cf = c.hf = c.cr = c.hr = c.qf = c.qr = c.ref_f = c.ref_r = 0.0;
    const double bk = P.beta * P.k;
    if (w == s) {
        // the unrestrained ensemble (d = xi - lambda_1): switching the restraint on
        // at lambda_1 or at lambda_s costs W_H = k/2 (x_0 - lambda)^2 (Eqs. 4, 6)
        c.kind_f = c.kind_r = 2;
        c.qf = c.qr = -0.5 * P.beta * P.k;
        c.ref_f = lam[s];                 // lambda_1
        c.ref_r = lam[s - 1];
    } else {
        if (w + 1 < s) {
            // a = -beta k/2 [(xi - lambda_{i+1})^2 - (xi - lambda_i)^2] = beta k dl (d - dl/2)
            const double dl = lam[w + 1] - lam[w];
            c.kind_f = 1; c.cf = bk * dl; c.hf = 0.5 * dl;
        } else if (P.free_ens) {
            // switching the restraint at lambda_s off: a = +beta k/2 d^2 (Eq. 5)
            c.kind_f = 2; c.qf = 0.5 * P.beta * P.k; c.ref_f = lam[w];
        }
        if (w > 0) {
            const double dl = lam[w - 1] - lam[w];
            c.kind_r = 1; c.cr = bk * dl; c.hr = 0.5 * dl;
        } else if (P.free_ens) {
            c.kind_r = 2; c.qr = 0.5 * P.beta * P.k; c.ref_r = lam[w];   // the same at lambda_1 (Eq. 5)
        }
    }
    return c;
}

// exp(-y0) and exp(-y1), y >= 0: 2^n e^r with n = -rint(y / ln 2), |r| <= ln 2 / 2,
// the series of e^r to r^13 (the next term is 4e-18); within 0.66 units in the last
// place (the library's exp: 0.86).
#define PPP_EXP_SERIES                                                                                                  \
    1.4426950408889634, -0.6931471805599453, -2.3190468138462996e-17 /* log2 e, -ln 2 high, low */,                    \
    1.6059043836821613e-10, 2.08767569878681e-09, 2.505210838544172e-08, 2.755731922398589e-07, 2.7557319223985893e-06, \
    2.48015873015873e-05, 1.984126984126984e-04, 1.3888888888888889e-03, 8.333333333333333e-03, 4.1666666666666664e-02, \
    1.6666666666666666e-01
template <typename Table>
__device__ __forceinline__ void exp_neg2(const Table &tab, double y0, double y1, double &t0, double &t1) {
    y0 = y0 > 800.0 ? 800.0 : y0;             // e^-800 is 0
    y1 = y1 > 800.0 ? 800.0 : y1;
    const double n0 = rint(-y0 * tab[0]), n1 = rint(-y1 * tab[0]);
    const double h0 = fma(n0, tab[1], -y0), h1 = fma(n1, tab[1], -y1);       // exact
    const double r0 = fma(n0, tab[2], h0), r1 = fma(n1, tab[2], h1);
    const double l0 = fma(n0, tab[2], h0 - r0), l1 = fma(n1, tab[2], h1 - r1);
    double p0 = tab[3], p1 = p0;
#pragma unroll
    for (int i = 4; i < 14; ++i) {
        p0 = fma(p0, r0, tab[i]);
        p1 = fma(p1, r1, tab[i]);
    }
    p0 = fma(fma(p0, r0, 0.5), r0 * r0, l0);
    p1 = fma(fma(p1, r1, 0.5), r1 * r1, l1);
    const double s0 = 1.0 + r0, s1 = 1.0 + r1;                               // what it drops goes to the tail
    t0 = ldexp(s0 + (((1.0 - s0) + r0) + p0), (int)n0);
    t1 = ldexp(s1 + (((1.0 - s1) + r1) + p1), (int)n1);
}

// Where a sample's exponentials come from.  EXP_SERIES holds the coefficients in
// registers over the step loop, as the library's exp does (some 38 of them).  EXP_LDS
// reads them from LDS where they are used, at an offset that the compiler cannot see
// through, for the kernels whose registers decide how many wavefronts a SIMD holds
// (scalar loads from memory instead cost the 16x4 kernel 1% where a SIMD has one
// wavefront).  The two give the same bits.
enum ExpFrom { EXP_LIBRARY, EXP_SERIES, EXP_LDS };
constexpr int kExpTerms = 14;
__constant__ double kExpSeries[kExpTerms] = {PPP_EXP_SERIES};
template <ExpFrom E>
__device__ __forceinline__ void exp_pair(const double *lds_tab, double y0, double y1, double &t0, double &t1) {
    if constexpr (E == EXP_LDS) {
        int at = 0;
        asm volatile("" : "+v"(at));
        exp_neg2(lds_tab + at, y0, y1, t0, t1);
    } else {
        constexpr double tab[kExpTerms] = {PPP_EXP_SERIES};
        exp_neg2(tab, y0, y1, t0, t1);
    }
}

// Folds one sample xi of window w into the replica's accumulator.  The
// histogram count goes to the workgroup's LDS copy of window w's histogram
// (lhist) when there is one, else straight to memory.
template <ExpFrom E>
__device__ __forceinline__ void accumulate(const DevProblem &P, const SampleCoef &C, int w, double xi,
                                           double *acc, unsigned long long *hist, unsigned int *lhist,
                                           const double *lds_exp) {
    const double d = xi - C.lam_w;
    acc[A_N] += 1.0;
    acc[A_S1] += d;
    acc[A_S2] += d * d;
    acc[A_XMIN] = fmin(acc[A_XMIN], xi);
    acc[A_XMAX] = fmax(acc[A_XMAX], xi);
    if constexpr (E != EXP_LIBRARY) {
        const double ef = xi - C.ref_f, er = xi - C.ref_r;
        const double af = C.kind_f == 1 ? C.cf * (d - C.hf) : C.qf * ef * ef;
        const double ar = C.kind_r == 1 ? C.cr * (d - C.hr) : C.qr * er * er;
        const double df = af - acc[A_MF], dr = ar - acc[A_MR];
        double tf, tr;
        exp_pair<E>(lds_exp, fabs(df), fabs(dr), tf, tr);
        if (C.kind_f) lse_fold(acc[A_MF], acc[A_SF], acc[A_MF2], acc[A_SF2], af, df > 0.0, tf);
        if (C.kind_r) lse_fold(acc[A_MR], acc[A_SR], acc[A_MR2], acc[A_SR2], ar, dr > 0.0, tr);
    } else {
        if (C.kind_f == 1) {
            lse_push_pair(acc[A_MF], acc[A_SF], acc[A_MF2], acc[A_SF2], C.cf * (d - C.hf));
        } else if (C.kind_f == 2) {
            const double e = xi - C.ref_f;
            lse_push_pair(acc[A_MF], acc[A_SF], acc[A_MF2], acc[A_SF2], C.qf * e * e);
        }
        if (C.kind_r == 1) {
            lse_push_pair(acc[A_MR], acc[A_SR], acc[A_MR2], acc[A_SR2], C.cr * (d - C.hr));
        } else if (C.kind_r == 2) {
            const double e = xi - C.ref_r;
            lse_push_pair(acc[A_MR], acc[A_SR], acc[A_MR2], acc[A_SR2], C.qr * e * e);
        }
    }
    const double fb = floor((xi - P.xi_min) / P.xi_bin);
    if (fb < 0.0) acc[A_UNDER] += 1.0;
    else if (fb >= (double)P.xi_nbins) acc[A_OVER] += 1.0;
    else if (lhist) atomicAdd(lhist + (int)fb, 1u);
    else atomicAdd(hist + (int64_t)w * P.xi_nbins + (int64_t)fb, 1ull);
}

// Workgroup-private histogram: cleared before an item, added to the window's
// histogram in memory after it (one atomic per non-empty bin).
__device__ __forceinline__ void lhist_clear(unsigned int *lhist, int K) {
    for (int b = threadIdx.x; b < K; b += blockDim.x) lhist[b] = 0u;
    __syncthreads();
}
__device__ __forceinline__ void lhist_flush(unsigned int *lhist, int K, unsigned long long *dst) {
    __syncthreads();
    for (int b = threadIdx.x; b < K; b += blockDim.x) {
        const unsigned int c = lhist[b];
        if (c) atomicAdd(dst + b, (unsigned long long)c);
    }
    __syncthreads();
}

// Bins of the workgroup histogram of an item: K for every window its replicas
// fall in (INT32_MAX when that would not fit an int).
__device__ __forceinline__ int item_hist_bins(const DevProblem &P, const WorkItem &item) {
    const int64_t last = (int64_t)item.window * P.n_replicas + item.rep_begin + item.n_reps - 1;
    const int64_t nw = last / P.n_replicas - item.window + 1;
    const int64_t nk = nw * (int64_t)P.xi_nbins;
    return nk < (int64_t)INT32_MAX ? (int)nk : INT32_MAX;
}

template <typename T> __device__ __forceinline__ T *state_ptr(char *ws, const DevProblem &P) {
    return reinterpret_cast<T *>(ws + P.off_state);
}

// ===========================================================================
// 1-D overdamped model: x_{n+1} = x_n + mu dt F(x_n) + sqrt(mu kT dt/2) (eta_n + eta_{n+1})
// (Leimkuhler-Matthews) or + sqrt(2 mu kT dt) eta_{n+1} (Euler-Maruyama).
// eta_n is component n mod 4 of the Philox block with counter (gid, n div 4, 0, 0).
//
// L consecutive lanes share a replica.  Bound: the instruction latency of one
// wavefront (4 to 6 cycles an instruction while a SIMD holds one), not memory:
// the double-well workload (21 windows x 256 replicas) fills 84 wavefronts at a
// lane per replica, for 1024 SIMDs.  A replica's noise and its sampling
// exponentials do not depend on the step in hand, so the lanes draw the normals
// of a tile of 4L steps at once, one Philox block each, and all of them take the
// tile's steps (five dependent products each), each block's normals broadcast
// from its lane by DPP moves: through LDS they cost a third more, its reads being
// shared by the CU's wavefronts.  Pending samples wait in a lane each until the
// next tile's might not fit, and are then folded together, every lane evaluating
// its sample's exponentials.  Only the sums that keep the samples' order are
// serial: one fused product per sample, each sum on a lane of its own.  20000
// steps of that workload in fp64: 12.3 ms at a lane per replica, 1.4 ms here;
// 21 x 4096 replicas, 2000 steps: 1.75 and 0.65 ms.
// ===========================================================================
// Orders a wavefront's LDS accesses before and after it (its lanes exchange data
// through LDS without a workgroup barrier; the hardware keeps one wavefront's LDS
// accesses in order, this keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <typename T, int POT>
__device__ __forceinline__ T step_1d(T x, T c0, T b, T centre, T kr, T mu_dt, T amp, T e) {
    // explicit fused products: the same rounding in the block loop and the edge loop
    const T f = POT == 0 ? (c0 * x) * fma_t(x, x, -b) : c0 * x;
    return fma_t(e, amp, fma_t(fma_t(-kr, x - centre, f), mu_dt, x));
}

template <typename T>
__device__ __forceinline__ T force_1d(const DevProblem &P, T x, T centre, T kr) {
    T f;
    if (P.pot_kind == 0) f = (T)(-4.0 * P.pot_a) * x * (x * x - (T)P.pot_b);
    else f = (T)(-P.pot_kappa) * x;
    return f - kr * (x - centre);
}

// Restraint stiffness of window w: k, or 0 for the unrestrained ensemble (w = s).
__device__ __forceinline__ double window_k(const DevProblem &P, int w) { return w < P.n_windows ? P.k : 0.0; }

// Lane l - OFF's value inside a row of 16 lanes (a DPP move: no trip through LDS).
template <int OFF> __device__ __forceinline__ double row_shr(double v) {
    I2 w = __builtin_bit_cast(I2, v);
    w.lo = __builtin_amdgcn_update_dpp(w.lo, w.lo, 0x110 + OFF, 0xf, 0xf, false);
    w.hi = __builtin_amdgcn_update_dpp(w.hi, w.hi, 0x110 + OFF, 0xf, 0xf, false);
    return __builtin_bit_cast(double, w);
}

// Running maximum of a over the group's lanes up to and including this one.
template <int L> __device__ __forceinline__ double group_prefix_max(double a) {
    const int l = (int)threadIdx.x & (L - 1);
    double v = a;
    if constexpr (L > 1) { const double o = row_shr<1>(v); v = l >= 1 ? fmax(v, o) : v; }
    if constexpr (L > 2) { const double o = row_shr<2>(v); v = l >= 2 ? fmax(v, o) : v; }
    if constexpr (L > 4) { const double o = row_shr<4>(v); v = l >= 4 ? fmax(v, o) : v; }
    if constexpr (L > 8) { const double o = row_shr<8>(v); v = l >= 8 ? fmax(v, o) : v; }
    return v;
}

// The sums of a record that depend on the order of the samples: S1, S2 and the
// two log-sum-exp pairs.  Each takes a sample as S <- S alpha + beta; the
// (alpha, beta) of a sample are found by its lane, and sum f is carried by lane
// f mod L of the group.
constexpr int kOrderedSums = 6;

// LDS of one workgroup: the (alpha, beta) of up to L samples per group (none at one
// lane a replica, which leaves the LDS to the histogram).  Seven
// places of 16 bytes a lane for the six pairs, and six more between groups of 16
// lanes, so that the lanes of a wavefront that read one sample's pairs for their
// groups reach different banks.
template <int L> struct Lds1d {
    double2 ab[L == 1 ? 1 : WG * 7 + (WG / 16) * 6];
};
template <int L> __device__ __forceinline__ int ab_place(int thread) { return thread * 7 + (L == 16 ? (thread >> 4) * 6 : 0); }

// Lane B's value of the group, in every lane of it (DPP moves: no trip through LDS).
template <int L, int B> __device__ __forceinline__ int group_bcast(int v) {
    if constexpr (L == 16) return __builtin_amdgcn_update_dpp(v, v, 0x150 + B, 0xf, 0xf, false);
    else if constexpr (L == 8) {      // two groups a row of 16: lanes 0-7, then 8-15
        const int lo = __builtin_amdgcn_update_dpp(v, v, 0x150 + B, 0xf, 0x3, false);
        return __builtin_amdgcn_update_dpp(lo, v, 0x150 + 8 + B, 0xf, 0xc, false);
    }
    else if constexpr (L == 4) return __builtin_amdgcn_update_dpp(v, v, B * 0x55, 0xf, 0xf, false);
    else if constexpr (L == 2) return __builtin_amdgcn_update_dpp(v, v, B * 0x55 + 0xa0, 0xf, 0xf, false);
    else return v;
}
template <int L, int B> __device__ __forceinline__ float group_bcast(float v) {
    return __int_as_float(group_bcast<L, B>(__float_as_int(v)));
}
template <int L, int B> __device__ __forceinline__ double group_bcast(double v) {
    const I2 w = __builtin_bit_cast(I2, v);
    return __builtin_bit_cast(double, I2{group_bcast<L, B>(w.lo), group_bcast<L, B>(w.hi)});
}

template <int N, typename Fn> __device__ __forceinline__ void static_for(Fn &&fn) {
    if constexpr (N > 0) {
        static_for<N - 1>(fn);
        fn(std::integral_constant<int, N - 1>{});
    }
}

// First sampled step of a launch that ends with step n_end, n_end + 1 if it has none: the
// next sampled step itself may lie beyond 2^32 (n_equil and sample_every are bounded by
// 2^32 and 2^31 alone).  A launch from step 0 ends below 2^32 - 1 (launch_items), so
// n_end + 1 is never step 0, which the first tile holds.  After a sample the number may
// wrap, but only to less than the step just sampled, which no later step equals.
__device__ __forceinline__ uint32_t first_sample_1d(const DevProblem &P, int64_t s0, int64_t step_begin, uint32_t n_end) {
    // (as a minimum: with a select the fp32 kernel of 8 lanes gets a register allocation
    // that takes 1.02 ms for the 0.97 of 21 x 256 replicas' 20000 steps)
    const int64_t next = s0 + next_sample_after(P, step_begin - s0), none = (int64_t)n_end + 1;
    return (uint32_t)(next < none ? next : none);
}

template <typename T, int L, int POT>
__device__ __forceinline__ void sim_1d_replica(const DevProblem &P, int w, int rep, char *ws, int64_t step_begin,
                                               int64_t step_end, double *traj, int traj_rep, unsigned int *lhist,
                                               Lds1d<L> &lds) {
    const int l = (int)threadIdx.x & (L - 1);
    // record (window, replica); the sequential protocol keeps one state per replica
    // and draws replica `rep`'s window-1 noise all the way
    const int64_t g = (int64_t)w * P.n_replicas + rep;
    const int64_t gs = P.sequential ? rep : g;
    const uint32_t gid = (uint32_t)gs;
    const int64_t s0 = P.sequential ? (int64_t)w * P.n_steps : 0;   // first step of this window
    const double *lam = reinterpret_cast<const double *>(ws + P.off_lambda);
    double *acc_g = reinterpret_cast<double *>(ws + P.off_acc) + g * A_NFIELDS;
    unsigned long long *hist = reinterpret_cast<unsigned long long *>(ws + P.off_hist);
    T *st = state_ptr<T>(ws, P) + gs * 2;
    const double lam_w = lam[w];
    const SampleCoef C = sample_coef(P, lam, w);
    const double x_start = reinterpret_cast<const double *>(ws + P.off_init)[0];
    // step numbers stay below 2^32 (the runtime checks n_steps, and n_windows n_steps when sequential)
    const uint32_t n_end = (uint32_t)(step_end < s0 + P.n_steps ? step_end : s0 + P.n_steps);

    double acc[A_NFIELDS];
    T x, eta_prev;
    if (step_begin == 0) {
        acc_empty(acc);
        x = (T)x_start;
        T z[4];
        Normal4<T>::get(P.seed, gid, 0u, 0u, 0u, z);
        eta_prev = z[0];
    } else if (step_begin == s0) {
        // sequential protocol entering window w: the state goes on, the record starts
        // empty, and a replica frozen in the previous window stays frozen
        acc_empty(acc);
        acc[A_BLOWN] = acc_g[-(int64_t)P.n_replicas * A_NFIELDS + A_BLOWN];
        x = st[0]; eta_prev = st[1];
    } else {
        for (int f = 0; f < A_NFIELDS; ++f) acc[f] = acc_g[f];
        x = st[0]; eta_prev = st[1];
    }
    const bool record = traj != nullptr && g == traj_rep && l == 0;
    if (record && step_begin == 0) traj[0] = (double)x;
    const T kr = (T)window_k(P, w);
    const T mu_dt = (T)(P.mobility * P.dt);
    const bool lm = P.integrator_1d == 0;
    const T amp = lm ? (T)sqrt(0.5 * P.mobility * P.kT * P.dt) : (T)sqrt(2.0 * P.mobility * P.kT * P.dt);
    const T w_prev = lm ? (T)1 : (T)0;
    const T c0 = POT == 0 ? (T)(-4.0 * P.pot_a) : (T)(-P.pot_kappa), pb = (T)P.pot_b;
    const T c_fix = (T)lam_w;
    bool alive = acc[A_BLOWN] == 0.0;
    T x_dead = x, eta_dead = eta_prev;             // where a frozen replica stopped; its lanes run on unread
    // the centre moves until step pull_end
    const uint32_t pull_end = (P.n_pull > 0 && (w == 0 || !P.sequential)) ? (uint32_t)P.n_pull : 0u;

    // fields read inside the loops, held in registers: the histogram's atomics keep
    // the compiler from carrying loads of the record across them
    const uint64_t seed = P.seed;
    const double bound = P.xi_bound, xi_min = P.xi_min, xi_bin = P.xi_bin, k_bins = (double)P.xi_nbins;
    const uint32_t every = (uint32_t)P.sample_every;
    unsigned long long *hist_w = hist + (int64_t)w * P.xi_nbins;

    // the forward and reverse exponents of a sample: c (e - h) or c e e with e = xi - ref
    const double ref_f = C.kind_f == 1 ? lam_w : C.ref_f, cf = C.kind_f == 1 ? C.cf : C.qf;
    const double ref_r = C.kind_r == 1 ? lam_w : C.ref_r, cr = C.kind_r == 1 ? C.cr : C.qr;

    const int t0 = (int)threadIdx.x & ~(L - 1), lane0 = lane_id() & ~(L - 1);
    const uint64_t group_mask = ((1ull << L) - 1) << lane0;
    constexpr uint32_t kTile = 4u * L;             // steps whose normals are drawn together
    const int per_tile = every < kTile ? (int)((kTile - 1u) / every) + 1 : 1;   // most samples in a tile
    int cnt = 0;                                   // pending samples, the j-th in lane j of the group
    T xs[4] = {0, 0, 0, 0}, es[4] = {0, 0, 0, 0};  // this lane's: xs[qs], and es[qs] the normal of its step
    int qs = 0;
    double x_min = acc[A_XMIN], x_max = acc[A_XMAX];
    constexpr int kSumField[kOrderedSums] = {A_S1, A_S2, A_SF, A_SF2, A_SR, A_SR2};
    constexpr int kOwn = (kOrderedSums + L - 1) / L;   // sums carried by one lane
    double own[kOwn];
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        own[i] = 0.0;
#pragma unroll
        for (int f = 0; f < kOrderedSums; ++f) own[i] = f == i * L + l ? acc[kSumField[f]] : own[i];
    }

    uint32_t n = (uint32_t)step_begin, drawn = 1u;   // drawn: the tile z belongs to (tiles start at multiples of 4)
    uint32_t n_sample = first_sample_1d(P, s0, step_begin, n_end);
    T z[4];
    while (n < n_end && __any(alive)) {
        // the tile of step n + 1: kTile steps from `base`, block b of four steps with its normals in lane b
        const uint32_t base = (n + 1) & ~(kTile - 1u), last = base + kTile - 1u;
        if (base != drawn) {
            Normal4<T>::get(seed, gid, (base >> 2) + (uint32_t)l, 0u, 0u, z);
            drawn = base;
        }
        const uint32_t first = n + 1 - base;
        if ((first == 0 || n == 0) && last <= n_end && n >= pull_end && every >= 4u && !traj) {
            // a whole tile (its step 0, at the very start, is none) with the centre at
            // rest and at most one sample in four steps
            static_for<L>([&](auto bi) {
                constexpr int b = bi.value;
                T e[4], xq[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) e[q] = group_bcast<L, b>(z[q]);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (b > 0 || q > 0 || first == 0)
                        x = step_1d<T, POT>(x, c0, pb, c_fix, kr, mu_dt, amp, fma_t(w_prev, eta_prev, e[q]));
                    eta_prev = e[q];
                    xq[q] = x;
                }
                const uint32_t q = n_sample - (base + 4u * b);
                if (q < 4u) {
                    // the block's four positions; the fold picks the sampled one
                    if (l == cnt) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) { xs[i] = xq[i]; es[i] = e[i]; }
                        qs = (int)q;
                    }
                    n_sample += every;
                    ++cnt;
                }
            });
            n = last;
        } else {
            const uint32_t stop = last < n_end ? last : n_end;
            do {
                const uint32_t k = ++n - base;
                T eta = z[0];
#pragma unroll
                for (int q = 1; q < 4; ++q) eta = (k & 3u) == (uint32_t)q ? z[q] : eta;
                if constexpr (L > 1) eta = __shfl(eta, (int)(k >> 2), L);
                const T cen = pull_end > 0 ? (T)centre_at(P, lam_w, (int64_t)n - 1) : c_fix;
                x = step_1d<T, POT>(x, c0, pb, cen, kr, mu_dt, amp, fma_t(w_prev, eta_prev, eta));
                eta_prev = eta;
                if (record && alive && n <= 100000u) traj[n] = (double)x;
                if (n == n_sample) {
                    if (l == cnt) { xs[0] = x; es[0] = eta; qs = 0; }
                    n_sample += every;
                    ++cnt;
                    if (traj || cnt == L) break;
                }
            } while (n < stop);
        }
        // fold the pending samples when the next tile's might not fit, and at the end
        if (cnt == 0 || (cnt + per_tile <= L && n < n_end && !traj)) continue;
        const double xi = (double)(qs < 2 ? (qs ? xs[1] : xs[0]) : (qs == 2 ? xs[2] : xs[3]));
        if constexpr (L == 1) {
            // One lane a replica: nothing to exchange.  The same sums as below, rounded
            // alike, without the pairs, the ballots and the selects for lanes without a
            // sample, which set the pace where a sample is taken every few steps: 344064
            // replicas in fp32, a sample every step, 500 steps: 1.56 -> 1.18 ms (1.20 with
            // a lane per replica and one step after another); every tenth 0.28 -> 0.23;
            // with 16384 bins 0.88 -> 0.46.
#pragma clang fp contract(off)
            cnt = 0;
            if (!alive) continue;
            if (!isfinite(xi) || fabs(xi) > bound) {
                x_dead = (T)xi;
                eta_dead = qs < 2 ? (qs ? es[1] : es[0]) : (qs == 2 ? es[2] : es[3]);
                acc[A_BLOWN] = 1.0;
                alive = false;
                continue;
            }
            auto fold = [&](int kind, double c, double h, double ref, double &m, double &S, double &S2) {
                const double e = xi - ref;
                const double a = kind == 1 ? c * (e - h) : c * e * e;
                const double da = a - m, t = exp(-fabs(da)), t2 = t * t;
                const bool up = da > 0.0;
                S = up ? fma(S, t, 1.0) : S + t;
                S2 = up ? fma(S2, t2, 1.0) : S2 + t2;
                m = fmax(m, a);
            };
            const double d = xi - lam_w;
            own[0] += d;
            own[1] += d * d;
            if (C.kind_f) fold(C.kind_f, cf, C.hf, ref_f, acc[A_MF], own[2], own[3]);
            if (C.kind_r) fold(C.kind_r, cr, C.hr, ref_r, acc[A_MR], own[4], own[5]);
            x_min = fmin(x_min, xi);
            x_max = fmax(x_max, xi);
            acc[A_N] += 1.0;
            const double fb = floor((xi - xi_min) / xi_bin);
            if (fb < 0.0) acc[A_UNDER] += 1.0;
            else if (fb >= k_bins) acc[A_OVER] += 1.0;
            else if (lhist) atomicAdd(lhist + (int)fb, 1u);
            else atomicAdd(hist_w + (int64_t)fb, 1ull);
            continue;
        }
        const uint64_t bad = __ballot(l < cnt && (!isfinite(xi) || fabs(xi) > bound)) & group_mask;
        bool mine = l < cnt && alive;
        if (alive && bad) {
            // frozen at its first bad sample: later ones are dropped, its state stays there
            const int at = __ffsll((unsigned long long)(bad >> lane0)) - 1;
            x_dead = (T)__shfl(xi, at, L);
            eta_dead = __shfl(qs < 2 ? (qs ? es[1] : es[0]) : (qs == 2 ? es[2] : es[3]), at, L);
            acc[A_BLOWN] = 1.0;
            alive = false;
            mine = mine && l < at;
        }
        const double d = mine ? xi - lam_w : 0.0;
        const double ef = xi - ref_f, er = xi - ref_r;
        const double f1 = cf * (ef - C.hf), f2 = cf * ef * ef, r1 = cr * (er - C.hr), r2 = cr * er * er;
        const double af = mine && C.kind_f ? (C.kind_f == 1 ? f1 : f2) : -INFINITY;
        const double ar = mine && C.kind_r ? (C.kind_r == 1 ? r1 : r2) : -INFINITY;
        const double pf = group_prefix_max<L>(af), pr = group_prefix_max<L>(ar);
        // the maximum before this sample, and after all
        double mf = row_shr<1>(pf), mr = row_shr<1>(pr);
        mf = l > 0 ? fmax(acc[A_MF], mf) : acc[A_MF];
        mr = l > 0 ? fmax(acc[A_MR], mr) : acc[A_MR];
        acc[A_MF] = fmax(acc[A_MF], group_bcast<L, L - 1>(pf));
        acc[A_MR] = fmax(acc[A_MR], group_bcast<L, L - 1>(pr));
        const double df = af - mf, dr = ar - mr;
        const bool uf = df > 0.0, ur = dr > 0.0;
        // no sample, or no step in this direction: alpha = 1, beta = 0
        double tf = exp(-fabs(df)), tr = exp(-fabs(dr));
        tf = mine && C.kind_f ? tf : 0.0;
        tr = mine && C.kind_r ? tr : 0.0;
        const double tf2 = tf * tf, tr2 = tr * tr;
        double2 *ab = lds.ab + ab_place<L>((int)threadIdx.x);
        ab[0] = double2{1.0, d};
        ab[1] = double2{1.0, d * d};
        ab[2] = double2{uf ? tf : 1.0, uf ? 1.0 : tf};
        ab[3] = double2{uf ? tf2 : 1.0, uf ? 1.0 : tf2};
        ab[4] = double2{ur ? tr : 1.0, ur ? 1.0 : tr};
        ab[5] = double2{ur ? tr2 : 1.0, ur ? 1.0 : tr2};
        wave_lds_sync();
        // in sample order, so the sums do not depend on how the run is cut into launches
        // (lanes without a sample left alpha = 1, beta = 0)
#pragma unroll
        for (int i = 0; i < kOwn; ++i) {
            const double2 *ab_f = lds.ab + ab_place<L>(t0) + (i * L + l < kOrderedSums ? i * L + l : kOrderedSums - 1);
            double2 v[L];
#pragma unroll
            for (int j = 0; j < L; ++j) v[j] = ab_f[7 * j];
#pragma unroll
            for (int j = 0; j < L; ++j) own[i] = fma(own[i], v[j].x, v[j].y);
        }
        wave_lds_sync();
        bool under = false, over = false;
        if (mine) {
            x_min = fmin(x_min, xi);
            x_max = fmax(x_max, xi);
            const double fb = floor((xi - xi_min) / xi_bin);
            if (fb < 0.0) under = true;
            else if (fb >= k_bins) over = true;
            else if (lhist) atomicAdd(lhist + (int)fb, 1u);
            else atomicAdd(hist_w + (int64_t)fb, 1ull);
        }
        acc[A_N] += (double)__popcll(__ballot(mine) & group_mask);
        acc[A_UNDER] += (double)__popcll(__ballot(under) & group_mask);
        acc[A_OVER] += (double)__popcll(__ballot(over) & group_mask);
        cnt = 0;
    }
#pragma unroll
    for (int off = 1; off < L; off <<= 1) {
        x_min = fmin(x_min, __shfl_xor(x_min, off, L));
        x_max = fmax(x_max, __shfl_xor(x_max, off, L));
    }
    acc[A_MF2] = 2.0 * acc[A_MF]; acc[A_MR2] = 2.0 * acc[A_MR];
    acc[A_XMIN] = x_min; acc[A_XMAX] = x_max;
    if constexpr (L == 1) {
        // the whole record in one run of stores: an advance by single steps is bound by it
        for (int f = 0; f < kOrderedSums; ++f) acc[kSumField[f]] = own[f];
        for (int f = 0; f < A_NFIELDS; ++f) acc_g[f] = acc[f];
        st[0] = alive ? x : x_dead; st[1] = alive ? eta_prev : eta_dead;
        return;
    }
    if (l == 0) {
        for (int f = 0; f < A_NFIELDS; ++f)
            if (f != A_S1 && f != A_S2 && f != A_SF && f != A_SF2 && f != A_SR && f != A_SR2) acc_g[f] = acc[f];
        st[0] = alive ? x : x_dead; st[1] = alive ? eta_prev : eta_dead;
    }
#pragma unroll
    for (int i = 0; i < kOwn; ++i)
        if (i * L + l < kOrderedSums) {
            const int f = i * L + l;
            acc_g[f < 2 ? A_S1 + f : (f < 4 ? (f == 2 ? A_SF : A_SF2) : (f == 4 ? A_SR : A_SR2))] = own[i];
        }
}

// Each of the n_runs runs is `reps` replicas of one window, in items of WG (the
// workspace does not depend on the lanes), and takes workgroups of WG / L replicas: none
// of them empty, as consecutive workgroups go round the eight XCDs (with the items'
// ends as workgroups' ends, 172 windows of 257 replicas took a third longer).
template <typename T, int L>
__global__ __launch_bounds__(WG) void sim_1d(const DevProblem *__restrict__ probs, const WorkItem *__restrict__ items,
                                             int n_runs, int reps, char *__restrict__ ws, int64_t step_begin,
                                             int64_t step_end, double *__restrict__ traj, int traj_rep, int lds_cap) {
    extern __shared__ unsigned int s_hist[];
    __shared__ Lds1d<L> lds;
    const int parts = (reps + WG / L - 1) / (WG / L), run = (int)blockIdx.x / parts;
    if (run >= n_runs) return;
    const WorkItem item = items[(int64_t)run * ((reps + WG - 1) / WG)];
    const DevProblem &P = probs[item.prob];
    const int w = P.sequential ? (int)seq_window(P, step_begin) : item.window;
    const int r = ((int)blockIdx.x - run * parts) * (WG / L) + (int)threadIdx.x / L;
    unsigned int *lhist = P.xi_nbins <= lds_cap ? s_hist : nullptr;
    if (lhist) lhist_clear(lhist, P.xi_nbins);
    if (r < reps) {
        if (P.pot_kind == 0) sim_1d_replica<T, L, 0>(P, w, item.rep_begin + r, ws, step_begin, step_end, traj, traj_rep, lhist, lds);
        else sim_1d_replica<T, L, 1>(P, w, item.rep_begin + r, ws, step_begin, step_end, traj, traj_rep, lhist, lds);
    }
    if (lhist) lhist_flush(lhist, P.xi_nbins, reinterpret_cast<unsigned long long *>(ws + P.off_hist) + (int64_t)w * P.xi_nbins);
}


// Shapes with the Lennard-Jones rounds in assembly (ASM): fp32, four beads a lane, two
// rounds or more after the first.  Such a kernel fetches the exponentials' coefficients
// and keeps the samples' in LDS: rounds and sampling together then fit the registers of
// three waves per SIMD (64x4: 165 instead of 197), which is where the rounds gain most.
// At two the groups of 8 to 32 lanes still gain or break even; 64x4 loses 5%, so it has
// the compiled kernel as well.  All kernels of such a shape use the same series, so a
// replica's record is the same whichever runs it.
template <typename T, int G, int B> constexpr bool asm_shape() { return sizeof(T) == 4 && chain_asm_rounds(G, B); }
template <typename T, int G, int B> constexpr bool asm_only() { return asm_shape<T, G, B>() && G < 64; }
template <typename T, int G, int B> constexpr ExpFrom exp_here() { return asm_shape<T, G, B>() ? EXP_SERIES : EXP_LIBRARY; }

// What a workgroup of a chain kernel keeps in LDS besides the histogram: its
// replicas' records and, with ASM, their coefficients and those of exp.
template <int G, bool ASM> struct ChainLds {
    // 16-byte accesses, but for the ASM kernels, which they cost 8 registers
    alignas(ASM ? 8 : 16) double acc[chain_reps_per_wg(G)][A_NFIELDS];
    SampleCoef coef[ASM ? chain_reps_per_wg(G) : 1];
    double exp[ASM ? kExpTerms : 1];
};

template <typename T, int G, int B, bool ASM, ExpFrom E>
__device__ __forceinline__ void run_chain_item(const DevProblem &P, const WorkItem &item, char *ws, int64_t step_begin,
                                               int64_t step_end, double *traj, int64_t traj_rep, ChainLds<G, ASM> &lds,
                                               unsigned int *lhist) {
    constexpr int NPAD = G * B;
    constexpr int GPW = groups_per_wave(G);
    const int lane = lane_id();
    const bool lane_used = lane < GPW * G;
    const int grp = (int)(threadIdx.x >> 6) * GPW + (lane_used ? lane / G : 0);
    const int g = lane_used ? lane % G : 0;
    const int gbase = lane_used ? lane - g : lane;
    const bool active = lane_used && grp < item.n_reps;
    const int N = P.n_beads;
    const int64_t gfirst = (int64_t)item.window * P.n_replicas + item.rep_begin;
    // gi: replica number (window * R + replica); the sequential protocol's items are
    // window-1 replicas that run window `stage` in this launch
    const int64_t gi = gfirst + (active ? grp : 0);
    const int64_t stage = seq_window(P, step_begin);
    const int64_t s0 = stage * P.n_steps;         // first step of this window (0: parallel protocol)
    const int w = P.sequential ? (int)stage : (int)(gi / P.n_replicas);   // this replica's window now
    const int64_t grec = P.sequential ? stage * P.n_replicas + gi : gi;   // its record
    const uint32_t gid = (uint32_t)gi;
    // the workgroup's histogram holds the windows item.window, item.window + 1, ...
    // (the one window `stage` in the sequential protocol)
    unsigned int *lhist_w = lhist ? lhist + (P.sequential ? 0 : (int64_t)(w - item.window) * P.xi_nbins) : nullptr;
    const double *lam = reinterpret_cast<const double *>(ws + P.off_lambda);
    const double *x0 = reinterpret_cast<const double *>(ws + P.off_init);
    unsigned long long *hist = reinterpret_cast<unsigned long long *>(ws + P.off_hist);
    double *acc_g = reinterpret_cast<double *>(ws + P.off_acc) + grec * A_NFIELDS;
    T *st = state_ptr<T>(ws, P) + gi * 6 * NPAD;
    const double lam_w = lam[w];
    const int64_t n_end = step_end < s0 + P.n_steps ? step_end : s0 + P.n_steps;
    auto centre = [&](int64_t n) { return stage == 0 ? centre_at(P, lam_w, n) : lam_w; };
    const T kr = (T)window_k(P, w);
    const int i0 = g * B;
    const int last = N - 1;
    const int owner = last / B;       // lane (within group) owning the pulled end
    double *acc = lds.acc[grp];
    SampleCoef coef_here;
    if constexpr (ASM) {
        // every wavefront writes all of them, so none waits for another
        if (E == EXP_LDS && lane < kExpTerms) lds.exp[lane] = kExpSeries[lane];
        if (lane_used && g == owner) lds.coef[grp] = sample_coef(P, lam, w);
    } else {
        coef_here = sample_coef(P, lam, w);
    }
    const SampleCoef &coef = ASM ? lds.coef[ASM ? grp : 0] : coef_here;

    T px[B], py[B], pz[B], vx[B], vy[B], vz[B], fx[B], fy[B], fz[B];
    if (step_begin == 0) {
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int i = i0 + b;
            if (i < N) { px[b] = (T)x0[3 * i]; py[b] = (T)x0[3 * i + 1]; pz[b] = (T)x0[3 * i + 2]; }
            else { px[b] = 0; py[b] = 0; pz[b] = (T)(P.pad_z0 + P.pad_dz * (i - N)); }
        }
        lane_noise<T, B>(P, gid, 0u, i0, [&](int b, const T *z) {
            const int i = i0 + b;
            const bool mobile = i > 0 && i < N;
            vx[b] = mobile ? (T)P.sd_v * z[0] : (T)0;
            vy[b] = mobile ? (T)P.sd_v * z[1] : (T)0;
            vz[b] = mobile ? (T)P.sd_v * z[2] : (T)0;
        });
        if (lane_used && g == owner) acc_empty(acc);
    } else {
#pragma unroll
        for (int b = 0; b < B; ++b) {
            px[b] = st[0 * NPAD + i0 + b]; py[b] = st[1 * NPAD + i0 + b]; pz[b] = st[2 * NPAD + i0 + b];
            vx[b] = st[3 * NPAD + i0 + b]; vy[b] = st[4 * NPAD + i0 + b]; vz[b] = st[5 * NPAD + i0 + b];
        }
        if (lane_used && g == owner) {
            if (step_begin == s0) {
                // sequential protocol entering window `stage`: the record starts empty,
                // and a replica frozen in the previous window stays frozen
                acc_empty(acc);
                acc[A_BLOWN] = acc_g[-(int64_t)P.n_replicas * A_NFIELDS + A_BLOWN];
            } else {
                for (int f = 0; f < A_NFIELDS; ++f) acc[f] = acc_g[f];
            }
        }
    }
    const bool record = traj != nullptr && gi == traj_rep && active;
    if (record && step_begin == 0) {
#pragma unroll
        for (int b = 0; b < B; ++b)
            if (i0 + b < N) { traj[3 * (i0 + b)] = (double)px[b]; traj[3 * (i0 + b) + 1] = (double)py[b]; traj[3 * (i0 + b) + 2] = (double)pz[b]; }
    }
    // group-uniform liveness (owner's accumulator holds the flag)
    const int blown0 = (g == owner) ? (int)acc[A_BLOWN] : 0;
    const uint64_t bal0 = __ballot(blown0 != 0);
    bool alive = active && ((bal0 >> gbase) & ((G == 64) ? ~0ull : ((1ull << G) - 1))) == 0ull;

    ChainForce<T, G, B, false, ASM>::compute(P, g, gbase, (T)centre(step_begin), kr, px, py, pz, fx, fy, fz, nullptr);

    const T h = (T)(0.5 * P.dt);
    const T c1 = (T)P.c1;
    const T hm = (T)(0.5 * P.dt * P.inv_mass);
    const T c2sd = (T)P.c2sd;
    int64_t n_sample = s0 + next_sample_after(P, step_begin - s0);
    for (int64_t n = step_begin + 1; n <= n_end; ++n) {
        if (!alive) break;
        baoab_step<T, G, B, ASM>(P, g, gbase, gid, (uint32_t)n, (T)centre(n), kr, h, hm, c1, c2sd, px, py, pz, vx, vy, vz,
                            fx, fy, fz);
        if (record && n <= 100000) {
#pragma unroll
            for (int b = 0; b < B; ++b)
                if (i0 + b < N) {
                    double *o = traj + (int64_t)n * 3 * N + 3 * (i0 + b);
                    o[0] = (double)px[b]; o[1] = (double)py[b]; o[2] = (double)pz[b];
                }
        }
        if (n == n_sample) {
            n_sample += P.sample_every;
            bool ok = true;
#pragma unroll
            for (int b = 0; b < B; ++b)
                if (i0 + b < N) ok = ok && isfinite((double)px[b]) && isfinite((double)py[b]) && isfinite((double)pz[b]);
            double xi = 0.0;
            if (g == owner) {
#pragma unroll
                for (int b = 0; b < B; ++b)
                    if (i0 + b == last) {
                        const double dx = (double)px[b] - P.fix_x, dy = (double)py[b] - P.fix_y, dz = (double)pz[b] - P.fix_z;
                        xi = P.rc_mode == 1 ? dz : sqrt(dx * dx + dy * dy + dz * dz);
                    }
                ok = ok && isfinite(xi) && fabs(xi) <= P.xi_bound;
            }
            const uint64_t bad = __ballot(!ok);
            const bool grp_bad = ((bad >> gbase) & ((G == 64) ? ~0ull : ((1ull << G) - 1))) != 0ull;
            if (grp_bad) {
                if (g == owner) acc[A_BLOWN] = 1.0;
                alive = false;
            } else if (g == owner) {
                accumulate<E>(P, coef, w, xi, acc, hist, lhist_w, lds.exp);
            }
        }
    }
    if (active) {
#pragma unroll
        for (int b = 0; b < B; ++b) {
            st[0 * NPAD + i0 + b] = px[b]; st[1 * NPAD + i0 + b] = py[b]; st[2 * NPAD + i0 + b] = pz[b];
            st[3 * NPAD + i0 + b] = vx[b]; st[4 * NPAD + i0 + b] = vy[b]; st[5 * NPAD + i0 + b] = vz[b];
        }
        if (g == owner) for (int f = 0; f < A_NFIELDS; ++f) acc_g[f] = acc[f];
    }
}

// Waves per SIMD the compiler schedules the chain kernels for.  The 64x4
// kernel keeps a replica's 16 pair distances and all its lane exchanges of a
// round in flight (about 250 registers): it runs two waves per SIMD whatever
// the schedule, and asked for more the scheduler trades that overlap away and
// the kernel slows by a sixth.  Every other shape keeps the default (8).
template <int G, int B, bool ASM> constexpr int chain_max_waves() { return (G == 64 && B == 4 && !ASM) ? 2 : 8; }

// Least waves per SIMD a direct launch is compiled for.  Left to itself the
// compiler lands the fp32 kernels of chains longer than ten beads a few
// registers above a wave boundary (16x2: 147 VGPRs, three waves; 3x4, 4x4:
// 171-173, two waves).  Asked for one wave more they fit under it (128, 168)
// without spilling and run 5-11% faster, with the same machine arithmetic.  The
// 5x2 kernel keeps the default: the 10-bead workload gives each SIMD fewer than
// two waves, and the tighter budget costs it 4%.  The persistent kernel keeps
// one: its item loop holds the fp64 exponential's constants in registers for the
// whole launch, and at these floors it spills.
template <typename T, int G, int B, bool ASM> constexpr int chain_min_waves() {
    return sizeof(T) != 4 ? 1 : (B == 2 && G >= 8) ? 4 : (ASM || (B == 4 && G >= 3 && G <= 32)) ? 3 : 1;
}

// Direct launch: one work item per workgroup.
template <typename T, int G, int B, bool ASM>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(chain_min_waves<T, G, B, ASM>(), chain_max_waves<G, B, ASM>()))) void sim_chain(const DevProblem *__restrict__ probs, const WorkItem *__restrict__ items,
                                                int n_items, char *__restrict__ ws, int64_t step_begin,
                                                int64_t step_end, double *__restrict__ traj, int64_t traj_rep,
                                                int lds_cap) {
    __shared__ ChainLds<G, ASM> lds;
    extern __shared__ unsigned int s_hist[];
    if ((int)blockIdx.x >= n_items) return;
    const WorkItem item = items[blockIdx.x];
    const DevProblem &P = probs[item.prob];
    const int nk = item_hist_bins(P, item);
    unsigned int *lhist = nk <= lds_cap ? s_hist : nullptr;
    if (lhist) lhist_clear(lhist, nk);
    run_chain_item<T, G, B, ASM, ASM ? EXP_LDS : exp_here<T, G, B>()>(P, item, ws, step_begin, step_end, traj, traj_rep, lds, lhist);
    const int64_t w0 = P.sequential ? seq_window(P, step_begin) : item.window;
    if (lhist) lhist_flush(lhist, nk, reinterpret_cast<unsigned long long *>(ws + P.off_hist) + w0 * P.xi_nbins);
}

// Persistent launch: workgroups take items from a queue (atomic ticket) until
// it is empty; items are ordered longest first by the host.
template <typename T, int G, int B, bool ASM, ExpFrom E>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(1, chain_max_waves<G, B, ASM>()))) void sim_chain_persistent(const DevProblem *__restrict__ probs,
                                                           const WorkItem *__restrict__ items, int n_items,
                                                           int *__restrict__ ticket, char *__restrict__ ws,
                                                           int lds_cap) {
    __shared__ ChainLds<G, ASM> lds;
    __shared__ int s_item;
    extern __shared__ unsigned int s_hist[];
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_item = atomicAdd(ticket, 1);
        __syncthreads();
        const int it = s_item;
        if (it >= n_items) break;
        const WorkItem item = items[it];
        const DevProblem &P = probs[item.prob];
        const int nk = item_hist_bins(P, item);
        unsigned int *lhist = nk <= lds_cap ? s_hist : nullptr;
        if (lhist) lhist_clear(lhist, nk);
        run_chain_item<T, G, B, ASM, E>(P, item, ws, 0, INT64_MAX, nullptr, -1, lds, lhist);
        if (lhist) lhist_flush(lhist, nk, reinterpret_cast<unsigned long long *>(ws + P.off_hist) + (int64_t)item.window * P.xi_nbins);
    }
}

// Energies and forces of configurations (parity hook): one group per configuration,
// with the compiled rounds for every shape (those in assembly form no energies; one
// step of theirs is held against the oracle instead).
// The problem comes with the kernel's arguments: copied to the workspace before every
// launch, with a wait for the copy, it was 19 of a small call's 30 us (256
// configurations of ten beads, 7 us on the GPU; now 11 us).
template <typename T, int G, int B>
__global__ __launch_bounds__(WG) void chain_eval(const DevProblem P, const double *__restrict__ coords,
                                                 int n_rep, double centre, double *__restrict__ forces,
                                                 double *__restrict__ energy) {
    constexpr int GPW = groups_per_wave(G);
    const int lane = lane_id();
    const bool lane_used = lane < GPW * G;
    const int grp = (int)(threadIdx.x >> 6) * GPW + (lane_used ? lane / G : 0);
    const int g = lane_used ? lane % G : 0;
    const int gbase = lane_used ? lane - g : lane;
    const int c = blockIdx.x * chain_reps_per_wg(G) + grp;
    const bool active = lane_used && c < n_rep;
    const int cc = active ? c : 0;
    const int N = P.n_beads;
    const int i0 = g * B;
    T px[B], py[B], pz[B], fx[B], fy[B], fz[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int i = i0 + b;
        if (i < N) { px[b] = (T)coords[(int64_t)cc * 3 * N + 3 * i]; py[b] = (T)coords[(int64_t)cc * 3 * N + 3 * i + 1]; pz[b] = (T)coords[(int64_t)cc * 3 * N + 3 * i + 2]; }
        else { px[b] = 0; py[b] = 0; pz[b] = (T)(P.pad_z0 + P.pad_dz * (i - N)); }
    }
    double e[4];
    ChainForce<T, G, B, true>::compute(P, g, gbase, (T)centre, (T)P.k, px, py, pz, fx, fy, fz, e);
    // group sums of the energy parts (fixed order over lanes)
    double tot[4];
    for (int q = 0; q < 4; ++q) {
        double s = 0.0;
        for (int l = 0; l < G; ++l) s += pull_f(lane_used ? gbase + l : lane, e[q]);
        tot[q] = s;
    }
    if (!active) return;
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const int i = i0 + b;
        if (i < N) {
            forces[(int64_t)c * 3 * N + 3 * i] = (double)fx[b];
            forces[(int64_t)c * 3 * N + 3 * i + 1] = (double)fy[b];
            forces[(int64_t)c * 3 * N + 3 * i + 2] = (double)fz[b];
        }
    }
    if (g == 0) {
        energy[c * 5 + 0] = tot[0] + tot[1] + tot[2] + tot[3];
        for (int q = 0; q < 4; ++q) energy[c * 5 + 1 + q] = tot[q];
    }
}

template <typename T>
__global__ void pot1d_eval(const DevProblem P, const double *__restrict__ coords, int n_rep,
                           double centre, double *__restrict__ forces, double *__restrict__ energy) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n_rep) return;
    const T x = (T)coords[c];
    forces[c] = (double)force_1d<T>(P, x, (T)centre, (T)P.k);
    double ho;
    if (P.pot_kind == 0) { const double q = (double)x * (double)x - P.pot_b; ho = P.pot_a * q * q; }
    else ho = 0.5 * P.pot_kappa * (double)x * (double)x;
    const double res = 0.5 * P.k * ((double)x - centre) * ((double)x - centre);
    energy[c * 5 + 0] = ho + res; energy[c * 5 + 1] = ho; energy[c * 5 + 2] = 0; energy[c * 5 + 3] = 0; energy[c * 5 + 4] = res;
}

// Per-shape launchers; each shape is instantiated in its own translation unit.
// wide: enough work for three waves per SIMD.
template <typename T, int G, int B> auto direct_kernel(bool wide) {
    return wide ? sim_chain<T, G, B, asm_shape<T, G, B>()> : sim_chain<T, G, B, asm_only<T, G, B>()>;
}
template <typename T, int G, int B> auto persistent_kernel(bool wide) {
    constexpr bool ASM = asm_shape<T, G, B>(), ONLY = asm_only<T, G, B>();
    return wide ? sim_chain_persistent<T, G, B, ASM, ASM ? EXP_LDS : EXP_LIBRARY>
                : sim_chain_persistent<T, G, B, ONLY, exp_here<T, G, B>()>;    // 190 registers and more: two waves
}
template <typename T, int G, int B>
hipError_t launch_chain_direct(const DevProblem *d_probs, const WorkItem *d_items, int n_items, char *ws,
                               int64_t step_begin, int64_t step_end, double *traj, int64_t traj_rep, int lds_cap,
                               bool wide, hipStream_t stream) {
    hipLaunchKernelGGL((direct_kernel<T, G, B>(wide)), dim3(n_items), dim3(WG), (size_t)lds_cap * 4, stream, d_probs, d_items,
                       n_items, ws, step_begin, step_end, traj, traj_rep, lds_cap);
    return hipGetLastError();
}
template <typename T, int G, int B>
hipError_t launch_chain_persistent(const DevProblem *d_probs, const WorkItem *d_items, int n_items, int *d_ticket,
                                   char *ws, int n_groups, int lds_cap, bool wide, hipStream_t stream) {
    hipLaunchKernelGGL((persistent_kernel<T, G, B>(wide)), dim3(n_groups), dim3(WG), (size_t)lds_cap * 4, stream,
                       d_probs, d_items, n_items, d_ticket, ws, lds_cap);
    return hipGetLastError();
}
template <typename T, int G, int B>
hipError_t launch_chain_eval(const DevProblem &prob, const double *coords, int n_rep, double centre,
                             double *forces, double *energy, hipStream_t stream) {
    const int per = chain_reps_per_wg(G);
    const int nb = (n_rep + per - 1) / per;
    hipLaunchKernelGGL((chain_eval<T, G, B>), dim3(nb), dim3(WG), 0, stream, prob, coords, n_rep, centre, forces,
                       energy);
    return hipGetLastError();
}
template <typename T, int G, int B>
int chain_blocks_per_cu(int lds_cap, bool wide) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, persistent_kernel<T, G, B>(wide), WG, (size_t)lds_cap * 4) != hipSuccess) n = 1;
    return n;
}

#define PPP_INSTANTIATE_SHAPE(T, G, B)                                                                              \
    template hipError_t launch_chain_direct<T, G, B>(const DevProblem *, const WorkItem *, int, char *, int64_t,   \
                                                     int64_t, double *, int64_t, int, bool, hipStream_t);          \
    template hipError_t launch_chain_persistent<T, G, B>(const DevProblem *, const WorkItem *, int, int *, char *, \
                                                         int, int, bool, hipStream_t);                             \
    template hipError_t launch_chain_eval<T, G, B>(const DevProblem &, const double *, int, double, double *,      \
                                                   double *, hipStream_t);                                         \
    template int chain_blocks_per_cu<T, G, B>(int, bool);

}  // namespace ppp
