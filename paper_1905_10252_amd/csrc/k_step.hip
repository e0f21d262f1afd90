// Sampler kernels of Alg 2 (SMC sampler with recycling), random-walk proposal
// and backward kernel L = q (so the incremental weight is pi(x_t)/pi(x_{t-1}),
// eq. smcs_drawing_weights):
//   k_is<target, init>  particles of one or two coordinates: draws x0 ~ q0 or
//                       x_t = x_{t-1} + rw_sd z, evaluates the target, updates
//                       the log-weights, and leaves per block estimate sums
//                       (against a block reference) and the grid max.
//   k_rows              the same for longer rows, and the
//                       weight update of the logistic regression after its
//                       proposal (k_propose) and likelihood kernels.
//   k_step_stats        estimates f_t (eq. estimation_at_t), c_t
//                       (eq. normconst) and the recycled estimate
//                       (eq. recycling) of a filter iteration (the other
//                       targets': k_decide).
//   k_is<BEARING>       one SIR particle-filter update (Alg 1, Sec. 5.2.2):
//                       constant-velocity transition as proposal, bearing
//                       likelihood as weight.
//   k_filter_step       its redistribution, with the mean of the resampled
//                       population; inside a call of several iterations the
//                       next update too, in the same pass.
//   k_small_step        a whole iteration of a small population.
//   k_logreg_f64 / k_logreg_bf16 + k_logreg_sum
//                       Bayesian logistic regression log-likelihood
//                       sum_m [y_m z_m - softplus(z_m)], z = X theta, in FP64 or
//                       as a BF16 MFMA contraction with FP32 accumulation.
#include <hip/hip_runtime.h>

#include <cmath>

#include "../../include/smc.h"
#include "afun.hpp"
#include "common.hpp"
#include "decide.hpp"
#include "det.hpp"
#include "kernels.hpp"
#include "reduce.hpp"
#include "rng_wave.hpp"
#include "segment.hpp"
#include "stats.hpp"
#include "step.hpp"

namespace smc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct TArgs {
    int kind, d, dp;
    const double *mean, *prec;
    double log_norm, mu, inv_nu, hnu1;
    double init_mean, init_sd, init_prec, init_log_norm, rw_sd;
    uint64_t seed;
    uint32_t sampler;
    unsigned short *thb;  // bf16 copy of the particles times log2 e [npad][dp] (nullable)
    // bearing-only particle filter
    const unsigned *uniform;  // lazy reset flag (NULL: weights always in logw)
    const double *obs;    // measurements, y_t = obs[t - 1]
    double delta, l11, l21, l22, obs_prec, obs_log_norm, reset;
};

__device__ inline unsigned short to_bf16(double v)
{
    const float f = (float)v;
    unsigned u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

__device__ inline double from_bf16(unsigned short h) { return (double)__uint_as_float((unsigned)h << 16); }

// The BF16 likelihood works in base 2: the bf16 particles hold theta log2 e, so
// that the MFMA yields t log2 e and the epilogue's exponentials need no scaling.
constexpr double kLog2e = 1.4426950408889634;
constexpr double kLn2 = 0.6931471805599453;

// ------------------------------------------------------------------ partials
// Estimate sums of k_is (D coordinates), in one pass: each thread keeps
// a reference and sums e = exp(l - ref), so the rows are read once; blocks
// combine the thread references by det_exp rescaling.  The reference is the
// first finite weight and moves (rescaling the sums) only when a weight exceeds
// it by more than kOnlineSlack nats: terms stay below e^64, far from FP64
// overflow, and a lane no longer pays a second exponential at every new
// maximum, which in a wave of 64 lanes happened on most iterations.
constexpr double kOnlineSlack = 64.0;

template <int D>
struct Online {
    double m, e0, e1[D], e2[D];
    __device__ void init()
    {
        m = -__builtin_huge_val();
        e0 = 0.0;
        for (int k = 0; k < D; ++k) e1[k] = e2[k] = 0.0;
    }
    __device__ void sum(double e, const double *xv)
    {
        e0 += e;
#pragma unroll
        for (int k = 0; k < D; ++k) {
            const double ex = e * xv[k];
            e1[k] += ex;
            e2[k] += ex * xv[k];
        }
    }
    __device__ void add(double lw, const double *xv)
    {
        if (!(lw > -__builtin_huge_val())) return;  // zero weight, or NaN (flagged elsewhere)
        if (lw > m + kOnlineSlack) {
            if (m > -__builtin_huge_val()) {
                const double sc = det_exp(m - lw);
                e0 *= sc;
                for (int k = 0; k < D; ++k) {
                    e1[k] *= sc;
                    e2[k] *= sc;
                }
            }
            m = lw;
        }
        sum(det_exp(lw - m), xv);
    }
    // Two particles of one coordinate: their exponentials share the polynomial's
    // coefficients.  A zero weight (or NaN) and a weight that moves the reference
    // take the one-by-one form.
    __device__ void add2(const double (&lw)[2], const double (&xv)[2])
    {
        static_assert(D == 1, "one coordinate a particle");
        const double hi = m + kOnlineSlack;
        if (!(lw[0] > -__builtin_huge_val() && lw[1] > -__builtin_huge_val() && lw[0] <= hi &&
              lw[1] <= hi)) {
            add(lw[0], xv);
            add(lw[1], xv + 1);
            return;
        }
        const double a[2] = {lw[0] - m, lw[1] - m};
        double e[2];
        det_exp_w<2>(a, e);
        sum(e[0], xv);
        sum(e[1], xv + 1);
    }
    // Block combine into the block's partial row (columns at stride gridDim.x).
    __device__ void finish(double *is_part)
    {
        constexpr int C = 1 + 2 * D;
        __shared__ double s_m[4], s_acc[4][C];
        const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
        const double mw = wave_max_f64(m);
        const double sc = m > -__builtin_huge_val() ? det_exp(m - mw) : 0.0;
        double a[C];
        a[0] = wave_sum_f64(e0 * sc);
#pragma unroll
        for (int k = 0; k < D; ++k) {
            a[1 + k] = wave_sum_f64(e1[k] * sc);
            a[1 + D + k] = wave_sum_f64(e2[k] * sc);
        }
        if (lane == 0) {
            s_m[wid] = mw;
            for (int c = 0; c < C; ++c) s_acc[wid][c] = a[c];
        }
        __syncthreads();
        if (tid == 0) {
            double mb = s_m[0];
            for (int w = 1; w < 4; ++w) mb = fmax(mb, s_m[w]);
            double scw[4];
            for (int w = 0; w < 4; ++w)
                scw[w] = s_m[w] > -__builtin_huge_val() ? det_exp(s_m[w] - mb) : 0.0;
            double *part = is_part + blockIdx.x;
            part[0] = mb;
            for (int c = 0; c < C; ++c) {
                double v = 0.0;
                for (int w = 0; w < 4; ++w) v += scw[w] * s_acc[w][c];
                part[(i64)(1 + c) * gridDim.x] = v;
            }
        }
    }
};

// ------------------------------------------------------- proposal + weights
typedef double f64x2s __attribute__((ext_vector_type(2)));
// The update of particles of one or two coordinates (kD; Gaussian and Student-t
// targets, the estimate sums in the same pass) and of the particle filter, which
// takes its estimate after resampling.  k_rows below is the update of longer rows:
// a particle that is one pair leaves it nothing to spread over the lanes, and its
// LDS passes cost more than they save (N = 2^20, two coordinates: 39 us there, 25
// here).
// Where the proposal goes.  kToCopy: to the workspace copy xo; the
// redistribution then maps it into x.  kToBoth: to x, and to xo as well, from
// which a resampling redistribution writes x; an iteration that keeps its
// weights is then done.  The second store costs its bytes in large populations
// (N = 2^24, one coordinate: 205 us an iteration that keeps its weights, 173 with
// one store and no redistribution) and saves a resampling iteration two passes over
// the rows (308 us; 389 with x mapped into a copy and back).  kInPlace: to x alone.
enum Dst { kInPlace, kToCopy, kToBoth };

// The particle filter's transition of one state and its weight.
__device__ inline double bearing_move(const TArgs &a, uint32_t t, const double (&s)[4],
                                      const double (&z)[4], double lw, double *xw)
{
    const double v0 = a.l11 * z[0];
    const double v1 = a.l21 * z[0] + a.l22 * z[1];
    const double v2 = a.l11 * z[2];
    const double v3 = a.l21 * z[2] + a.l22 * z[3];
    const double n0 = (s[0] + a.delta * s[1]) + v0;
    const double n1 = s[1] + v1;
    const double n2 = (s[2] + a.delta * s[3]) + v2;
    const double n3 = s[3] + v3;
    xw[0] = n0;
    xw[1] = n1;
    xw[2] = n2;
    xw[3] = n3;
    const double e = a.obs[t - 1] - det_atan(n2 / n0);
    return lw + (a.obs_log_norm - 0.5 * ((e * e) * a.obs_prec));
}

template <int kKind, bool kInit, Dst kDst, int kD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_is(
    TArgs a, i64 n, uint32_t t, double *__restrict__ x, double *__restrict__ logw,
    double *__restrict__ lp, u64 *slots_p, double *is_part, double *__restrict__ xo,
    double *__restrict__ lpo)
{
    constexpr bool kFilter = kKind == SMC_TARGET_BEARING;
    __shared__ uint4 s_xch[4][64];  // normal generator exchange, one row per wave
    const int tid = threadIdx.x;
    const i64 gtid = (i64)blockIdx.x * 256 + tid, gsz = (i64)gridDim.x * 256;
    const bool uni = !kInit && a.uniform && *a.uniform;  // lazy reset: weights are -ln N
    const uint32_t tag = kInit ? (uint32_t)kTagInit : (uint32_t)kTagPropose;
    const uint32_t tt_ = kInit ? 0u : t;
    u64 key = 0;
    unsigned bad = 0;
    double mx = -__builtin_huge_val();  // largest weight seen
    Online<kD> on;
    on.init();
    // the largest weight, and a flag for NaN or +inf (never on a sound path)
    auto note = [&](double lw) {
        mx = fmax(mx, lw);
        if (!(lw < __builtin_huge_val())) {
            bad = 1u;
            const u64 kk = okey(lw);
            key = kk > key ? kk : key;
        }
    };
    // Log-targets of W 1-D particles of the Gaussian or Student-t target: always
    // the same operations, so a value recomputed from a particle equals the one
    // computed when the particle was proposed, bit for bit.  The
    // previous and new values of a lane's two particles go in together, so
    // the four logarithms share their coefficients.
    auto lpt1 = [&](auto &v, auto &lpv) {
        constexpr int W = sizeof(v) / sizeof(v[0]);
        if (kKind == SMC_TARGET_GAUSS) {
            const double mn = a.mean[0], pr = a.prec[0];
#pragma unroll
            SMC_EACH {
                const double tt = v[w] - mn;
                lpv[w] = a.log_norm - 0.5 * ((tt * tt) * pr);
            }
        } else {
            double u[W], lg[W];
#pragma unroll
            SMC_EACH {
                const double tt = v[w] - a.mu;
                u[w] = 1.0 + (tt * tt) * a.inv_nu;
            }
            det_log_w<W, true>(u, lg);
#pragma unroll
            SMC_EACH lpv[w] = a.log_norm - a.hnu1 * lg[w];
        }
    };
    if constexpr (kD == 2) {
        // Two coordinates: one pair and one row of 16 bytes a particle.
        static_assert(kKind == SMC_TARGET_GAUSS, "the only target of two coordinates here");
        const bool v2 = (((uintptr_t)x | (uintptr_t)xo) & 15) == 0;
        for (i64 base = gtid - (tid & 63); base < n; base += gsz) {
            const i64 i = base + (tid & 63);
            const bool act = i < n;
            const i64 ic = act ? i : n - 1;
            // requested before the normals are drawn, as below
            double xk[2] = {a.init_mean, a.init_mean}, lw_old = a.reset, lp_old = 0.0;
            if (!kInit) {
                if (v2) {
                    const f64x2s v = *reinterpret_cast<const f64x2s *>(x + 2 * ic);
                    xk[0] = v[0];
                    xk[1] = v[1];
                } else {
                    xk[0] = x[2 * ic];
                    xk[1] = x[2 * ic + 1];
                }
                if (!uni) lw_old = logw[ic];
                lp_old = lp[ic];
            }
            asm volatile("" ::: "memory");
            double z[2];
            normal_pair_wave(a.seed, tag, a.sampler, tt_, (uint32_t)i, 0u, act, z[0], z[1],
                             s_xch[tid >> 6]);
            if (!act) continue;
            double acc = 0.0, acc0 = 0.0;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                xk[k] = xk[k] + (kInit ? a.init_sd : a.rw_sd) * z[k];
                const double tt = xk[k] - a.mean[k], t0 = xk[k] - a.init_mean;
                acc = acc + (tt * tt) * a.prec[k];
                acc0 = acc0 + (t0 * t0) * a.init_prec;
            }
            const double lpn = a.log_norm - 0.5 * acc;
            const double lw = kInit ? lpn - (a.init_log_norm - 0.5 * acc0) : lw_old + (lpn - lp_old);
            if (v2) {
                if (kDst != kToCopy)
                    *reinterpret_cast<f64x2s *>(x + 2 * i) = f64x2s{xk[0], xk[1]};
                if (kDst != kInPlace)
                    *reinterpret_cast<f64x2s *>(xo + 2 * i) = f64x2s{xk[0], xk[1]};
            } else {
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    if (kDst != kToCopy) x[2 * i + k] = xk[k];
                    if (kDst != kInPlace) xo[2 * i + k] = xk[k];
                }
            }
            if (kDst != kToCopy) lp[i] = lpn;
            if (kDst != kInPlace) lpo[i] = lpn;
            logw[i] = lw;
            note(lw);
            on.add(lw, xk);
        }
    } else if constexpr (!kFilter) {
        // One coordinate a particle: particles 2p and 2p + 1 take the two
        // values of the pair drawn for index p, so each lane draws one pair
        // for two particles (a wave-uniform trip count over the pairs).  The
        // Gaussian and Student-t targets keep no cached log-target here: the
        // previous one is recomputed from the particle (for the Student-t one
        // more logarithm, against 16 bytes less read and written per particle
        // here and in the redistribution, which then moves 8-byte rows only).
        // The initial pass still writes it, for the one-workgroup iteration
        // that small populations step with.
        const i64 np = (n + 1) >> 1;
        // v2 (n even, 16-byte aligned arrays): a lane moves its two particles' values as one 16-byte access per
        // array, so every wave instruction uses whole cache lines (about 2 %
        // faster per iteration at N = 2^24); otherwise 8-byte accesses
        const uintptr_t al = (uintptr_t)x | (uintptr_t)logw | (uintptr_t)xo;
        const bool v2 = (n & 1) == 0 && (al & 15) == 0;
        for (i64 base = gtid - (tid & 63); base < np; base += gsz) {
            const i64 p = base + (tid & 63);
            const bool pact = p < np;
            // the pair's rows are requested before the normals are drawn, so the
            // loads overlap the generator (the empty asm keeps the compiler from
            // sinking them into their use): about 1 % faster
            double xa0 = 0.0, xa1 = 0.0;
            if (v2) {
                const i64 pc = pact ? p : np - 1;
                if (!kInit) {
                    const f64x2s v = *reinterpret_cast<const f64x2s *>(x + 2 * pc);
                    xa0 = v[0];
                    xa1 = v[1];
                }
            } else if (!kInit) {
                const i64 ic0 = 2 * p < n ? 2 * p : n - 1, ic1 = 2 * p + 1 < n ? 2 * p + 1 : n - 1;
                xa0 = x[ic0];
                xa1 = x[ic1];
            }
            asm volatile("" ::: "memory");
            double z[2];
            normal_pair_wave(a.seed, tag, a.sampler, tt_, (uint32_t)p, 0u, pact, z[0], z[1],
                             s_xch[tid >> 6]);
            if (!pact) continue;
            {
                const bool two = 2 * p + 1 < n;  // false: the lone last particle of an odd n
                double lw[2] = {a.reset, a.reset};
                if (!kInit && !uni) {
                    if (v2) {
                        const f64x2s w = *reinterpret_cast<const f64x2s *>(logw + 2 * p);
                        lw[0] = w[0];
                        lw[1] = w[1];
                    } else {
                        lw[0] = logw[2 * p];
                        if (two) lw[1] = logw[2 * p + 1];
                    }
                }
                const double xh[2] = {xa0, xa1};
                double xk[2], lpn[2];
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    xk[h] = kInit ? a.init_mean + a.init_sd * z[h] : xh[h] + a.rw_sd * z[h];
                if (kInit) {
                    lpt1(xk, lpn);
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const double t0 = xk[h] - a.init_mean;
                        lw[h] = lpn[h] - (a.init_log_norm - 0.5 * ((t0 * t0) * a.init_prec));
                    }
                    // the one-workgroup iteration (N <= 2048) reads the cache
                    lp[2 * p] = lpn[0];
                    if (two) lp[2 * p + 1] = lpn[1];
                } else {
                    const double v4[4] = {xh[0], xh[1], xk[0], xk[1]};
                    double l4[4];
                    lpt1(v4, l4);
#pragma unroll
                    for (int h = 0; h < 2; ++h) lw[h] = lw[h] + (l4[2 + h] - l4[h]);
                }
                if (v2) {
                    if (kDst != kToCopy)
                        *reinterpret_cast<f64x2s *>(x + 2 * p) = f64x2s{xk[0], xk[1]};
                    if (kDst != kInPlace)
                        *reinterpret_cast<f64x2s *>(xo + 2 * p) = f64x2s{xk[0], xk[1]};
                    *reinterpret_cast<f64x2s *>(logw + 2 * p) = f64x2s{lw[0], lw[1]};
                } else {
                    if (kDst != kToCopy) x[2 * p] = xk[0];
                    if (kDst != kInPlace) xo[2 * p] = xk[0];
                    logw[2 * p] = lw[0];
                    if (two) {
                        if (kDst != kToCopy) x[2 * p + 1] = xk[1];
                        if (kDst != kInPlace) xo[2 * p + 1] = xk[1];
                        logw[2 * p + 1] = lw[1];
                    } else {
                        lw[1] = -__builtin_huge_val();  // no particle: weight zero
                    }
                }
                note(lw[0]);
                note(lw[1]);
                on.add2(lw, xk);
            }
        }
    } else {
        // wave-uniform trip count: the normal generator is wave-cooperative
        for (i64 base = gtid - (tid & 63); base < n; base += gsz) {
            const i64 i = base + (tid & 63);
            const bool act = i < n;
            double *xi = x + i * 4;
            double *xw = (kDst == kToCopy ? xo : x) + i * 4;
            // the particle's state and weight are requested before the
            // normals are drawn, so the loads overlap the generator
            const i64 ic = act ? i : 0;
            const double s0 = kInit ? 0.0 : x[ic * 4], s1 = kInit ? 0.0 : x[ic * 4 + 1];
            const double s2 = kInit ? 0.0 : x[ic * 4 + 2], s3 = kInit ? 0.0 : x[ic * 4 + 3];
            const double lw0 = (kInit || uni) ? 0.0 : logw[ic];
            asm volatile("" ::: "memory");
            const uint32_t idx[2] = {(uint32_t)i, (uint32_t)i}, pair[2] = {0u, 1u};
            const bool act2[2] = {act, act};
            double z[4];
            normal_pairs_wave<2>(a.seed, tag, a.sampler, tt_, idx, pair, 2, act2, z,
                                 s_xch[tid >> 6]);
            if (!act) continue;
            double lw;
            if (kInit) {
                for (int k = 0; k < 4; ++k) xi[k] = a.mean[k] + a.init_sd * z[k];
                lw = a.reset;
                lp[i] = 0.0;
            } else {
                const double st[4] = {s0, s1, s2, s3};
                lw = bearing_move(a, t, st, z, uni ? a.reset : lw0, xw);
            }
            logw[i] = lw;
            note(lw);
        }
    }
    key = okey(mx) > key ? okey(mx) : key;
    const u64 bk = block_max_key(key, bad);
    if (!kFilter) on.finish(is_part);
    slot_publish(slots_p, bk, bad);
}

// Between two iterations of the particle filter in one call: the redistribution
// of the one and the update of the next (step t) in one pass over the rows.  Each
// workgroup takes a segment of the merge path; a particle is read from its
// source's row, counted in the mean of the resampled population, moved, weighted
// and written once (kMove false, the last iteration of a call: counted and written
// as it is, with its reset weight).  The population in between is never stored: 64 bytes a
// particle less, and a launch (35.0 us at N = 2^20; redistribution 21.6 us and
// update 25.7 us as kernels of their own).  Vector unit busy 55 % of the time (the
// normals foremost), the waves waiting 37 % of theirs on the segment's phases.  An iteration that kept its weights or found an error moves each
// particle from its own row, as the separate kernels do.
struct FilterArgs {
    i64 n;
    uint32_t t;
    const u64 *pref, *pref64, *tpre;
    const Ctrl *ctrl;
    int tsh;
    const double *x;  // the proposals of the iteration before
    double *xo;       // these
    double *logw;
    u64 *slots_p;
    double *est_part;  // [kEstCols][segments]
    unsigned *uniform; // kMove false: the mark set instead of writing reset weights
};

template <int SEG, bool kMove>
__global__ __launch_bounds__(kExpandThreads) __attribute__((amdgpu_waves_per_eu(4))) void
k_filter_step(TArgs a, FilterArgs g)
{
    constexpr int NW = kExpandThreads / 64;
    union Lds {
        struct {
            SegLds<SEG> seg;
            uint4 xch[NW][64];
        } m;
        double red[8][kExpandThreads];
    };
    __shared__ Lds L;
    __shared__ double s_e[NW];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    AFun f;
    bool failed = false;
    if (!make_afun(g.ctrl, g.pref, g.tpre, g.tsh, g.n, 0, f, false)) {
        failed = true;
        f.mode = 0;
    }
    const Segment sg = segment_cut<SEG>(f, g.pref64, L.m.seg);
    segment_map<SEG>(f, sg, L.m.seg);
    const int np = sg.np;
    const bool kept = f.mode == 0;  // the weights of the iteration before still stand
    const double m = kept && !failed ? g.ctrl->m : a.reset;
    double s1[4] = {0.0, 0.0, 0.0, 0.0}, s2[4] = {0.0, 0.0, 0.0, 0.0}, se = 0.0;
    double mx = -__builtin_huge_val();
    u64 key = 0;
    unsigned bad = 0;
    // wave-uniform trip count; the wavefronts of neighbouring segments start
    // apart, so that the SIMDs share the remainders
    for (int r0 = ((wid + (int)blockIdx.x) & (NW - 1)) * 64; r0 < np; r0 += kExpandThreads) {
        const int r = r0 + lane;
        const bool act = r < np;
        const i64 i = sg.p0 + r;
        const double *xs = g.x + (i64)L.m.seg.anc[act ? r : 0] * 4;
        const double st[4] = {xs[0], xs[1], xs[2], xs[3]};
        double lw = kept && act ? g.logw[i] : a.reset;
        asm volatile("" ::: "memory");
        double z[4];
        if constexpr (kMove) {
            const uint32_t idx[2] = {(uint32_t)i, (uint32_t)i}, pair[2] = {0u, 1u};
            const bool act2[2] = {act, act};
            normal_pairs_wave<2>(a.seed, kTagPropose, a.sampler, g.t, idx, pair, 2, act2, z,
                                 L.m.xch[wid]);
        }
        if (!act) continue;
        const double w = kept && !failed ? det_exp(lw - m) : 1.0;
        se += w;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double wx = w * st[k];
            s1[k] += wx;
            s2[k] += wx * st[k];
        }
        double nx[4] = {st[0], st[1], st[2], st[3]};
        if constexpr (kMove) lw = bearing_move(a, g.t, st, z, lw, nx);
        double *xw = g.xo + i * 4;
        xw[0] = nx[0];
        xw[1] = nx[1];
        xw[2] = nx[2];
        xw[3] = nx[3];
        if constexpr (!kMove) {
            if (!kept && !g.uniform) g.logw[i] = lw;
            continue;
        }
        g.logw[i] = lw;
        mx = fmax(mx, lw);
        if (!(lw < __builtin_huge_val())) {  // NaN or +inf
            bad = 1u;
            const u64 kk = okey(lw);
            key = kk > key ? kk : key;
        }
    }
    key = okey(mx) > key ? okey(mx) : key;
    se = wave_sum_f64(se);
    __syncthreads();  // the map is done with
    if (lane == 0) s_e[wid] = se;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        L.red[k][tid] = s1[k];
        L.red[4 + k][tid] = s2[k];
    }
    u64 bk = 0;
    if constexpr (kMove) bk = block_max_key(key, bad);
    __syncthreads();
    {
        const int c = tid >> 5, l = tid & 31;  // 32 threads a column
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < kExpandThreads / 32; ++k) v += L.red[c][32 * k + l];
        for (int o = 16; o; o >>= 1) v += __shfl_xor(v, o, 64);
        double *out = g.est_part + blockIdx.x;
        if (l == 0) out[(i64)(2 + c) * gridDim.x] = v;
        if (tid == 0) {
            out[0] = failed ? -__builtin_huge_val() : m;
            out[gridDim.x] = (s_e[0] + s_e[1]) + (s_e[2] + s_e[3]);
        }
    }
    if constexpr (kMove) slot_publish(g.slots_p, bk, bad);
    else if (!kept && g.uniform && blockIdx.x == 0 && tid == 0) *g.uniform = 1u;
}

// ------------------------------------------------ rows of several coordinates
// Coordinates c and, if two, c + 1 of a row at dst (vec: 16-byte aligned; the
// workspace copy is aligned wherever x is).
__device__ inline void put_pair(double *dst, bool two, bool vec, double v0, double v1)
{
    if (vec) {
        *reinterpret_cast<f64x2s *>(dst) = f64x2s{v0, v1};
    } else {
        dst[0] = v0;
        if (two) dst[1] = v1;
    }
}

// The proposal (or x0) of particles [base, base + cnt): see draw_rows.
template <bool kInit, int kMaxBlock, class Slot, class Put>
__device__ inline void draw_rows(const TArgs &a, int d, i64 base, int cnt, i64 total, uint32_t t,
                                 const double *x, uint32_t (&queue)[4][kDrawQueue], Slot &&slot,
                                 Put &&put)
{
    draw_rows<kInit, kMaxBlock>(RowDraw{a.seed, a.sampler, kInit ? a.init_mean : 0.0,
                             kInit ? a.init_sd : a.rw_sd},
                     d, base, cnt, total, t, x, (((uintptr_t)x & 15) == 0), queue, slot, put);
}

// Particles of a workgroup of k_rows / k_propose: a power of two with at most
// 24 KB of rows in LDS (six workgroups on a CU), smaller where the population
// would otherwise make fewer than two workgroups per CU.
__host__ __device__ inline int row_stride(int d) { return ((d + 1) | 1); }  // odd, whole pairs
inline int rows_per_block(int64_t n, int d)
{
    const int ds = row_stride(d);
    int P = 256;
    while (P > 32 && P * ds * 8 > 24 * 1024) P >>= 1;
    while (P > 32 && n < 512ll * P) P >>= 1;
    return P;
}

inline int64_t row_chunks(int64_t n, int d)
{
    const int P = rows_per_block(n, d);
    return (n + P - 1) / P;
}

// Proposal of the logistic regression's particles (its log-target comes from
// the likelihood kernels, its weights from k_rows), to x and (xo not NULL) to
// the workspace copy.  With d = 1 particles 2p
// and 2p + 1 take the pair drawn for index p: rows of two values.  65536 particles of
// 32 coordinates: 16 us (46 with the weights' update in one kernel, pairs resolved one
// by one), vector unit busy 37 % of them in a single round of workgroups.
template <bool kInit>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_propose(
    TArgs a, i64 n, uint32_t t, int P, double *__restrict__ x, double *__restrict__ xo)
{
    __shared__ uint32_t s_queue[4][kDrawQueue];
    __shared__ double s_draw[4][kDrawBlock][2];
    const int tid = threadIdx.x;
    const int dv = a.d == 1 ? 2 : a.d;
    const i64 rows = a.d == 1 ? (n + 1) >> 1 : n;
    const i64 base = (i64)blockIdx.x * P;
    if (base >= rows) return;
    const int cnt = (int)(rows - base < P ? rows - base : P);
    draw_rows<kInit, kDrawBlock>(a, dv, base, cnt, n * a.d, t, x, s_queue,
                     [&](int it) { return s_draw[tid >> 6][it % kDrawBlock]; },
                     [&](int p, int c, bool two, bool vec, double v0, double v1) {
                         const i64 o = (base + p) * dv + c;
                         put_pair(x + o, two, vec, v0, v1);
                         if (xo) put_pair(xo + o, two, vec, v0, v1);
                         if (a.thb) {
                             // particle and column of value o (rows of two: one column)
                             const i64 i0 = a.d == 1 ? o : base + p;
                             const int k0 = a.d == 1 ? 0 : c;
                             a.thb[i0 * a.dp + k0] = to_bf16(v0 * kLog2e);
                             if (two)
                                 a.thb[(a.d == 1 ? o + 1 : i0) * a.dp + (a.d == 1 ? 0 : k0 + 1)] =
                                     to_bf16(v1 * kLog2e);
                         }
                     });
}

// What the weight of a logistic-regression particle needs beside its row.
struct LrArgs {
    const double *lpart;  // [msplit][n] partial log-likelihoods
    int msplit;
    const double *csum;   // [d] column sums of X (1 - 2 y)
    double usc, prior_prec;
    int bf16;
};

// log pi of a logistic-regression particle from its row (element k at
// row[k]) and the sum of its partial likelihoods: log_norm - prior_prec
// |theta|^2 / 2 + lik - usc (theta' . csum), theta' the bf16 copy (it holds
// theta log2 e) in that precision and theta otherwise.
__device__ inline double logreg_lp_row(const double *row, int d, double lik, const double *csum,
                                       const LrArgs &lr, double log_norm)
{
    double pr = 0.0, su = 0.0;
    for (int k = 0; k < d; ++k) {
        const double v = row[k];
        pr += v * v;
        su += (lr.bf16 ? from_bf16(to_bf16(v * kLog2e)) : v) * csum[k];
    }
    return log_norm - 0.5 * lr.prior_prec * pr + (lik - lr.usc * su);
}

// The update of particles with d >= 3 coordinates (any d for the logistic
// regression): rows drawn (Gaussian) or read (logistic regression) into LDS by
// the whole workgroup, then one thread per particle for the target and weight,
// then the estimate sums with threads over (column, share of the particles).
// Sums are against the workgroup's reference weight, the first chunk's maximum,
// moved only when a weight exceeds it by kOnlineSlack nats.  Rows are touched
// once in memory; a second pass over the population for the estimates, with
// the exponential formed again for every coordinate, took 30 of 50 us at
// N = 300007, d = 10; one pass takes 28, vector unit busy 44 % and the waves waiting
// 39 % of their time: fewer workgroups than the chip holds at once, so that their
// phases hardly overlap.
template <int kKind, bool kInit, Dst kDst>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_rows(
    TArgs a, i64 n, uint32_t t, int P, double *__restrict__ x, double *__restrict__ logw,
    double *__restrict__ lp, u64 *slots_p, double *is_part, double *__restrict__ xo,
    double *__restrict__ lpo, LrArgs lr)
{
    extern __shared__ double s_dyn[];  // [P][row_stride(d)] rows, [P] exponentials
    __shared__ uint32_t s_queue[4][kDrawQueue];
    __shared__ double s_red[2][256];
    __shared__ double s_par[2][kMaxDim];
    __shared__ double s_w[4];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int d = a.d, ds = row_stride(d);
    double *rows = s_dyn, *s_e = s_dyn + P * ds;
    const bool uni = !kInit && a.uniform && *a.uniform;  // lazy reset: weights are -ln N
    const double ninf = -__builtin_huge_val();
    if (tid < d) {
        s_par[0][tid] = kKind == SMC_TARGET_GAUSS ? a.mean[tid] : lr.csum[tid];
        if (kKind == SMC_TARGET_GAUSS) s_par[1][tid] = a.prec[tid];
    }
    const int parts = 256 / d, part = tid / d, col = tid - part * d;
    const float inv = 1.0f / (float)d;
    u64 key = 0;
    unsigned bad = 0;
    double ref = ninf, e0 = 0.0, s1 = 0.0, s2 = 0.0;
    for (i64 base = (i64)blockIdx.x * P; base < n; base += (i64)gridDim.x * P) {
        const int cnt = (int)(n - base < P ? n - base : P);
        const i64 i = base + tid;
        const bool act = tid < cnt;
        double lw_old = 0.0, lp_old = 0.0, lik = 0.0;
        if (act && !kInit) {
            lw_old = uni ? a.reset : logw[i];
            lp_old = lp[i];
        }
        if (kKind == SMC_TARGET_GAUSS) {
            // the uniforms wait where the row's values will be
            const int np = (d + 1) >> 1;
            const float invp = 1.0f / (float)np;
            draw_rows<kInit, 4096>(a, d, base, cnt, n * d, t, x, s_queue,
                             [&](int it) {
                                 const int p = (int)(((float)it + 0.5f) * invp);
                                 return rows + p * ds + 2 * (it - p * np);
                             },
                             [&](int p, int c, bool two, bool vec, double v0, double v1) {
                                 const i64 o = (base + p) * d + c;
                                 rows[p * ds + c] = v0;
                                 if (two) rows[p * ds + c + 1] = v1;
                                 if (kDst != kToCopy) put_pair(x + o, two, vec, v0, v1);
                                 if (kDst != kInPlace) put_pair(xo + o, two, vec, v0, v1);
                             });
        } else {
            if (act)
                for (int j = 0; j < lr.msplit; ++j) lik += lr.lpart[(i64)j * n + i];
            constexpr int U = 4;
            for (int q0 = tid; q0 < cnt * d; q0 += 256 * U) {
                double v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int q = q0 + 256 * u;
                    v[u] = x[base * d + (q < cnt * d ? q : q0)];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int q = q0 + 256 * u;
                    const int p = (int)(((float)q + 0.5f) * inv);
                    if (q < cnt * d) rows[p * ds + (q - p * d)] = v[u];
                }
            }
        }
        __syncthreads();
        double lw = ninf;
        if (act) {
            const double *row = rows + tid * ds;
            double acc = 0.0, acc0 = 0.0, lpn;
            if (kKind == SMC_TARGET_GAUSS || kInit) {
                for (int k = 0; k < d; ++k) {
                    if (kKind == SMC_TARGET_GAUSS) {
                        const double tt = row[k] - s_par[0][k];
                        acc = acc + (tt * tt) * s_par[1][k];
                    }
                    if (kInit) {
                        const double t0 = row[k] - a.init_mean;
                        acc0 = acc0 + (t0 * t0) * a.init_prec;
                    }
                }
            }
            if (kKind == SMC_TARGET_GAUSS) lpn = a.log_norm - 0.5 * acc;
            else lpn = logreg_lp_row(row, d, lik, s_par[0], lr, a.log_norm);
            lw = kInit ? lpn - (a.init_log_norm - 0.5 * acc0) : lw_old + (lpn - lp_old);
            if (kDst != kToCopy) lp[i] = lpn;
            if (kDst != kInPlace) lpo[i] = lpn;
            logw[i] = lw;
            bad |= !(lw < __builtin_huge_val());  // NaN or +inf
            const u64 kk = okey(lw);
            key = kk > key ? kk : key;
        }
        const double wm = wave_max_f64(lw);
        if (lane == 0) s_w[wid] = wm;
        __syncthreads();
        const double cm = fmax(fmax(s_w[0], s_w[1]), fmax(s_w[2], s_w[3]));
        if (ref == ninf ? cm > ninf : cm > ref + kOnlineSlack) {  // uniform over the workgroup
            const double sc = ref == ninf ? 0.0 : det_exp(ref - cm);
            e0 *= sc;
            s1 *= sc;
            s2 *= sc;
            ref = cm;
        }
        const double e = lw > ninf ? det_exp(lw - ref) : 0.0;
        e0 += e;
        if (act) s_e[tid] = e;
        __syncthreads();
        if (part < parts) {
            for (int p = part; p < cnt; p += parts) {
                const double ep = s_e[p];
                const double xv = ep != 0.0 ? rows[p * ds + col] : 0.0;
                const double ex = ep * xv;
                s1 += ex;
                s2 += ex * xv;
            }
        }
        __syncthreads();  // the next chunk overwrites the rows
    }
    s_red[0][tid] = s1;
    s_red[1][tid] = s2;
    const double we = wave_sum_f64(e0);
    if (lane == 0) s_w[wid] = we;
    __syncthreads();
    double *out = is_part + blockIdx.x;
    if (tid < 2 * d) {
        const double *red = tid < d ? s_red[0] + tid : s_red[1] + (tid - d);
        double v = 0.0;
        for (int q = 0; q < parts; ++q) v += red[q * d];
        out[(i64)(2 + tid) * gridDim.x] = v;
    }
    if (tid == 0) {
        out[0] = ref;
        out[gridDim.x] = ((s_w[0] + s_w[1]) + s_w[2]) + s_w[3];
    }
    const u64 bk = block_max_key(key, bad);
    slot_publish(slots_p, bk, bad);
}

// -------------------------------------------- estimates, c_t and recycling
// One workgroup: the statistics of a filter iteration ...
__global__ __launch_bounds__(1024) void k_step_stats(Ctrl *ctrl, const double *is_part, int nblk,
                                                     int d, double *rec_num, double *est,
                                                     smc_resample_info *info)
{
    filter_stats<1024>(ctrl, is_part, nblk, d, rec_num, est, info);
}

// ... and of an initialisation: log sum w_0, cleared recycling sums.
__global__ __launch_bounds__(1024) void k_init_stats(Ctrl *ctrl, const double *is_part, int nblk,
                                                     int d, double *rec_num)
{
    __shared__ StatsLds s_st;
    const int tid = threadIdx.x;
    StepStats<1024> ss;
    ss.begin(s_st, is_part, nblk);
    __syncthreads();
    const double m = ss.scale(s_st, nblk);
    __syncthreads();
    const double z = tid < 64 ? ss.column(s_st, is_part, nblk, 1) : 0.0;
    if (tid == 0) {
        ctrl->logZ_prev = m + log(z);
        ctrl->lc_max = -__builtin_huge_val();
        ctrl->rec_den = 0.0;
        ctrl->rec_steps = 0;
    }
    if (tid < 2 * d) rec_num[tid] = 0.0;
}

// The filter's row sums of more than kIsBlocks expand workgroups, gathered
// into kFoldBlocks rows (workgroup b adds segments b, b + kFoldBlocks, ... of
// each column, in that order; all of them carry the same reference).
constexpr int kFoldBlocks = 256;

__global__ __launch_bounds__(64) void k_fold_rows(const double *epart, i64 nseg, double *is_part)
{
    const int c = threadIdx.x;
    if (c >= kEstCols) return;
    const double *col = epart + c * nseg;
    double v = 0.0;
    if (c == 0) v = col[blockIdx.x];
    else
        for (i64 g = blockIdx.x; g < nseg; g += kFoldBlocks) v += col[g];
    is_part[c * kFoldBlocks + blockIdx.x] = v;
}

// Weighted sums of the initial population, one partial row per block with one
// common reference weight.
template <int DT>
__global__ __launch_bounds__(256) void k_post_est(const Ctrl *ctrl, i64 n, int d,
                                                  const double *__restrict__ x,
                                                  const double *__restrict__ logw,
                                                  double *is_part)
{
    __shared__ double s_acc[4][1 + 2 * DT];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const i64 gtid = (i64)blockIdx.x * 256 + tid, gsz = (i64)gridDim.x * 256;
    const double m = ctrl->m;
    double e0 = 0.0, e1[DT], e2[DT];
    for (int k = 0; k < DT; ++k) e1[k] = e2[k] = 0.0;
    for (i64 i = gtid; i < n; i += gsz) {
        const double e = det_exp(logw[i] - m);
        e0 += e;
        for (int k = 0; k < DT; ++k) {
            const double xk = x[i * DT + k];
            const double ex = e * xk;
            e1[k] += ex;
            e2[k] += ex * xk;
        }
    }
    e0 = wave_sum_f64(e0);
    for (int k = 0; k < DT; ++k) {
        e1[k] = wave_sum_f64(e1[k]);
        e2[k] = wave_sum_f64(e2[k]);
    }
    if (lane == 0) {
        s_acc[wid][0] = e0;
        for (int k = 0; k < DT; ++k) {
            s_acc[wid][1 + k] = e1[k];
            s_acc[wid][1 + DT + k] = e2[k];
        }
    }
    __syncthreads();
    double *part = is_part + blockIdx.x;
    for (int c = tid; c < 2 + 2 * DT; c += 256)
        part[(i64)c * gridDim.x] = c == 0 ? m : ((s_acc[0][c - 1] + s_acc[1][c - 1]) + s_acc[2][c - 1]) +
                                   s_acc[3][c - 1];
}


// ------------------------------------------------- small-N fused iteration
// One workgroup runs a whole iteration of Alg 2 for at most kSmallN particles
// of a cheap target with up to kSmallD coordinates, two consecutive particles
// a thread and only as many wavefronts as that takes: proposal and weights;
// after a barrier the fixed-point weights, their prefix and every sum; after
// another the integer decision, c_t and recycling, which every thread forms
// for itself from the wavefronts' totals; when it resamples, the sources mark
// their first outputs in LDS and a max-scan over the outputs carries the marks
// (two more barriers; a binary search per output took eleven dependent LDS
// reads).  Rows wait in LDS, and each particle is stored once.  Same arithmetic
// per particle and same integers as the multi-kernel path; only the order of
// the FP64 sums differs.  It keeps the control block as the multi-kernel path
// does and clears the other parity's max slots.  Bound by latency: 7.2 us a
// call at N = 1024 with one coordinate (1024 threads whatever N, a search per
// output and six barriers: 10.1).
constexpr int kSmallN = 2048, kSmallD = 8;
constexpr int kSmallPairs = 3072;  // most (particle, pair) items
constexpr int kSmallRows = 2 * kSmallPairs;  // row values in LDS

template <int kKind, int kDim, int kMaxN>  // kDim: largest d (1, 4 or 8)
__global__ __launch_bounds__(kMaxN / 2) void k_small_step(TArgs a, i64 n, uint32_t t, int K, int mode,
                                                        int ess_num, int ess_den,
                                                        double *__restrict__ x,
                                                        double *__restrict__ logw,
                                                        double *__restrict__ lp, Ctrl *ctrl,
                                                        u64 *slots_other, double *rec_num,
                                                        smc_resample_info *info, double *est,
                                                        double reset)
{
    constexpr int NW = kMaxN / 128, DM = kDim;
    constexpr bool kD1 = kDim == 1;
    __shared__ double s_x[kD1 ? kMaxN : kSmallRows], s_lp[kMaxN];
    __shared__ unsigned s_mark[kMaxN];
    __shared__ uint4 s_xch[NW][64];
    __shared__ double s_col[2 * DM][NW], s_z[NW], s_z2[NW];
    __shared__ u64 s_key[NW], s_wsum[NW], s_lo[NW], s_hi[NW];
    __shared__ unsigned s_bad[NW], s_wmax[NW];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, nw = blockDim.x >> 6;
    const int d = kD1 ? 1 : a.d, ni = (int)n, i0 = 2 * tid;
    const double ninf = -__builtin_huge_val();
    const bool act[2] = {i0 < ni, i0 + 1 < ni};
    const RecState rec(ctrl);
    const double rec_old = tid < 2 * d ? rec_num[tid] : 0.0;
    const u64 r = resample_word(a.seed, a.sampler, t);

    // the thread's particles, requested before the normals are drawn
    double xr[2][DM], lw[2], lp_old[2], lpn[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int i = act[j] ? i0 + j : 0;
#pragma unroll
        for (int k = 0; k < DM; ++k) xr[j][k] = k < d ? x[i * d + k] : 0.0;
        lw[j] = logw[i];
        lp_old[j] = lp[i];
    }
    for (int k = tid; k < kSlots * kSlotStride; k += blockDim.x) slots_other[k] = 0;
    s_mark[i0] = 0u;
    s_mark[i0 + 1] = 0u;
    asm volatile("" ::: "memory");
    if constexpr (kD1) {
        double z[2];
        normal_pair_wave(a.seed, kTagPropose, a.sampler, t, (uint32_t)tid, 0u, act[0], z[0], z[1],
                         s_xch[wid]);
        xr[0][0] = xr[0][0] + a.rw_sd * z[0];
        xr[1][0] = xr[1][0] + a.rw_sd * z[1];
    } else {
        for (int q = 0; 2 * q < d; ++q) {
            const uint32_t idx[2] = {(uint32_t)i0, (uint32_t)(i0 + 1)};
            const uint32_t pair[2] = {(uint32_t)q, (uint32_t)q};
            double z[4];
            normal_pairs_wave<2>(a.seed, kTagPropose, a.sampler, t, idx, pair, 2, act, z,
                                 s_xch[wid]);
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int k = 0; k < DM; ++k)
                    if (k >> 1 == q && k < d) xr[j][k] = xr[j][k] + a.rw_sd * z[2 * j + (k & 1)];
        }
    }
    if (kKind == SMC_TARGET_GAUSS) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            double acc = 0.0;
#pragma unroll
            for (int k = 0; k < DM; ++k)
                if (k < d) {
                    const double tt = xr[j][k] - a.mean[k];
                    acc = acc + (tt * tt) * a.prec[k];
                }
            lpn[j] = a.log_norm - 0.5 * acc;
        }
    } else {
        double u[2], lg[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const double tt = xr[j][0] - a.mu;
            u[j] = 1.0 + (tt * tt) * a.inv_nu;
        }
        det_log_w<2, true>(u, lg);
#pragma unroll
        for (int j = 0; j < 2; ++j) lpn[j] = a.log_norm - a.hnu1 * lg[j];
    }
    u64 key = 0;
    unsigned bad = 0;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        lw[j] = act[j] ? lw[j] + (lpn[j] - lp_old[j]) : ninf;
        bad |= !(lw[j] < __builtin_huge_val());  // NaN or +inf
        const u64 kk = okey(lw[j]);
        key = kk > key ? kk : key;
    }
    key = wave_max_u64(key);
    bad = wave_or(bad);
    if (lane == 0) {
        s_key[wid] = key;
        s_bad[wid] = bad;
    }
    __syncthreads();
    key = wave_max_u64(lane < nw ? s_key[lane & (NW - 1)] : 0ull);
    bad = wave_or(lane < nw ? s_bad[lane & (NW - 1)] : 0u);
    const double m = okey_inv(key);

    // fixed-point weights, their prefix, the FP64 sums, the estimate sums
    const double v[2] = {lw[0], lw[1]};
    double z = 0.0, z2 = 0.0, e[2];
    SqSum sq;
    u64 q[2];
    quant_w<2>(v, m, K, q, z, z2, sq, e);
    const u64 run = q[0] + q[1], incl = wave_incl_scan_u64(run);
    z = wave_sum_f64(z);
    z2 = wave_sum_f64(z2);
    const U128 q2 = wave_sum_u128(sq.total());
    double c1[DM], c2[DM];
#pragma unroll
    for (int k = 0; k < DM; ++k) {
        c1[k] = c2[k] = 0.0;
        if (k >= d) continue;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const double ex = act[j] ? e[j] * xr[j][k] : 0.0;
            c1[k] += ex;
            c2[k] += ex * xr[j][k];
        }
        c1[k] = wave_sum_f64(c1[k]);
        c2[k] = wave_sum_f64(c2[k]);
    }
    if (lane == 63) s_wsum[wid] = incl;
    if (lane == 0) {
        s_z[wid] = z;
        s_z2[wid] = z2;
        s_lo[wid] = q2.lo;
        s_hi[wid] = q2.hi;
#pragma unroll
        for (int k = 0; k < DM; ++k)
            if (k < d) {
                s_col[k][wid] = c1[k];
                s_col[d + k][wid] = c2[k];
            }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
        if (act[j]) {
#pragma unroll
            for (int k = 0; k < DM; ++k)
                if (k < d) s_x[(i0 + j) * d + k] = xr[j][k];
            s_lp[i0 + j] = lpn[j];
        }
    __syncthreads();

    // decision, c_t and recycling, by every thread from the wavefronts' totals
    const bool in = lane < nw;
    const u64 wincl = wave_incl_scan_u64(in ? s_wsum[lane & (NW - 1)] : 0ull);
    const u64 S = lane63_u64(wincl);
    const u64 wpre = wid ? (u64)__shfl((long long)wincl, wid - 1, 64) : 0ull;
    const double Z = wave_sum_f64(in ? s_z[lane & (NW - 1)] : 0.0);
    const double Z2 = wave_sum_f64(in ? s_z2[lane & (NW - 1)] : 0.0);
    const U128 Q2 =
        wave_sum_u128(in ? U128{s_lo[lane & (NW - 1)], s_hi[lane & (NW - 1)]} : U128{0, 0});
    const Decision dec = decide(key, bad, S, Z, Z2, Q2, n, r, mode, ess_num, ess_den);
    if (wid == 0) {  // 2 d <= 16 estimate threads, all in the first wavefront
        double bc[3] = {1.0, 0.0, 0.0}, logc = 0.0;
        RecNext nx;
        if (!dec.err) logc = recycle_step(rec, dec.logZ, bc, nx);
        if (tid == 0) {
            store_decision(dec, K, logc, ctrl, info);
            ctrl->pending = 0;
            if (!dec.err) store_recycling(nx, logc, dec.logZ, dec.resample, ctrl);
        }
        if (tid < 2 * d && !dec.err) {
            double tot = 0.0;
            for (int w = 0; w < nw; ++w) tot += s_col[tid][w];
            const double f = tot / Z;
            const double num = rec_old * bc[0] + bc[1] * f;
            rec_num[tid] = num;
            if (est) {
                est[tid] = f;
                est[2 * d + tid] = num / bc[2];
            }
        }
    }
    if (!dec.resample) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (act[j]) {
#pragma unroll
                for (int k = 0; k < DM; ++k)
                    if (k < d) x[(i0 + j) * d + k] = xr[j][k];
                lp[i0 + j] = lpn[j];
                logw[i0 + j] = lw[j];
            }
        return;
    }

    // redistribution: source j's copies start at output A_{j-1}
    AFun f;
    f.n = n;
    f.set_systematic(S, dec.U);
    const u64 pre = wpre + incl - run;
    unsigned a0 = i0 > 0 ? f.A_of(0, pre) : 0u;
    u64 sj = pre;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (!act[j]) break;
        sj += q[j];
        const unsigned a1 = f.A_of(0, sj);
        if (a1 > a0) s_mark[a0] = (unsigned)(i0 + j + 1);
        a0 = a1;
    }
    __syncthreads();
    unsigned mk[2] = {s_mark[i0], s_mark[i0 + 1]};
    mk[1] = mk[1] > mk[0] ? mk[1] : mk[0];
    const unsigned minc = wave_scan_max_u32(mk[1]);
    if (lane == 63) s_wmax[wid] = minc;
    unsigned carry = (unsigned)__shfl_up((int)minc, 1, 64);
    carry = lane ? carry : 0u;
    __syncthreads();
    for (int w = 0; w < wid; ++w) carry = s_wmax[w] > carry ? s_wmax[w] : carry;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (!act[j]) continue;
        const int src = (int)(mk[j] > carry ? mk[j] : carry) - 1;
#pragma unroll
        for (int k = 0; k < DM; ++k)
            if (k < d) x[(i0 + j) * d + k] = s_x[src * d + k];
        lp[i0 + j] = s_lp[src];
        logw[i0 + j] = reset;
    }
}

// ------------------------------------------------------ cheap log-targets
__global__ __launch_bounds__(256) void k_lp_cheap(TArgs a, i64 n, const double *x, double *lp)
{
    const i64 gtid = (i64)blockIdx.x * 256 + threadIdx.x, gsz = (i64)gridDim.x * 256;
    for (i64 i = gtid; i < n; i += gsz) {
        const double *xi = x + i * a.d;
        if (a.kind == SMC_TARGET_GAUSS) {
            double acc = 0.0;
            for (int k = 0; k < a.d; ++k) {
                const double tt = xi[k] - a.mean[k];
                acc = acc + (tt * tt) * a.prec[k];
            }
            lp[i] = a.log_norm - 0.5 * acc;
        } else {
            const double tt = xi[0] - a.mu;
            lp[i] = a.log_norm - a.hnu1 * det_log(1.0 + (tt * tt) * a.inv_nu);
        }
    }
}

// --------------------------------------------- logistic regression, FP64
// With s_m = 1 - 2 y_m and u = s_m z_m, y_m z_m - softplus(z_m) = -softplus(u),
// and softplus(u) = (u + |u|) / 2 + log1p(e^(-|u|)).  The kernel sums |u| and
// the logs of products of 512 factors 1 + e^(-|u|) in (1, 2];
// the sum of u over all rows, theta . (sum_m s_m x_m), is added once per
// particle by k_logreg_sum.
//
// u = (X s) theta runs on v_mfma_f64_16x16x4_f64, so the matrix unit takes the
// contraction while the vector ALU runs the exponentials.  One wavefront owns
// 16 particles (MFMA columns) and streams 16-row tiles of X s (MFMA rows) from
// xf, where each tile is stored in the order the MFMA A operand is read:
// xf[tile][lane][s] = s_m x_{m,k}, m = 16 tile + lane % 16, k = 4 s + lane / 16
// (zero beyond M and d), so a lane's KS values are contiguous and a tile is
// one contiguous 512 KS-byte read per wavefront.  The epilogue relies only on
// each lane's accumulators belonging to column lane % 16: it sums a column's
// rows whatever their order across lanes.
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2v __attribute__((ext_vector_type(2)));

// The FP64 matrix and vector instructions share one pipe on this chip: the
// 8 MFMAs of a D = 32 tile (512 cycles a SIMD) and its 4 x 22 vector
// instructions took 981 cycles together, so the epilogue counts in full.  Its
// exponential: with a = |u| <= 700 and k = rint(a 2048 / ln 2),
// e^-a = 2^(-k / 2048) e^-r, |r| <= ln 2 / 4096, the first factor from a table of
// 2048 values (exact to 0.5 ulp, in LDS) and an exponent shift in 32-bit
// arithmetic, the second 1 - r + r^2 / 2 - r^3 / 6 with the r^4 term folded into
// r^2 (off by at most 8.6e-18; the constant enters as 1 + e^-a, whose rounding
// is 1.1e-16).  Nine FP64 instructions an element instead of nineteen.  The
// clamp of a (in its high word: infinities and NaN too) keeps the exponent in
// range; e^-700 adds nothing to 1.
constexpr int kExpBits = 11, kExpN = 1 << kExpBits;
static_assert(kExpN == kExpTabN, "table size");

__device__ inline void softplus_acc64(double u, const double *tab, double &sa, double &prod)
{
    const double magic = 0x1.8p52;  // its last place is 1: adding it rounds to an integer
    const unsigned uh = (unsigned)__double2hiint(u) & 0x7FFFFFFFu;
    const double ac = __hiloint2double((int)(uh < 0x4085E000u ? uh : 0x4085E000u),
                                       __double2loint(u));
    const double kd = fma(ac, 0x1.71547652b82fep+11, magic);
    const int k = __double2loint(kd);
    const double r = fma(kd - magic, -0x1.62e42fefa39efp-12, ac);
    const double t0 = tab[k & (kExpN - 1)];
    const double t = __hiloint2double(
        __double2hiint(t0) - (int)(((unsigned)k << (20 - kExpBits)) & 0xFFF00000u),
        __double2loint(t0));
    const double q = fma(fma(r, -0x1.5555555555555p-3, 0x1.0000000a3fea0p-1), r, -1.0) * r;
    prod = fma(prod, fma(t, q, t), prod);
    sa += fabs(u);
}

// The table of 2^(-j / 2048): products of double-double powers, rounded once.
__device__ inline void two_prod(double a, double b, double &p, double &e)
{
    p = a * b;
    e = fma(a, b, -p);
}

__global__ __launch_bounds__(256) void k_exp_table(double *tab)
{
    const double pw[kExpBits][2] = {
        {0x1.ffd3a565efb65p-1, -0x1.54441c5aeb90fp-57},  // 2^(-1/2048)
        {0x1.ffa74ea381efcp-1, 0x1.0bd3b9f8ae013p-56},   // 2^(-2/2048)
        {0x1.ff4eaca4391b6p-1, -0x1.2e60c5e4b7047p-56},
        {0x1.fe9d96b2a23d9p-1, 0x1.4a6037442fde3p-57},
        {0x1.fd3c22b8f71f1p-1, 0x1.2eb74966579e7p-58},
        {0x1.fa7c1819e90d8p-1, 0x1.74853f3a5931ep-56},
        {0x1.f50765b6e4540p-1, 0x1.9d3e12dd8a18bp-55},
        {0x1.ea4afa2a490dap-1, -0x1.e9c23179c2893p-55},
        {0x1.d5818dcfba487p-1, 0x1.2ed02d75b3707p-56},
        {0x1.ae89f995ad3adp-1, 0x1.7a1cd345dcc81p-55},
        {0x1.6a09e667f3bcdp-1, -0x1.bdd3413b26456p-55},  // 2^(-1024/2048)
    };
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= kExpN) return;
    double hi = 1.0, lo = 0.0;
#pragma unroll
    for (int i = 0; i < kExpBits; ++i) {
        if (!((j >> i) & 1)) continue;
        double p, e;
        two_prod(hi, pw[i][0], p, e);
        e += hi * pw[i][1] + lo * pw[i][0];
        hi = p + e;
        lo = e - (hi - p);
    }
    tab[j] = hi;
}

template <int KS>
__global__ __launch_bounds__(256) void k_logreg_f64(const double *__restrict__ theta, i64 n, int d,
                                                    const double *__restrict__ xf,
                                                    const double *__restrict__ etab, i64 m_rows,
                                                    i64 mpad, double *__restrict__ lpart)
{
    __shared__ double s_tab[kExpN];
#pragma unroll
    for (int i = 0; i < kExpN / 512; ++i)
        reinterpret_cast<f64x2v *>(s_tab)[256 * i + threadIdx.x] =
            reinterpret_cast<const f64x2v *>(etab)[256 * i + threadIdx.x];
    __syncthreads();
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const i64 p0 = ((i64)blockIdx.x * 4 + wid) * 16;
    if (p0 >= n) return;
    const int col = lane & 15, kq = lane >> 4;
    const i64 p = p0 + col;
    double b[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int k = 4 * s + kq;
        b[s] = (p < n && k < d) ? theta[p * d + k] : 0.0;
    }
    const i64 tiles = mpad / 16;
    const i64 per = (tiles + gridDim.y - 1) / gridDim.y;
    const i64 t0 = (i64)blockIdx.y * per;
    const i64 t1 = t0 + per < tiles ? t0 + per : tiles;
    double sa = 0.0, lg = 0.0, prod = 1.0;
    int cnt = 0;
    auto contract = [&](i64 tt) {
        const double *ap = xf + (tt * 64 + lane) * KS;
        double a[KS];
        if constexpr (KS == 1) {
            a[0] = ap[0];
        } else {
#pragma unroll
            for (int s = 0; s < KS; s += 2) {
                const f64x2v v = *reinterpret_cast<const f64x2v *>(ap + s);
                a[s] = v[0];
                a[s + 1] = v[1];
            }
        }
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < KS; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], acc, 0, 0, 0);
        return acc;
    };
    const i64 whole = m_rows / 16 < t1 ? m_rows / 16 : t1;
    for (i64 tt = t0; tt < whole; ++tt) {
        const f64x4 acc = contract(tt);
#pragma unroll
        for (int v = 0; v < 4; ++v) softplus_acc64(acc[v], s_tab, sa, prod);
        if (++cnt == 128) {  // 512 factors in (1, 2]: at most 2^512
            lg += log(prod);
            prod = 1.0;
            cnt = 0;
        }
    }
    // A last tile with rows beyond M: those add nothing.  The row of each
    // accumulator comes from a product of its own (row index times one).
    if (t0 <= whole && whole < t1 && m_rows > whole * 16) {
        const f64x4 acc = contract(whole);
        const double ri = kq == 0 ? (double)col : 0.0, one = kq == 0 ? 1.0 : 0.0;
        f64x4 row = {0.0, 0.0, 0.0, 0.0};
        row = __builtin_amdgcn_mfma_f64_16x16x4f64(ri, one, row, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (whole * 16 + (i64)row[v] < m_rows) softplus_acc64(acc[v], s_tab, sa, prod);
    }
    double sp = 0.5 * sa + (lg + log(prod));
    sp += __shfl_xor(sp, 16, kWave);
    sp += __shfl_xor(sp, 32, kWave);
    if (lane < 16 && p < n) lpart[(i64)blockIdx.y * n + p] = -sp;
}

// xf (above) from the caller's X and y.
__global__ __launch_bounds__(256) void k_prep_xf(const double *X, const double *y, i64 m_rows,
                                                 int d, i64 mpad, int ks, double *xf)
{
    const i64 gtid = (i64)blockIdx.x * 256 + threadIdx.x, gsz = (i64)gridDim.x * 256;
    const i64 per_tile = 64 * (i64)ks;
    for (i64 e = gtid; e < mpad * 4 * ks; e += gsz) {
        const i64 t = e / per_tile;
        const int rem = (int)(e - t * per_tile);
        const int lane = rem / ks, sidx = rem - lane * ks;
        const i64 m = 16 * t + (lane & 15);
        const int k = 4 * sidx + (lane >> 4);
        double v = 0.0;
        if (m < m_rows && k < d) {
            v = X[m * d + k];
            if (y[m] != 0.0) v = -v;
        }
        xf[e] = v;
    }
}

// Column sums of X s (rows below m_rows), one workgroup per column, FP64 in
// a fixed order.
__global__ __launch_bounds__(256) void k_x_colsum(const double *X, const double *y, i64 m_rows,
                                                  int d, double *csum)
{
    __shared__ double red[4];
    const int k = blockIdx.x, tid = threadIdx.x;
    double v = 0.0;
    for (i64 m = tid; m < m_rows; m += 256) {
        const double xv = X[m * d + k];
        v += y[m] != 0.0 ? -xv : xv;
    }
    v = wave_sum_f64(v);
    if ((tid & 63) == 0) red[tid >> 6] = v;
    __syncthreads();
    if (tid == 0) csum[k] = (red[0] + red[1]) + (red[2] + red[3]);
}

// ------------------------------------ logistic regression, BF16 MFMA (gfx950)
// X is stored pre-multiplied by s_m = 1 - 2 y_m (exact in bf16), so that
// y_m z_m - softplus(z_m) = -softplus(s_m z_m) and the epilogue needs no labels.
// One wavefront owns 32 particles (MFMA columns) and streams 32-row tiles of X
// (MFMA rows) through v_mfma_f32_32x32x16_bf16; the softplus epilogue runs on
// the FP32 accumulators, which hold u = t log2 e for t = s_m z_m.
// softplus(t) = ln 2 [(u + |u|) / 2 + log2(1 + 2^(-|u|))].  A lane's 16
// accumulator values of one tile each give a factor 1 + 2^(-|u|) in (1, 2];
// their product (at most 2^16) takes one log2 per tile.  The kernel sums |u|
// and the log2 terms; the sum of u over all rows is theta . (sum_m x_m s_m)
// log2 e, added once per particle by k_logreg_sum from the column sums of X.
//
// X s is stored in the order the MFMA A operand is read: tile of 32 rows, k-step of
// 16, lane (row % 32 of its low half of eight columns, then of the high half), eight
// columns.  A wavefront's read is one contiguous kilobyte; from rows of 128 bytes
// (D > 48) each read touched 32 lines and the loop waited on the address unit:
// 65536 particles, 32768 rows, D = 64: 1018 us an iteration by rows, 498 now.
__device__ inline i64 xs_at(i64 m, int k, int dp)
{
    const i64 step = (m >> 5) * (dp >> 4) + (k >> 4);
    return (step * 64 + ((k >> 3) & 1) * 32 + (m & 31)) * 8 + (k & 7);
}

__device__ inline void softplus_acc(float u, float &sa, float &prod)
{
    const float e = __builtin_amdgcn_exp2f(-fabsf(u));
    prod = fmaf(prod, e, prod);
    sa += fabsf(u);
}

template <int KS>
__global__ __launch_bounds__(256) void k_logreg_bf16(const unsigned short *__restrict__ thb, i64 n,
                                                     const unsigned short *__restrict__ xs,
                                                     i64 m_rows, i64 mpad, int dp,
                                                     double *__restrict__ lpart)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const i64 p0 = ((i64)blockIdx.x * 4 + wid) * 32;
    if (p0 >= n) return;
    const int col = lane & 31, kh = lane >> 5;
    bf16x8 bfr[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s)
        bfr[s] = *reinterpret_cast<const bf16x8 *>(thb + (p0 + col) * dp + 16 * s + 8 * kh);
    const i64 tiles = mpad / 32;
    const i64 per = (tiles + gridDim.y - 1) / gridDim.y;
    const i64 t0 = (i64)blockIdx.y * per;
    const i64 t1 = t0 + per < tiles ? t0 + per : tiles;
    float sa = 0.0f, lg = 0.0f;
    // the next tile's rows are requested before this one's are used (4001 particles, 9973
    // rows, one wave a SIMD: 15.4 us without, 13.3 with)
    const bf16x8 *xr = reinterpret_cast<const bf16x8 *>(xs) + t0 * (64 * KS) + lane;
    bf16x8 nx[KS];
    if (t0 < t1)
#pragma unroll
        for (int s = 0; s < KS; ++s) nx[s] = xr[64 * s];
    for (i64 tt = t0; tt < t1; ++tt) {
        const i64 m0 = tt * 32;
        bf16x8 afr[KS];
        if (tt + 1 < t1) xr += 64 * KS;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            afr[s] = nx[s];
            nx[s] = xr[64 * s];
        }
        asm volatile("" ::: "memory");
        f32x16 acc = {};
#pragma unroll
        for (int s = 0; s < KS; ++s)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afr[s], bfr[s], acc, 0, 0, 0);
        float prod = 1.0f;
        if (m0 + 32 <= m_rows) {
#pragma unroll
            for (int r = 0; r < 16; ++r) softplus_acc(acc[r], sa, prod);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const i64 row = m0 + 8 * (r >> 2) + 4 * kh + (r & 3);
                if (row < m_rows) softplus_acc(acc[r], sa, prod);
            }
        }
        lg += __builtin_amdgcn_logf(prod);
    }
    float sp = 0.5f * sa + lg;
    sp += __shfl_xor(sp, 32, kWave);
    if (lane < 32 && p0 + lane < n) lpart[(i64)blockIdx.y * n + p0 + lane] = -kLn2 * (double)sp;
}

// Column sums of the stored bf16 X s (rows below m_rows; padding is zero), one
// workgroup per column, FP64 in a fixed order.
__global__ __launch_bounds__(256) void k_xs_colsum(const unsigned short *xs, i64 m_rows, int dp,
                                                   double *csum)
{
    __shared__ double red[4];
    const int k = blockIdx.x, tid = threadIdx.x;
    double v = 0.0;
    for (i64 m = tid; m < m_rows; m += 256) v += from_bf16(xs[xs_at(m, k, dp)]);
    v = wave_sum_f64(v);
    if ((tid & 63) == 0) red[tid >> 6] = v;
    __syncthreads();
    if (tid == 0) csum[k] = (red[0] + red[1]) + (red[2] + red[3]);
}

// log pi at caller points (smc_log_target) from the partial likelihoods.
__global__ __launch_bounds__(256) void k_logreg_sum(const double *theta, i64 n, int d, LrArgs lr,
                                                    double log_norm, double *lp)
{
    const i64 gtid = (i64)blockIdx.x * 256 + threadIdx.x, gsz = (i64)gridDim.x * 256;
    for (i64 i = gtid; i < n; i += gsz) {
        double lik = 0.0;
        for (int j = 0; j < lr.msplit; ++j) lik += lr.lpart[(i64)j * n + i];
        lp[i] = logreg_lp_row(theta + i * d, d, lik, lr.csum, lr, log_norm);
    }
}

__global__ __launch_bounds__(256) void k_prep_x(const double *X, const double *y, i64 m_rows,
                                                int d, i64 mpad, int dp, unsigned short *xs,
                                                unsigned short *thb, i64 thb_elems)
{
    const i64 gtid = (i64)blockIdx.x * 256 + threadIdx.x, gsz = (i64)gridDim.x * 256;
    for (i64 e = gtid; e < mpad * dp; e += gsz) {
        const i64 m = e / dp;
        const int k = (int)(e - m * dp);
        double v = 0.0;
        if (m < m_rows && k < d) v = (y[m] != 0.0 ? -1.0 : 1.0) * X[m * d + k];
        xs[xs_at(m, k, dp)] = to_bf16(v);
    }
    for (i64 e = gtid; e < thb_elems; e += gsz) thb[e] = 0;
}

__global__ __launch_bounds__(256) void k_theta_bf16(const double *x, i64 n, int d, int dp,
                                                    unsigned short *thb)
{
    const i64 gtid = (i64)blockIdx.x * 256 + threadIdx.x, gsz = (i64)gridDim.x * 256;
    for (i64 e = gtid; e < n * d; e += gsz) {
        const i64 i = e / d;
        const int k = (int)(e - i * d);
        thb[i * dp + k] = to_bf16(x[e] * kLog2e);
    }
}

// ================================================================= host side
namespace {

TArgs targs(const smc_config &c, const Work &w, bool with_bf16)
{
    TArgs a;
    a.kind = c.target;
    a.d = c.d;
    a.dp = w.dp;
    a.mean = c.mean;
    a.prec = c.prec;
    a.log_norm = c.log_norm;
    a.mu = c.mu;
    a.inv_nu = c.target == SMC_TARGET_STUDENT ? 1.0 / c.nu : 0.0;
    a.hnu1 = 0.5 * (c.nu + 1.0);
    a.init_mean = c.init_mean;
    a.init_sd = c.init_sd;
    a.init_prec = 1.0 / (c.init_sd * c.init_sd);
    a.init_log_norm = c.init_log_norm;
    a.rw_sd = c.rw_sd;
    a.seed = c.seed;
    a.sampler = c.sampler_id;
    a.thb = with_bf16 ? w.thb : nullptr;
    a.obs = c.obs;
    a.delta = c.delta;
    const double s11 = 5.0 * c.delta * c.delta * c.delta / 3.0;
    const double s21 = 5.0 * c.delta * c.delta / 2.0;
    const double s22 = 5.0 * c.delta;
    a.l11 = std::sqrt(s11);
    a.l21 = s21 / a.l11;
    a.l22 = std::sqrt(s22 - a.l21 * a.l21);
    a.obs_prec = c.target == SMC_TARGET_BEARING ? 1.0 / c.obs_var : 0.0;
    a.obs_log_norm = c.obs_log_norm;
    a.reset = -std::log((double)c.n);
    a.uniform = c.lazy_reset ? &w.ctrl->uniform : nullptr;
    return a;
}

int grid_for(int64_t n)
{
    int64_t b = (n + 255) / 256;
    return (int)(b < 1 ? 1 : (b > kMaxBlocks ? kMaxBlocks : b));
}

bool is_bf16(const smc_config &c)
{
    return c.target == SMC_TARGET_LOGREG && c.loglik_precision == SMC_PREC_BF16;
}

LrArgs lr_args(const smc_config &c, const Work &w)
{
    const bool bf = is_bf16(c);
    return LrArgs{w.lpart, kLogregSplit, w.csum, bf ? 0.5 * kLn2 : 0.5, c.prior_prec, bf ? 1 : 0};
}

// Partial log-likelihoods at x[n][d] into lpart.
hipError_t logreg_lik(const smc_config &c, const Work &w, const double *x, int64_t n,
                      bool theta_ready, hipStream_t s)
{
    if (c.target != SMC_TARGET_LOGREG || !w.lpart || !w.csum || (is_bf16(c) && (!w.xs || !w.thb)) ||
        (!is_bf16(c) && (!w.xf || !w.etab)))
        return hipErrorInvalidValue;
    const int msplit = kLogregSplit;
    if (is_bf16(c)) {
        if (!theta_ready) {
            hipLaunchKernelGGL(k_theta_bf16, dim3(grid_for(n * c.d)), dim3(256), 0, s, x, (i64)n,
                               c.d, w.dp, w.thb);
        }
        const dim3 grid((unsigned)((n + 127) / 128), msplit);
        const unsigned short *xs = w.xs;
        switch (w.dp / 16) {
        case 1: hipLaunchKernelGGL(k_logreg_bf16<1>, grid, dim3(256), 0, s, w.thb, (i64)n, xs, c.m_rows, w.mpad, w.dp, w.lpart); break;
        case 2: hipLaunchKernelGGL(k_logreg_bf16<2>, grid, dim3(256), 0, s, w.thb, (i64)n, xs, c.m_rows, w.mpad, w.dp, w.lpart); break;
        case 3: hipLaunchKernelGGL(k_logreg_bf16<3>, grid, dim3(256), 0, s, w.thb, (i64)n, xs, c.m_rows, w.mpad, w.dp, w.lpart); break;
        default: hipLaunchKernelGGL(k_logreg_bf16<4>, grid, dim3(256), 0, s, w.thb, (i64)n, xs, c.m_rows, w.mpad, w.dp, w.lpart); break;
        }
    } else {
        const dim3 grid((unsigned)((n + 63) / 64), msplit);
        const double *xf = w.xf;
        switch (lr_ks(c.d)) {
#define SMC_LR64_CASE(KS)                                                                      \
    case KS:                                                                                   \
        hipLaunchKernelGGL(k_logreg_f64<KS>, grid, dim3(256), 0, s, x, (i64)n, c.d, xf, w.etab, \
                           c.m_rows, w.mpad, w.lpart);                                         \
        break;
            SMC_LR64_CASE(1) SMC_LR64_CASE(2) SMC_LR64_CASE(4) SMC_LR64_CASE(6) SMC_LR64_CASE(8)
            SMC_LR64_CASE(10) SMC_LR64_CASE(12) SMC_LR64_CASE(14) SMC_LR64_CASE(16)
#undef SMC_LR64_CASE
        default: return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

template <int kKind, bool kInit, int kD = 1>
void launch_is_k(dim3 g, hipStream_t s, const TArgs &a, i64 n, uint32_t t, double *x, double *logw,
                 const Work &w, u64 *sp, Dst dst)
{
    auto kern = k_is<kKind, kInit, kInPlace, kD>;
    if constexpr (!kInit) {
        if (dst == kToCopy) kern = k_is<kKind, false, kToCopy, kD>;
        if constexpr (kKind != SMC_TARGET_BEARING)
            if (dst == kToBoth) kern = k_is<kKind, false, kToBoth, kD>;
    }
    hipLaunchKernelGGL(kern, g, dim3(256), 0, s, a, n, t, x, logw, w.lp, sp, w.is_part, w.x_scr,
                       w.lp_scr);
}

// The same for rows of several coordinates, with their log-targets.
template <int kKind, bool kInit>
void launch_rows_k(dim3 g, hipStream_t s, const TArgs &a, i64 n, uint32_t t, double *x,
                   double *logw, const Work &w, u64 *sp, Dst dst, const LrArgs &lr)
{
    const int P = rows_per_block(n, a.d);
    const size_t lds = (size_t)P * (row_stride(a.d) + 1) * sizeof(double);
    auto kern = k_rows<kKind, kInit, kInPlace>;
    if constexpr (!kInit) {
        if (dst == kToCopy) kern = k_rows<kKind, false, kToCopy>;
        if (dst == kToBoth) kern = k_rows<kKind, false, kToBoth>;
    }
    hipLaunchKernelGGL(kern, g, dim3(256), lds, s, a, n, t, P, x, logw, w.lp, sp, w.is_part,
                       w.x_scr, w.lp_scr, lr);
}

template <bool kInit>
hipError_t launch_is(const smc_config &c, const Work &w, int par, uint32_t t, double *x,
                     double *logw, hipStream_t s, Dst out = kInPlace)
{
    const TArgs a = targs(c, w, is_bf16(c));
    const dim3 g(w.is_grid);
    const i64 n = c.n;
    u64 *sp = w.slots + (par & 1) * kSlots * kSlotStride;
    switch (c.target) {
    case SMC_TARGET_GAUSS:
        if (c.d == 1) launch_is_k<SMC_TARGET_GAUSS, kInit>(g, s, a, n, t, x, logw, w, sp, out);
        else if (c.d == 2)
            launch_is_k<SMC_TARGET_GAUSS, kInit, 2>(g, s, a, n, t, x, logw, w, sp, out);
        else launch_rows_k<SMC_TARGET_GAUSS, kInit>(g, s, a, n, t, x, logw, w, sp, out, LrArgs{});
        break;
    case SMC_TARGET_STUDENT:
        launch_is_k<SMC_TARGET_STUDENT, kInit>(g, s, a, n, t, x, logw, w, sp, out);
        break;
    case SMC_TARGET_BEARING:
        launch_is_k<SMC_TARGET_BEARING, kInit>(g, s, a, n, t, x, logw, w, sp, out);
        break;
    case SMC_TARGET_LOGREG: {
        const int P = rows_per_block(n, c.d);
        hipLaunchKernelGGL(k_propose<kInit>, dim3((unsigned)row_chunks(n, c.d)), dim3(256), 0, s,
                           a, n, t, P, x, out == kInPlace ? nullptr : w.x_scr);
        if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
        if (logreg_lik(c, w, x, n, true, s) != hipSuccess) return hipErrorLaunchFailure;
        launch_rows_k<SMC_TARGET_LOGREG, kInit>(g, s, a, n, t, x, logw, w, sp, out,
                                                lr_args(c, w));
        break;
    }
    default:
        return hipErrorInvalidValue;
    }
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    // initialisation has no scan; its max is folded on its own
    return kInit ? launch_fold(w, par, s) : hipSuccess;
}

template <int kKind, int kD = 1>
int resident_blocks()
{
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_is<kKind, false, kInPlace, kD>, 256, 0) !=
        hipSuccess)
        return 0;
    return nb;
}

}  // namespace

int sampler_grid(const smc_config &c)
{
    // k_rows: one workgroup per chunk of rows
    if (c.target == SMC_TARGET_LOGREG || (c.target == SMC_TARGET_GAUSS && c.d > 2)) {
        const int64_t g = row_chunks(c.n, c.d);
        return (int)(g < kIsBlocks ? g : kIsBlocks);
    }
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    int per_cu = 0;
    switch (c.target) {
    case SMC_TARGET_GAUSS:
        per_cu = c.d == 1 ? resident_blocks<SMC_TARGET_GAUSS>()
                          : resident_blocks<SMC_TARGET_GAUSS, 2>();
        break;
    case SMC_TARGET_STUDENT: per_cu = resident_blocks<SMC_TARGET_STUDENT>(); break;
    case SMC_TARGET_BEARING: per_cu = resident_blocks<SMC_TARGET_BEARING>(); break;
    default: return 0;
    }
    if (per_cu < 1) return 0;
    int64_t g = (int64_t)per_cu * cus;
    const int64_t need = (c.n + 255) / 256;
    g = g < need ? g : need;
    g = g < kIsBlocks ? g : kIsBlocks;
    return (int)(g < 1 ? 1 : g);
}

smc_status step_init(const smc_config &c, const Work &w, int par, double *x, double *logw,
                     hipStream_t s)
{
    if (c.target == SMC_TARGET_LOGREG && is_bf16(c)) {
        const int64_t thb_elems = w.npad * w.dp;
        hipLaunchKernelGGL(k_prep_x, dim3(grid_for(w.mpad * w.dp)), dim3(256), 0, s,
                           reinterpret_cast<const double *>(c.X), c.y, (i64)c.m_rows, c.d,
                           (i64)w.mpad, w.dp, w.xs, w.thb, (i64)thb_elems);
        hipLaunchKernelGGL(k_xs_colsum, dim3(c.d), dim3(256), 0, s, w.xs, (i64)c.m_rows, w.dp,
                           w.csum);
        if (hipGetLastError() != hipSuccess) return SMC_E_DEVICE;
    } else if (c.target == SMC_TARGET_LOGREG) {
        const int ks = lr_ks(c.d);
        hipLaunchKernelGGL(k_prep_xf, dim3(grid_for(w.mpad * 4 * ks)), dim3(256), 0, s,
                           reinterpret_cast<const double *>(c.X), c.y, (i64)c.m_rows, c.d,
                           (i64)w.mpad, ks, w.xf);
        hipLaunchKernelGGL(k_exp_table, dim3(kExpN / 256), dim3(256), 0, s, w.etab);
        hipLaunchKernelGGL(k_x_colsum, dim3(c.d), dim3(256), 0, s,
                           reinterpret_cast<const double *>(c.X), c.y, (i64)c.m_rows, c.d, w.csum);
        if (hipGetLastError() != hipSuccess) return SMC_E_DEVICE;
    }
    if (launch_is<true>(c, w, par, 0u, x, logw, s) != hipSuccess) return SMC_E_DEVICE;
    if (c.target == SMC_TARGET_BEARING)  // equal initial weights: sums from the common reference
        hipLaunchKernelGGL(k_post_est<4>, dim3(w.is_grid), dim3(256), 0, s, w.ctrl, (i64)c.n,
                           c.d, x, logw, w.is_part);
    hipLaunchKernelGGL(k_init_stats, dim3(1), dim3(1024), 0, s, w.ctrl, w.is_part, w.is_grid,
                       c.d, w.rec_num);
    return hipGetLastError() == hipSuccess ? SMC_OK : SMC_E_DEVICE;
}

// The one-workgroup iteration where it is the faster one.  Against the separate
// kernels' 22.5 to 23.5 us (18.5 with one coordinate) at these sizes it takes
// 6.1 us at N = 256, 7.2 at 1024 and 10.4 at 2048 with one coordinate, 14.8 at
// N = 2048 with two, 19.2 at 1536 with four, 20.4 at 1024 with six, 20.6 at 512 and
// 25.0 at 640 with eight; the draws of one compute unit set the line.  Above eight
// coordinates the separate kernels take 17.5 us whatever the few particles, and one
// workgroup 16 to 17 up to 2 particles of nine or ten, 18 to 20 at 8, 21 to 27 at 64:
// they go to the separate kernels at every size.
bool small_path(const smc_config &c)
{
    if (c.n > kSmallN) return false;
    if (c.target == SMC_TARGET_STUDENT) return true;
    if (c.target != SMC_TARGET_GAUSS || c.d > kSmallD) return false;
    return c.d == 1 || c.n * ((c.d + 1) / 2) <= (c.d <= 6 ? kSmallPairs : 2048);
}

// Small population: the whole iteration in one workgroup and one launch.
smc_status small_step(const smc_config &c, const Work &w, int K, int par, uint32_t t, double *x,
                      double *logw, smc_resample_info *info, double *est, hipStream_t s)
{
    const int64_t n = c.n;
    const TArgs a = targs(c, w, false);
    const double reset = -std::log((double)n);
    u64 *other = w.slots + ((par & 1) ^ 1) * kSlots * kSlotStride;
    auto kern = c.target == SMC_TARGET_GAUSS
                    ? (c.d == 1   ? k_small_step<SMC_TARGET_GAUSS, 1, kSmallN>
                       : c.d <= 4 ? k_small_step<SMC_TARGET_GAUSS, 4, kSmallN>
                                  : k_small_step<SMC_TARGET_GAUSS, 8, 1024>)
                    : k_small_step<SMC_TARGET_STUDENT, 1, kSmallN>;
    static_assert(kSmallPairs / 3 <= 1024, "rows of five and more coordinates");
    hipLaunchKernelGGL(kern, dim3(1), dim3((unsigned)((n + 127) / 128 * 64)), 0, s, a, (i64)n, t,
                       K, c.mode, c.ess_num, c.ess_den, x, logw, w.lp, w.ctrl, other, w.rec_num,
                       info, est, reset);
    return hipGetLastError() == hipSuccess ? SMC_OK : SMC_E_DEVICE;
}

// The filter's row sums of an iteration, in at most kIsBlocks rows.
static StatsArgs filter_sums(const smc_config &c, const Work &w, double *est,
                             smc_resample_info *info, hipStream_t s)
{
    const int64_t nseg = filter_segments(c.n);
    const bool fold = nseg > kIsBlocks;
    if (fold)
        hipLaunchKernelGGL(k_fold_rows, dim3(kFoldBlocks), dim3(64), 0, s, w.epart, (i64)nseg,
                           w.is_part);
    StatsArgs st;
    st.is_part = fold ? w.is_part : w.epart;
    st.nblk = fold ? kFoldBlocks : (int)nseg;
    st.d = c.d;
    st.rec_num = w.rec_num;
    st.est = est;
    st.info = info;
    return st;
}

// Where a resampling iteration's weights go instead of logw (lazy reset);
// populations of at most kSmallN particles always write them.
static unsigned *uniform_mark(const smc_config &c, const Work &w)
{
    return c.lazy_reset && c.n > kSmallN ? &w.ctrl->uniform : nullptr;
}

template <bool kMove>
static hipError_t launch_filter_step(const smc_config &c, const Work &w, int par, uint32_t t,
                                     const double *x, double *xo, double *logw, hipStream_t s)
{
    FilterArgs g;
    g.n = c.n;
    g.t = t;
    g.pref = w.pref;
    g.pref64 = w.pref64;
    g.tpre = w.tsum;
    g.ctrl = w.ctrl;
    g.tsh = w.tile_shift;
    g.x = x;
    g.xo = xo;
    g.logw = logw;
    g.slots_p = w.slots + (par & 1) * kSlots * kSlotStride;
    g.est_part = w.epart;
    g.uniform = uniform_mark(c, w);
    const int seg = filter_seg_len(c.n);
    auto kern = seg == 256    ? k_filter_step<256, kMove>
                : seg == 512  ? k_filter_step<512, kMove>
                : seg == 1024 ? k_filter_step<1024, kMove>
                              : k_filter_step<kSegLen, kMove>;
    hipLaunchKernelGGL(kern, dim3((unsigned)filter_segments(c.n)), dim3(kExpandThreads), 0, s,
                       targs(c, w, false), g);
    return hipGetLastError();
}

// The end of a filter iteration: the redistribution into x, and the mean, which
// Alg 1 takes after resampling (the same sums in the same order as inside a call).
static smc_status filter_finish(const smc_config &c, const Work &w, double *x, double *logw,
                                double *est, smc_resample_info *info, hipStream_t s)
{
    if (launch_filter_step<false>(c, w, 0, 0, w.x_scr, x, logw, s) != hipSuccess)
        return SMC_E_DEVICE;
    const StatsArgs st = filter_sums(c, w, est, info, s);
    hipLaunchKernelGGL(k_step_stats, dim3(1), dim3(1024), 0, s, w.ctrl, st.is_part, st.nblk, c.d,
                       w.rec_num, est, info);
    return hipGetLastError() == hipSuccess ? SMC_OK : SMC_E_DEVICE;
}

// Several iterations of the particle filter: the rows go back and forth between x
// and the workspace copy, so that the last proposals end in the copy and the
// redistribution writes x.
static smc_status filter_run_n(const smc_config &c, const Work &w, int K, int par0, uint32_t t0,
                               int nsteps, double *x, double *logw, smc_resample_info *info,
                               double *est, hipStream_t s)
{
    StatsArgs tail;  // of the iteration before: formed beside the next one's scan
    for (int i = 0; i < nsteps; ++i) {
        const int par = par0 ^ (i & 1);
        const uint32_t t = t0 + (uint32_t)i;
        const bool to_copy = ((nsteps - 1 - i) & 1) == 0;
        if (i == 0) {
            if (launch_is<false>(c, w, par, t, x, logw, s, to_copy ? kToCopy : kInPlace) !=
                hipSuccess)
                return SMC_E_DEVICE;
        } else {
            double *from = to_copy ? x : w.x_scr, *to = to_copy ? w.x_scr : x;
            if (launch_filter_step<true>(c, w, par, t, from, to, logw, s) != hipSuccess)
                return SMC_E_DEVICE;
            tail = filter_sums(c, w, est ? est + (int64_t)(i - 1) * 4 * c.d : nullptr,
                               info ? info + (i - 1) : nullptr, s);
        }
        if (launch_quant_scan(w, logw, c.n, K, par, s, c.lazy_reset != 0, tail) != hipSuccess)
            return SMC_E_DEVICE;
        if (launch_decide(w, par, c.n, K, resample_word(c.seed, c.sampler_id, t), c.mode,
                          c.ess_num, c.ess_den, info ? info + i : nullptr, s) != hipSuccess)
            return SMC_E_DEVICE;
    }
    return filter_finish(c, w, x, logw, est ? est + (int64_t)(nsteps - 1) * 4 * c.d : nullptr,
                         info ? info + (nsteps - 1) : nullptr, s);
}

smc_status step_run_n(const smc_config &c, const Work &w, int K, int par0, uint32_t t0,
                      int nsteps, double *x, double *logw, smc_resample_info *info, double *est,
                      hipStream_t s)
{
    if (c.target == SMC_TARGET_BEARING && nsteps > 1)
        return filter_run_n(c, w, K, par0, t0, nsteps, x, logw, info, est, s);
    for (int i = 0; i < nsteps; ++i) {
        const smc_status st = step_run(c, w, K, par0 ^ (i & 1), t0 + (uint32_t)i, x, logw,
                                       info ? info + i : nullptr,
                                       est ? est + (int64_t)i * 4 * c.d : nullptr, s);
        if (st != SMC_OK) return st;
    }
    return SMC_OK;
}

smc_status step_run(const smc_config &c, const Work &w, int K, int par, uint32_t t, double *x,
                    double *logw, smc_resample_info *info, double *est, hipStream_t s)
{
    if (small_path(c)) return small_step(c, w, K, par, t, x, logw, info, est, s);
    const int64_t n = c.n;
    const bool pf = c.target == SMC_TARGET_BEARING;
    // Resampling forced every iteration, and the particle filter (its weights
    // collapse almost every update, and its redistribution adds up the rows that it
    // writes): the proposal goes to the workspace copy
    // and the redistribution writes x (an identity copy if the step found an
    // error or kept the weights).  ESS rule: to both, and a resampling
    // redistribution overwrites x.  The logistic regression reads its proposal
    // back from x and so always writes it there.
    const bool fwd = (c.mode == SMC_MODE_FORCE && c.target != SMC_TARGET_LOGREG) || pf;
    const bool keep = c.mode == SMC_MODE_NEVER && !pf;
    if (launch_is<false>(c, w, par, t, x, logw, s,
                         fwd ? kToCopy : keep ? kInPlace : kToBoth) != hipSuccess)
        return SMC_E_DEVICE;
    // Alg 2 estimates come before resampling: their sums are folded beside the scan
    // and finished by the decision's workgroup (the filter takes its mean after
    // resampling, below)
    StatsArgs st;
    if (!pf) {
        st.is_part = w.is_part;
        st.nblk = w.is_grid;
        st.d = c.d;
        st.cols = w.cols;
        st.rec_num = w.rec_num;
        st.est = est;
    }
    if (launch_quant_scan(w, logw, n, K, par, s, c.lazy_reset != 0, st) != hipSuccess)
        return SMC_E_DEVICE;
    const uint64_t r = resample_word(c.seed, c.sampler_id, t);
    if (launch_decide(w, par, n, K, r, c.mode, c.ess_num, c.ess_den, info, s, st) != hipSuccess)
        return SMC_E_DEVICE;
    if (keep) return SMC_OK;
    if (pf) return filter_finish(c, w, x, logw, est, info, s);
    ExpandOut o;
    o.mode = fwd ? ExpandMode::kForward : ExpandMode::kIfResampled;
    o.logw = logw;
    o.reset = -std::log((double)n);
    o.uniform = uniform_mark(c, w);
    // the 1-D Gaussian and Student-t samplers carry no cached log-target
    if (!(c.d == 1 && (c.target == SMC_TARGET_GAUSS || c.target == SMC_TARGET_STUDENT))) {
        o.aux = w.lp_scr;
        o.aux_out = w.lp;
    }
    return launch_expand(w, n, 0, w.x_scr, x, c.d * 8, s, o) == hipSuccess ? SMC_OK : SMC_E_DEVICE;
}

__global__ __launch_bounds__(256) void k_sync_weights(const Ctrl *ctrl, i64 n, double *logw,
                                                      double reset)
{
    if (!ctrl->uniform) return;
    const i64 gtid = (i64)blockIdx.x * 256 + threadIdx.x, gsz = (i64)gridDim.x * 256;
    for (i64 i = gtid; i < n; i += gsz) logw[i] = reset;
}

smc_status step_sync_weights(const smc_config &c, const Work &w, double *logw, hipStream_t s)
{
    if (!c.lazy_reset) return SMC_OK;
    hipLaunchKernelGGL(k_sync_weights, dim3(grid_for(c.n)), dim3(256), 0, s, w.ctrl, (i64)c.n,
                       logw, -std::log((double)c.n));
    return hipGetLastError() == hipSuccess ? SMC_OK : SMC_E_DEVICE;
}

smc_status step_log_target(const smc_config &c, const Work &w, const double *x, int64_t n,
                           double *lp, hipStream_t s)
{
    if (n > c.n) return SMC_E_ARG;
    if (c.target == SMC_TARGET_LOGREG) {
        if (logreg_lik(c, w, x, n, false, s) != hipSuccess) return SMC_E_DEVICE;
        hipLaunchKernelGGL(k_logreg_sum, dim3(grid_for(n)), dim3(256), 0, s, x, (i64)n, c.d,
                           lr_args(c, w), c.log_norm, lp);
        return hipGetLastError() == hipSuccess ? SMC_OK : SMC_E_DEVICE;
    }
    const TArgs a = targs(c, w, false);
    hipLaunchKernelGGL(k_lp_cheap, dim3(grid_for(n)), dim3(256), 0, s, a, (i64)n, x, lp);
    return hipGetLastError() == hipSuccess ? SMC_OK : SMC_E_DEVICE;
}

}  // namespace smc
