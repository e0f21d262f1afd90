// The sampler's per-iteration statistics, by workgroups beside other work.
//
// Every block of the update leaves one row of partial sums, stored by columns
// (column c of block b at part[c nblk + b]: the folding wavefronts read whole
// cache lines; stored by rows, the reads of 22 columns alone took 9 us):
// the block's reference weight, sum e, sum e x_k (k < d), sum e x_k^2, with e
// relative to the reference.  A block without weight carries -inf and zeros.
#pragma once

#include "../../include/smc.h"
#include "common.hpp"
#include "det.hpp"
#include "kernels.hpp"

namespace smc {

// LDS of the statistics.
struct StatsLds {
    double sc[kIsBlocks];  // scale of each block's sums
    double mk[16];
};

template <int NT>
struct StepStats {
    static constexpr int NW = NT / 64;
    static constexpr int kPer = (kIsBlocks + NT - 1) / NT;
    static_assert(NW <= 16, "wave totals");
    double mb[kPer];

    // References of this thread's blocks; their maximum per wavefront into LDS.
    __device__ void begin(StatsLds &L, const double *part, int nblk)
    {
        const int tid = threadIdx.x;
        double m = -__builtin_huge_val();
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int b = tid + NT * j;
            mb[j] = b < nblk ? part[b] : -__builtin_huge_val();
            m = fmax(m, mb[j]);
        }
        m = wave_max_f64(m);
        if ((tid & 63) == 0) L.mk[tid >> 6] = m;
    }

    // After a barrier: the scale of every block against the largest reference,
    // which it returns.
    __device__ double scale(StatsLds &L, int nblk)
    {
        const int tid = threadIdx.x;
        double m = L.mk[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) m = fmax(m, L.mk[w]);
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int b = tid + NT * j;
            if (b < nblk) L.sc[b] = mb[j] > -__builtin_huge_val() ? det_exp(mb[j] - m) : 0.0;
        }
        return m;
    }

    // After another barrier: column c by one wavefront, lanes over the blocks (a
    // fixed order), 16 loads in flight; in every lane.
    __device__ double column(const StatsLds &L, const double *part, int nblk, int c)
    {
        const int lane = threadIdx.x & 63;
        const double *pc = part + (i64)c * nblk;
        double acc = 0.0;
        constexpr int U = 16;
        for (int b0 = lane; b0 < nblk; b0 += 64 * U) {
            double v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int b = b0 + 64 * u;
                v[u] = pc[b < nblk ? b : b0];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int b = b0 + 64 * u;
                const double s = b < nblk ? L.sc[b] : 0.0;
                acc += s != 0.0 ? s * v[u] : 0.0;
            }
        }
        return wave_sum_f64(acc);
    }
};

// Workgroup `g` of the fold of an iteration's sums: columns 1 + NW g .. of `part`, a
// wavefront each, into cols.
template <int NT>
__device__ inline void fold_columns(StatsLds &L, const StatsArgs &st, int g)
{
    StepStats<NT> ss;
    ss.begin(L, st.is_part, st.nblk);
    __syncthreads();
    ss.scale(L, st.nblk);
    __syncthreads();
    const int c = 1 + StepStats<NT>::NW * g + (int)(threadIdx.x >> 6);
    if (c < 2 + 2 * st.d) {
        const double v = ss.column(L, st.is_part, st.nblk, c);
        if ((threadIdx.x & 63) == 0) st.cols[c] = v;
    }
}

// The control block's part of c_t and recycling, read before it is needed.
struct RecState {
    double logZ_prev, lc_max, rec_den;
    int rec_steps;
    __device__ explicit RecState(const Ctrl *c)
        : logZ_prev(c->logZ_prev), lc_max(c->lc_max), rec_den(c->rec_den), rec_steps(c->rec_steps)
    {
    }
};

// c_t (eq. normconst) and the recycling weights (eq. recycling) of an iteration
// without error; returns log c_t, leaves bc = (scale of the old sums, weight of
// this iteration, their denominator) and the state to store.
struct RecNext {
    double lc_max, rec_den;
    int rec_steps;
};

__device__ inline double recycle_step(const RecState &r, double logZ, double *bc, RecNext &nx)
{
    const double logc = logZ - r.logZ_prev;
    double sc = 1.0, den = r.rec_den, lc_max = r.lc_max;
    if (logc > lc_max) {
        sc = r.rec_steps ? exp(lc_max - logc) : 0.0;
        den *= sc;
        lc_max = logc;
    }
    const double wgt = exp(logc - lc_max);
    den += wgt;
    nx.lc_max = lc_max;
    nx.rec_den = den;
    nx.rec_steps = r.rec_steps + 1;
    bc[0] = sc;
    bc[1] = wgt;
    bc[2] = den;
    return logc;
}

__device__ inline void store_recycling(const RecNext &nx, double logc, double logZ, bool resampled,
                                       Ctrl *ctrl)
{
    ctrl->lc_max = nx.lc_max;
    ctrl->rec_den = nx.rec_den;
    ctrl->rec_steps = nx.rec_steps;
    ctrl->log_c = logc;
    ctrl->logZ_prev = resampled ? 0.0 : logZ;
}

// Estimate k < 2 d: f_t (eq. estimation_at_t) and the recycled one, from the
// sums' columns (1: the weights), the recycling's bc and rec_old = rec_num[k].
__device__ inline void write_estimate(int k, int d, double sum, double weights, double rec_old,
                                      const double *bc, double *rec_num, double *est)
{
    const double f = sum / weights;
    const double num = rec_old * bc[0] + bc[1] * f;
    rec_num[k] = num;
    if (est) {
        est[k] = f;
        est[2 * d + k] = num / bc[2];
    }
}

// The statistics of a filter iteration, whose weights, decision and log Z are in
// the control block, by one workgroup of NT threads.  The rows of `part` all carry
// the same reference, so their sums are added as they are: a wavefront takes a
// column, lanes over the rows, every load of a trip in flight.
template <int NT>
__device__ inline void filter_stats(Ctrl *ctrl, const double *part, int nblk, int d,
                                    double *rec_num, double *est, smc_resample_info *info)
{
    constexpr int NW = NT / 64;
    __shared__ double s_col[kEstCols], s_bc[3];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const RecState rec(ctrl);
    const unsigned err = ctrl->err_call, resampled = ctrl->resample;
    const double logZ = ctrl->logZ;
    const double rec_old = tid < 2 * d ? rec_num[tid] : 0.0;
    if (err) return;
    for (int c = 1 + wid; c < 2 + 2 * d; c += NW) {
        const double *pc = part + (i64)c * nblk;
        double acc = 0.0;
        constexpr int U = 16;
        for (int b0 = lane; b0 < nblk; b0 += 64 * U) {
            double v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int b = b0 + 64 * u;
                v[u] = pc[b < nblk ? b : b0];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) acc += b0 + 64 * u < nblk ? v[u] : 0.0;
        }
        acc = wave_sum_f64(acc);
        if (lane == 0) s_col[c] = acc;
    }
    if (tid == 0) {
        double bc[3];
        RecNext nx;
        const double logc = recycle_step(rec, logZ, bc, nx);
        store_recycling(nx, logc, logZ, resampled != 0, ctrl);
        if (info) info->log_c = logc;
        for (int i = 0; i < 3; ++i) s_bc[i] = bc[i];
    }
    __syncthreads();
    if (tid < 2 * d)
        write_estimate(tid, d, s_col[2 + tid], s_col[1], rec_old, s_bc, rec_num, est);
}

}  // namespace smc
