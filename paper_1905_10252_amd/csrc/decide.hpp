// Fixed-point weights, their sums and the resampling decision, shared by the
// tile scan, the one-workgroup resampling and the one-workgroup iteration.
#pragma once

#include "../../include/smc.h"
#include "common.hpp"
#include "det.hpp"

namespace smc {

// Sums of one thread's fixed-point weights squared, q = h 2^26 + l: each part
// adds up at most 16 products below 2^54, so plain 64-bit sums hold
// them (one multiply-add a part; carries enter once, in total()).
struct SqSum {
    u64 ll = 0, hl = 0, hh = 0;
    __device__ inline void add(u64 q)
    {
        const unsigned l = (unsigned)q & 0x3FFFFFFu, h = (unsigned)(q >> 26);
        ll += (u64)l * l;
        hl += (u64)h * l;
        hh += (u64)h * h;
    }
    __device__ inline U128 total() const  // ll + hl 2^27 + hh 2^52
    {
        const U128 t = add128(U128{hl << 27, hl >> 37}, U128{hh << 52, hh >> 12});
        return add128(t, ll);
    }
};

// Fixed-point weights floor(2^K e), e = exp(l - m) <= 1, of W log-weights, and
// their FP64 sums.  The integer is cut from the significand of e by one shift
// (at least 52 - K: e = 1 gives 2^K).  A NaN gives e = 0 (the max pass has
// flagged it).
template <int W>
__device__ inline void quant_w(const double (&v)[W], double m, int K, u64 (&q)[W], double &z,
                               double &z2, SqSum &q2, double (&e)[W])
{
    double a[W];
#pragma unroll
    SMC_EACH a[w] = v[w] - m;
    det_exp_w<W>(a, e);
#pragma unroll
    SMC_EACH {
        z += e[w];
        z2 = fma(e[w], e[w], z2);
        const unsigned hi = (unsigned)__double2hiint(e[w]);
        int sh = 1075 - K - (int)(hi >> 20);
        sh = sh > 63 ? 63 : (sh < 52 - K ? 52 - K : sh);
        const u64 sig = ((u64)((hi & 0xFFFFFu) | 0x100000u) << 32) | (unsigned)__double2loint(e[w]);
        q[w] = sig >> sh;
        q2.add(q[w]);
    }
}

template <int W>
__device__ inline void quant_w(const double (&v)[W], double m, int K, u64 (&q)[W], double &z,
                               double &z2, SqSum &q2)
{
    double e[W];
    quant_w<W>(v, m, K, q, z, z2, q2, e);
}

struct Decision {
    u64 key, S, U;
    U128 Q2;
    double m, logZ, ess, Z, Z2;
    unsigned err;
    bool resample;
};

// The error of the call, the exact integer ESS rule of Alg 2 and the
// systematic offset, from the max key and the sums.
__device__ inline Decision decide(u64 key, unsigned bad, u64 S, double Z, double Z2, U128 Q2,
                                  i64 n, u64 r, int mode, int ess_num, int ess_den)
{
    Decision d;
    d.key = key;
    d.m = okey_inv(key);
    d.err = 0;
    if (bad) d.err = kErrNonfinite;
    else if (key <= okey(-__builtin_huge_val())) d.err = kErrDegenerate;
    if (mode == SMC_MODE_FORCE) {
        d.resample = true;
    } else if (mode == SMC_MODE_NEVER) {
        d.resample = false;
    } else {
        // ess_den * S^2 < ess_num * N * Q2; both sides stay below 2^127
        const U128 lhs = mul128_small(mul64(S, S), (u64)ess_den);
        const U128 rhs = mul128_small(mul128_small(Q2, (u64)n), (u64)ess_num);
        d.resample = lt128(lhs, rhs);
    }
    if (d.err) d.resample = false;
    d.S = S;
    d.U = mul64(r, S).hi;
    d.Q2 = Q2;
    d.Z = Z;
    d.Z2 = Z2;
    d.logZ = d.m + log(Z);
    d.ess = (Z * Z) / Z2;
    return d;
}

// The control block and the caller's record, by one thread.
__device__ inline void store_decision(const Decision &d, int K, double log_c, Ctrl *ctrl,
                                      smc_resample_info *info)
{
    ctrl->mkey = d.key;
    ctrl->m = d.m;
    ctrl->err_call = d.err;
    if (d.err && !ctrl->err_latch) ctrl->err_latch = d.err;
    ctrl->S = d.S;
    ctrl->U = d.U;
    ctrl->Q2lo = d.Q2.lo;
    ctrl->Q2hi = d.Q2.hi;
    ctrl->Z = d.Z;
    ctrl->Z2 = d.Z2;
    ctrl->logZ = d.logZ;
    ctrl->ess = d.ess;
    ctrl->K = K;
    ctrl->resample = d.resample ? 1u : 0u;
    ctrl->pending = d.err ? 0 : 1;
    if (info) {
        info->m = d.m;
        info->logZ = d.logZ;
        info->ess = d.ess;
        info->Z = d.Z;
        info->Z2 = d.Z2;
        info->S = d.S;
        info->U = d.U;
        info->Q2_hi = d.Q2.hi;
        info->Q2_lo = d.Q2.lo;
        info->K = K;
        info->resampled = d.resample ? 1 : 0;
        info->err = (int)d.err;
        info->pad = 0;
        info->log_c = log_c;
    }
}

}  // namespace smc
