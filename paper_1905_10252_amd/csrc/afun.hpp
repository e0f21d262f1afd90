// The number of output rows taken from the first sources, A_j, and the test
// of the merge path on it, shared by the expand, the copy counts and the
// one-workgroup resampling.
#pragma once

#include "common.hpp"
#include "kernels.hpp"

namespace smc {

// n is below 2^31 (the library's limit), so n, A_j <= n and k - j <= 2n all
// fit 32 bits and every product below is a 32 x 64-bit one.
//
// (N S_j + U) / S is first formed in FP64 as S_j (N / S) + U / S.  Its value is
// at most N + 1 <= 2^31 and takes eight roundings of at most 2^-53 each, so it
// is within 2^-19 of the quotient: more than kSlack = 2^-18 away from an
// integer it settles the floor and every comparison with an integer.  The
// 128-bit products decide the rest, about one value in 2^17.
constexpr double kSlack = 0x1p-18;

__host__ __device__ inline double u64_to_f64(u64 v)
{
    return fma((double)(unsigned)(v >> 32), 0x1p32, (double)(unsigned)v);
}

struct AFun {
    i64 n;
    const u64 *pref;  // tile-local inclusive prefix
    const u64 *tpre;  // exclusive prefix of the tile totals
    int tsh;          // log2 of the tile size
    int mode;  // 0: identity, 1: systematic from S_j, 2: caller counts (A_j = prefix)
    u64 S, U;
    double nS, uS;  // N / S and U / S

    __host__ __device__ inline u64 at(i64 j) const { return pref[j] + tpre[j >> tsh]; }

    // Systematic copies from the fixed-point sum S and the offset U.
    __host__ __device__ inline void set_systematic(u64 S_, u64 U_)
    {
        mode = 1;
        S = S_;
        U = U_;
        const double invS = 1.0 / u64_to_f64(S);
        nS = (double)n * invS;
        uS = u64_to_f64(U) * invS;
    }

    // A_j + j < k, given the prefix value pj of source j
    __host__ __device__ inline bool pred_at(i64 j, u64 pj, i64 k) const
    {
        if (mode == 0) return 2 * j + 1 < k;
        if (mode == 2) return (i64)pj + j < k;
        const i64 c = k - j;
        if (c <= 0) return false;
        const double diff = fma(u64_to_f64(pj), nS, uS) - (double)(unsigned)c;
        if (fabs(diff) > kSlack) return diff < 0.0;
        const U128 lhs = add128(mul32x64((unsigned)n, pj), U);
        const U128 rhs = mul32x64((unsigned)c, S);
        return lt128(lhs, rhs);
    }

    __host__ __device__ inline bool pred(i64 j, i64 k) const
    {
        return pred_at(j, mode == 0 ? 0ull : at(j), k);
    }

    // A_j given the prefix value sj of source j
    __host__ __device__ inline unsigned A_of(i64 j, u64 sj) const
    {
        if (mode == 0) return (unsigned)(j + 1);
        if (mode == 2) return (unsigned)sj;
        const double est = fma(u64_to_f64(sj), nS, uS);
        unsigned a = (unsigned)est;
        const double fr = est - (double)a;
        if (fabs(fr - 0.5) < 0.5 - kSlack) return a;
        // exact correction to a S <= num < (a + 1) S
        const U128 num = add128(mul32x64((unsigned)n, sj), U);
        a = a <= (unsigned)n ? a : (unsigned)n;
        U128 aS = mul32x64(a, S);
        while (lt128(num, aS)) {
            --a;
            aS = mul32x64(a, S);
        }
        U128 a1S = add128(aS, S);
        while (!lt128(num, a1S)) {
            ++a;
            a1S = add128(a1S, S);
        }
        return a;
    }
};

// Chooses the A function of this call; false if nothing may be written.
__device__ inline bool make_afun(const Ctrl *ctrl, const u64 *pref, const u64 *tpre, int tsh,
                                 i64 n, int count_mode, AFun &f, bool report)
{
    f.n = n;
    f.pref = pref;
    f.tpre = tpre;
    f.tsh = tsh;
    f.S = 1;
    f.U = 0;
    f.nS = 0.0;
    f.uS = 0.0;
    if (count_mode) {
        if (ctrl->ncopy_bad || ctrl->ctotal != (u64)n) {
            if (report) {
                const unsigned err = kErrArg;
                Ctrl *c = const_cast<Ctrl *>(ctrl);
                c->err_call = err;
                if (!c->err_latch) c->err_latch = err;
            }
            return false;
        }
        f.mode = 2;
        return true;
    }
    if (!ctrl->pending || ctrl->err_call) return false;
    f.mode = 0;
    if (ctrl->resample) f.set_systematic(ctrl->S, ctrl->U);
    return true;
}

}  // namespace smc
