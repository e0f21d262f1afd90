// Wave-cooperative standard normals: for pair `pair` of particle `idx`, the
// polar method on the uniforms of attempts 0, 1, ... (at most 32) until one is
// accepted, (0, 0) if none is.
//
// The polar method accepts a Philox draw with probability pi/4, so a wave of
// 64 lanes that retries in lockstep runs about 3.5 attempts (the maximum of 64
// geometric counts) although each lane needs 1.27 on average, and repeats the
// logarithm for every attempt in which some lane accepts.  Here every lane
// first tries attempt 0 of its own pair; the pairs still pending are then
// spread over the whole wave, L = floor(64 / pending) lanes per pair, each
// lane trying one later attempt of its pair (jobs and results pass through a
// per-wave LDS buffer).  A pair takes the lowest attempt
// that accepted, which is the draw the sequential definition takes, and the
// logarithm runs once per lane at the end, for the W pairs of a lane together
// (their polynomials share the coefficients).  All 64 lanes must call it in
// convergent control flow; lanes without a pair pass active = false.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "det.hpp"

namespace smc {

// k 2^-52 - 1 for the top 53 bits k of the 64-bit word (hi, lo), exact: both
// parts of k are placed in the low bits of a double whose exponent gives them
// their weight (2^21 + hi 2^-31, and 1 + (lo >> 11) 2^-52), two exact sums
// remove the offsets.  No integer conversion, product or scaling.
__device__ inline double unit_pm1(uint32_t hi, uint32_t lo)
{
    const double a = __hiloint2double(0x41400000, (int)hi);
    const double b = __hiloint2double(0x3FF00000, (int)(lo >> 11));
    return (a - 2097154.0) + b;
}

__device__ inline bool polar_uniforms(uint64_t seed, uint32_t tag, uint32_t sampler, uint32_t t,
                                      uint32_t idx, uint32_t sub, double &v1, double &v2)
{
    const Philox4 w = draw(seed, tag, sampler, t, idx, sub);
    v1 = unit_pm1(w.v[1], w.v[0]);
    v2 = unit_pm1(w.v[3], w.v[2]);
    const double s = v1 * v1 + v2 * v2;
    return s > 0.0 && s < 1.0;
}

// The accepted uniforms of one pair per lane; false (and 0, 0) for an idle
// lane or after 32 rejections.  xch: this wave's 64-entry exchange buffer in
// LDS (16 bytes a lane).  Lanes of one wave read and write it in program
// order, so no barrier is needed.
__device__ inline bool polar_wave(uint64_t seed, uint32_t tag, uint32_t sampler, uint32_t t,
                                  uint32_t idx, uint32_t pair, bool active, double &v1,
                                  double &v2, uint4 *xch)
{
    constexpr uint32_t kAttempts = 32;
    const int lane = (int)__lane_id();
    v1 = v2 = 0.0;
    bool ok = polar_uniforms(seed, tag, sampler, t, idx, pair << 16, v1, v2) && active;
    bool dead = false;         // all attempts rejected: the pair is (0, 0)
    uint32_t next = 1;         // next attempt of this lane's pair
    uint64_t pend = __ballot(active && !ok);
    while (pend) {
        const int r = __popcll(pend);
        // floor(64 / r) and floor(lane / L) from FP32 reciprocals of small
        // integers, half a unit away from every rounding edge: exact
        const int L = __builtin_amdgcn_readfirstlane(
            (int)(64.5f * __builtin_amdgcn_rcpf((float)r)));
        const bool own = (pend >> lane) & 1ull;
        const int rank = (int)__builtin_amdgcn_mbcnt_hi(
            (unsigned)(pend >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)pend, 0u));
        // pending pair number `rank` is posted at entry `rank`; helpers of
        // pair j (L lanes each) read entry j and try the next L attempts
        if (own) xch[rank] = make_uint4(idx, pair, next, 0u);
        __builtin_amdgcn_wave_barrier();
        const int j = (int)(((float)lane + 0.5f) * __builtin_amdgcn_rcpf((float)L));
        const int k = lane - j * L;
        const bool helper = j < r;
        const uint4 job = xch[helper ? j : 0];
        const uint32_t a = job.z + (uint32_t)k;
        double h1 = 0.0, h2 = 0.0;
        const bool hok = polar_uniforms(seed, tag, sampler, t, job.x, (job.y << 16) | a, h1, h2) &&
                         helper && a < kAttempts;
        const uint64_t acc = __ballot(hok);
        __builtin_amdgcn_wave_barrier();
        xch[lane] = make_uint4((uint32_t)__double2loint(h1), (uint32_t)__double2hiint(h1),
                               (uint32_t)__double2loint(h2), (uint32_t)__double2hiint(h2));
        __builtin_amdgcn_wave_barrier();
        const uint64_t seg = own ? (acc >> (rank * L)) & (L == 64 ? ~0ull : ((1ull << L) - 1ull))
                                 : 0ull;
        if (seg) {
            const uint4 h = xch[rank * L + __ffsll((long long)seg) - 1];
            v1 = __hiloint2double((int)h.y, (int)h.x);
            v2 = __hiloint2double((int)h.w, (int)h.z);
            ok = true;
        } else if (own) {
            next += (uint32_t)L;
            dead = next >= kAttempts;
        }
        __builtin_amdgcn_wave_barrier();
        pend = __ballot(own && !ok && !dead);
    }
    return ok;
}

// W pairs per lane: pair[q] of particle idx[q] gives z[2 q], z[2 q + 1].  np
// (wave-uniform): pairs from np on are skipped (their z are 0).
// s = v1^2 + v2^2 lies in [2^-104, 1), so the logarithm, quotient and root take
// the in-range forms.
template <int W>
__device__ inline void normal_pairs_wave(uint64_t seed, uint32_t tag, uint32_t sampler,
                                         uint32_t t, const uint32_t (&idx)[W],
                                         const uint32_t (&pair)[W], int np,
                                         const bool (&active)[W], double (&z)[2 * W], uint4 *xch)
{
    double v1[W], v2[W], s[W], c[W];
    bool ok[W];
#pragma unroll
    SMC_EACH {
        ok[w] = false;
        if (w < np)
            ok[w] = polar_wave(seed, tag, sampler, t, idx[w], pair[w], active[w], v1[w], v2[w],
                               xch);
        if (!ok[w]) {
            v1[w] = 0.5;  // any accepted draw: keeps the arithmetic in range
            v2[w] = 0.0;
        }
        s[w] = v1[w] * v1[w] + v2[w] * v2[w];
    }
    det_log_w<W>(s, c);
#pragma unroll
    SMC_EACH c[w] = -2.0 * c[w];
    det_div_w<W>(c, s, c);
    det_sqrt_w<W>(c, c);
#pragma unroll
    SMC_EACH {
        z[2 * w] = ok[w] ? v1[w] * c[w] : 0.0;
        z[2 * w + 1] = ok[w] ? v2[w] * c[w] : 0.0;
        // keeps the arithmetic here: sunk under the caller's guard it would
        // leave the coefficients behind, all of them live at once
        asm volatile("" : "+v"(z[2 * w]), "+v"(z[2 * w + 1]));
    }
}

__device__ inline void normal_pair_wave(uint64_t seed, uint32_t tag, uint32_t sampler, uint32_t t,
                                        uint32_t idx, uint32_t pair, bool active, double &z1,
                                        double &z2, uint4 *xch)
{
    const uint32_t i[1] = {idx}, p[1] = {pair};
    const bool act[1] = {active};
    double z[2];
    normal_pairs_wave<1>(seed, tag, sampler, t, i, p, 1, act, z, xch);
    z1 = z[0];
    z2 = z[1];
}

}  // namespace smc
