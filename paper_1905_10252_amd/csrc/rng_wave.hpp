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

// What the rows of a population are drawn from.
struct RowDraw {
    uint64_t seed;
    uint32_t sampler;
    double mean, sd;  // x0 ~ N(mean, sd^2 I); a step adds sd z to the row
};

typedef double f64x2r __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) double gdouble;
__device__ const f64x2r *vec_of(const double *);
__device__ const __attribute__((address_space(1))) f64x2r *vec_of(const gdouble *);

// Draws the proposal (kInit: x0) of particles [base, base + cnt) with d >= 2
// coordinates by the whole workgroup of 256 threads: items (particle, pair),
// neighbouring threads on neighbouring addresses.  put(p, c, two, vec, v0, v1):
// coordinates c and, if two, c + 1 of particle base + p; vec: both there, and
// 16-byte aligned in x.  total: values in x (an odd 1-D population drawn as
// rows of two ends early).  vec: x is 16-byte aligned.  cnt times the row's
// pairs is at most 2^14.  slot(it): where two doubles of item `it` wait in LDS.
//
// Nothing ties an item to a lane here, so the rejected ones are not resolved
// where they arose.  A wavefront takes a block of up to kMaxBlock items: it tries
// 64 new ones at a time, leaves the accepted uniforms in their slots and queues
// the others in LDS with their next attempt; a queue of 64 makes a trial of its
// own, and the last ones share the wavefront, floor(64 / pending) lanes trying
// consecutive attempts of each (the lowest accepted counts).  For 64 items that is
// 1.5 trials in blocks of 256 to 384, 1.9 in blocks of 128 and 2.1 in blocks of 64,
// where nothing is queued together; resolving every 64 items at once also takes 2.1,
// with an exchange of results each.  The logarithms and roots then run on whole
// wavefronts, two items a lane, and rows are read and written in whole lines
// (finishing each item where it was accepted scattered a fifth of the stores:
// 630 us against 478, proposal of the 256-sampler workload; vector unit busy 85 %).
constexpr int kDrawBlock = 256;  // where the items wait in a buffer of their own
constexpr int kDrawQueue = 128;  // entries a wavefront: fewer than 64 before a trial

template <bool kInit, int kMaxBlock, class Ptr, class Slot, class Put>
__device__ inline void draw_rows(const RowDraw &g, int d, long long base, int cnt,
                                 long long total, uint32_t t, Ptr x, bool vec,
                                 uint32_t (&queue)[4][kDrawQueue], Slot &&slot, Put &&put)
{
    constexpr uint32_t kAttempts = 32;
    const uint32_t tag = kInit ? (uint32_t)kTagInit : (uint32_t)kTagPropose;
    const int np = (d + 1) >> 1, items = cnt * np;
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float inv = 1.0f / (float)np;  // quotients below 2^14, half a unit from every edge
    const bool v2 = vec && (d & 1) == 0 && (total & 1) == 0;
    const Ptr xb = x + base * d;
    const long long left = total - base * d;  // values from here to the end of x
    const int lim = left < (1 << 30) ? (int)left : 1 << 30;
    uint32_t *q = queue[wid];
    int blk = (items + 255) / 256 * 64;  // an equal share, in whole wavefronts
    blk = blk < kMaxBlock ? blk : kMaxBlock;
    for (int it0 = wid * blk; it0 < items; it0 += 4 * blk) {
        const int m = items - it0 < blk ? items - it0 : blk;
        int qn = 0;
        // posts `e` of the lanes in `again` to the queue
        auto post = [&](bool again, uint32_t e) {
            const uint64_t mask = __ballot(again);
            __builtin_amdgcn_wave_barrier();
            if (again)
                q[qn + __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u))] =
                    e;
            qn += __popcll(mask);
            __builtin_amdgcn_wave_barrier();
            asm volatile("" ::: "memory");
        };
        // up to 64 queued items, L consecutive attempts of each
        auto queued = [&]() {
            const int n = qn < 64 ? qn : 64;
            qn -= n;
            // floor(64 / n) and floor(lane / L) from FP32 reciprocals of small
            // integers, half a unit away from every edge: exact
            const int L = __builtin_amdgcn_readfirstlane(
                (int)(64.5f * __builtin_amdgcn_rcpf((float)n)));
            const int j = (int)(((float)lane + 0.5f) * __builtin_amdgcn_rcpf((float)L));
            const int k = lane - j * L;
            const uint32_t e = q[qn + (j < n ? j : 0)];
            const uint32_t it = e & 0xFFFFu, first = e >> 16, attempt = first + (uint32_t)k;
            const int p = (int)(((float)it + 0.5f) * inv);
            const uint32_t pair = it - (uint32_t)(p * np);
            double v1, w1;
            const bool ok = polar_uniforms(g.seed, tag, g.sampler, kInit ? 0u : t,
                                           (uint32_t)(base + p), (pair << 16) | attempt, v1, w1) &&
                            j < n && attempt < kAttempts;
            const uint64_t acc = __ballot(ok);
            // accepted attempts of this lane's item, lowest first
            const uint64_t seg = (acc >> ((j * L) & 63)) & (L == 64 ? ~0ull : (1ull << L) - 1ull);
            const bool lost = j < n && k == 0 && seg == 0ull;
            const bool again = lost && first + (uint32_t)L < kAttempts;
            if (ok && (seg & ((1ull << k) - 1ull)) == 0ull) {
                double *s = slot((int)it);
                s[0] = v1;
                s[1] = w1;
            } else if (lost && !again) {  // every attempt rejected: the pair is (0, 0)
                double *s = slot((int)it);
                s[0] = s[1] = 0.0;
            }
            post(again, it | ((first + (uint32_t)L) << 16));
        };
        for (int next = 0; next < m; next += 64) {
            const bool act = next + lane < m;
            const int it = it0 + next + (act ? lane : 0);
            const int p = (int)(((float)it + 0.5f) * inv);
            const uint32_t pair = (uint32_t)(it - p * np);
            double v1, w1;
            const bool ok = polar_uniforms(g.seed, tag, g.sampler, kInit ? 0u : t,
                                           (uint32_t)(base + p), pair << 16, v1, w1);
            if (ok && act) {
                double *s = slot(it);
                s[0] = v1;
                s[1] = w1;
            }
            post(act && !ok, (uint32_t)it | (1u << 16));
            if (qn >= 64) queued();
        }
        while (qn > 0) queued();
        constexpr int W = 2;
        for (int i0 = 0; i0 < m; i0 += 64 * W) {
            int p[W], c[W];
            bool act[W], two[W];
            double x0[W], x1[W], v1[W], w1[W], s[W], f[W];
#pragma unroll
            SMC_EACH {
                act[w] = i0 + 64 * w + lane < m;
                const int it = it0 + (act[w] ? i0 + 64 * w + lane : 0);
                p[w] = (int)(((float)it + 0.5f) * inv);
                c[w] = 2 * (it - p[w] * np);
                const int o = p[w] * d + c[w];
                two[w] = c[w] + 1 < d && o + 1 < lim;
                const double *sl = slot(it);
                v1[w] = sl[0];
                w1[w] = sl[1];
                x0[w] = x1[w] = 0.0;
                if (!kInit) {
                    if (v2) {
                        const f64x2r v = *(decltype(vec_of(xb)))(xb + o);
                        x0[w] = v[0];
                        x1[w] = v[1];
                    } else {
                        x0[w] = xb[o];
                        x1[w] = xb[two[w] ? o + 1 : o];
                    }
                }
            }
            asm volatile("" ::: "memory");  // all requested before the first use
#pragma unroll
            SMC_EACH s[w] = v1[w] * v1[w] + w1[w] * w1[w];
            if (__any(!(s[0] > 0.0 && s[1] > 0.0))) {  // a pair of (0, 0): any value in range
#pragma unroll
                SMC_EACH s[w] = s[w] > 0.0 ? s[w] : 0.25;
            }
            det_log_w<W>(s, f);
#pragma unroll
            SMC_EACH f[w] = -2.0 * f[w];
            det_div_w<W>(f, s, f);
            det_sqrt_w<W>(f, f);
#pragma unroll
            SMC_EACH {
                if (!act[w]) continue;
                const double z0 = v1[w] * f[w], z1 = w1[w] * f[w];
                if (kInit) put(p[w], c[w], two[w], v2, g.mean + g.sd * z0, g.mean + g.sd * z1);
                else put(p[w], c[w], two[w], v2, x0[w] + g.sd * z0, x1[w] + g.sd * z1);
            }
            asm volatile("" ::: "memory");
        }
        __builtin_amdgcn_wave_barrier();  // the slots are free for the next block
    }
}

}  // namespace smc
