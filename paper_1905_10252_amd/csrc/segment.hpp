// One segment of the merge path between the sources (A_j + j) and the outputs
// (p): its sources, its outputs, and for each output its source.  A workgroup
// of kExpandThreads calls these; the redistribution and the particle filter's
// fused iteration work on top of them.
#pragma once

#include "afun.hpp"
#include "common.hpp"
#include "kernels.hpp"

namespace smc {

// First index in [lo, hi) where a predicate that is true on a prefix turns
// false (hi if none), by rounds of 64 probes, one per lane.
template <class P>
__device__ inline i64 wave_first_false(const P &pred, i64 lo, i64 hi)
{
    const int lane = threadIdx.x & 63;
    while (hi > lo) {
        const i64 len = hi - lo;
        const i64 stride = (len + 63) / 64;
        const i64 pos = lo + (i64)lane * stride;
        const bool t = pos < hi ? pred(pos) : false;
        const int c = __popcll(__ballot(t));
        if (c == 0) {
            hi = lo;
            break;
        }
        const i64 nlo = lo + (i64)(c - 1) * stride + 1;
        i64 nhi = lo + (i64)c * stride;
        if (nhi > hi) nhi = hi;
        lo = nlo;
        hi = nhi;
    }
    return lo;
}

// j(k) = #{j : A_j + j < k}, the number of sources consumed after k merge
// steps, known to lie in [lo, hi].  The test is monotone in j, so it is first
// searched on the sampled prefix values S_{64g+63} (a small array that stays
// in cache), then among the 64 consecutive sources of one group.
__device__ inline i64 wave_search(const AFun &f, const u64 *pref64, i64 k, i64 lo, i64 hi)
{
    if (f.mode == 0) {
        auto p = [&](i64 j) { return f.pred(j, k); };
        return wave_first_false(p, lo, hi);
    }
    const i64 G = f.n >> 6;  // full groups, each with a sample
    const i64 glo = lo >> 6;
    i64 ghi = (hi >> 6) + 1;
    ghi = ghi < G ? ghi : G;
    i64 g = glo;
    if (ghi > glo) {
        auto ps = [&](i64 gg) {
            return f.pred_at(gg * 64 + 63, pref64[gg] + f.tpre[gg >> (f.tsh - 6)], k);
        };
        g = wave_first_false(ps, glo, ghi);
    }
    i64 lo2 = g * 64 > lo ? g * 64 : lo;
    lo2 = lo2 < hi ? lo2 : hi;
    i64 hi2 = g * 64 + 64 < hi ? g * 64 + 64 : hi;
    hi2 = hi2 > lo2 ? hi2 : lo2;
    auto p = [&](i64 j) { return f.pred(j, k); };
    return wave_first_false(p, lo2, hi2);
}

struct Segment {
    i64 j0, p0;  // first source, first output
    int ns, np;
};

template <int SEG>
struct SegLds {
    unsigned A[SEG + 1];
    unsigned anc[SEG] __attribute__((aligned(16)));
    i64 j[2];
    unsigned wmax[kExpandThreads / 64];
};

// The segment of this workgroup (one barrier).
template <int SEG>
__device__ inline Segment segment_cut(const AFun &f, const u64 *pref64, SegLds<SEG> &L)
{
    const int tid = threadIdx.x, wid = tid >> 6;
    const i64 n = f.n;
    const i64 k0 = (i64)blockIdx.x * SEG;
    const i64 k1 = (k0 + SEG < 2 * n) ? k0 + SEG : 2 * n;
    if (wid < 2) {
        const i64 k = wid == 0 ? k0 : k1;
        const i64 lo = k - n > 0 ? k - n : 0;
        const i64 hi = k < n ? k : n;
        const i64 j = wave_search(f, pref64, k, lo, hi);
        if ((tid & 63) == 0) L.j[wid] = j;
    }
    __syncthreads();
    const i64 j0 = L.j[0], j1 = L.j[1];
    Segment g;
    g.j0 = j0;
    g.p0 = k0 - j0;
    g.ns = (int)(j1 - j0);
    g.np = (int)((k1 - j1) - g.p0);
    return g;
}

// Into L.A: A of the sources before, between and in the segment; into L.anc: the
// source of each output of the segment (any valid one past np).  U prefix values
// are requested at a time.
template <int SEG, int U = 1>
__device__ inline void segment_map(const AFun &f, const Segment &g, SegLds<SEG> &L)
{
    unsigned *const sA = L.A, *const sAnc = L.anc;
    const int tid = threadIdx.x, wid = tid >> 6, ns = g.ns, np = g.np;
    const i64 n = f.n, j0 = g.j0;
    // In 32 bits: sources, outputs and A are below 2^31.
    const unsigned p0u = (unsigned)g.p0, j0u = (unsigned)j0;
    if (f.mode == 0) {
        for (int i = tid; i <= ns; i += kExpandThreads) sA[i] = j0u + (unsigned)i;
    } else {
        // sA[i] is A of source j0 - 1 + i
        const int skip = j0 == 0 ? 1 : 0;  // A before the first source is 0
        const i64 jb = j0 - 1 + skip;
        if (skip && tid == 0) sA[0] = 0u;
        const int last = ns - skip;
        if constexpr (U == 1) {
            for (int i = tid; i <= last; i += kExpandThreads)
                sA[i + skip] = f.A_of(0, f.at(jb + i));
        } else {
            for (int i0 = tid; i0 <= last; i0 += U * kExpandThreads) {
                u64 s[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = i0 + u * kExpandThreads;
                    s[u] = f.at(jb + (i <= last ? i : i0));
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = i0 + u * kExpandThreads;
                    if (i <= last) sA[i + skip] = f.A_of(0, s[u]);
                }
            }
        }
    }
    for (int r = tid; r < np; r += kExpandThreads) sAnc[r] = 0u;
    __syncthreads();
    // Output p comes from local source t, the first with sA[1 + t] > p, so
    // sA[t] <= p < sA[1 + t] (sA[0] <= p0 by the merge-path cut).  Each source
    // with copies marks the first of its outputs inside the segment with
    // t + 1; an inclusive max-scan over the outputs carries every mark over
    // the rest of its source's outputs.  Local source ns (source j1) owns
    // whatever follows sA[ns].  Marks land on distinct outputs (sources with
    // copies start at distinct outputs) and output p0 always holds one.
    for (int t = tid; t <= ns; t += kExpandThreads) {
        const unsigned lo = sA[t], hi = t < ns ? sA[t + 1] : 0xFFFFFFFFu;
        if (hi > lo && hi > p0u) {
            const unsigned st = lo > p0u ? lo - p0u : 0u;
            if (st < (unsigned)np) sAnc[st] = (unsigned)(t + 1);
        }
    }
    __syncthreads();
    constexpr int E = SEG / kExpandThreads;  // outputs per thread, contiguous
    static_assert(E >= 1 && E * kExpandThreads == SEG, "whole outputs a thread");
    const int lane = tid & 63;
    // entries past np are stale; they reach only positions past np
    unsigned v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = sAnc[tid * E + e];
#pragma unroll
    for (int e = 1; e < E; ++e) v[e] = v[e] > v[e - 1] ? v[e] : v[e - 1];
    const unsigned incl = wave_scan_max_u32(v[E - 1]);
    if (lane == 63) L.wmax[wid] = incl;
    unsigned carry = (unsigned)__shfl_up((int)incl, 1, 64);
    carry = lane ? carry : 0u;
    __syncthreads();
    for (int w = 0; w < wid; ++w) carry = L.wmax[w] > carry ? L.wmax[w] : carry;
    const unsigned last = (unsigned)n - 1u;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        unsigned anc = j0u + (v[e] > carry ? v[e] : carry) - 1u;
        anc = anc < last ? anc : last;  // entries past np: any valid source
        sAnc[tid * E + e] = anc;
    }
    __syncthreads();
}

}  // namespace smc
