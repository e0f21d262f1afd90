// Redistribute (Alg 5 semantics) as a load-balanced expand.
//
// With A_j = (number of output rows taken from sources 0..j), output row p
// comes from anc(p) = #{j : A_j <= p}, so the ancestors are non-decreasing and
// the output order is exactly that of the sequential redistribute.  Copies per
// source range from 0 to N, so a source-parallel copy is unbalanced; instead
// the merge of the two sorted sequences (A_j + j over sources, p over outputs)
// is cut into equal segments of up to kSegLen merge steps (merge path).  Every
// workgroup owns one segment: a few sources and a few outputs, never more than
// the segment's length in total, whatever the weights.
//
// A_j is computed from the fixed-point prefix as floor((N S_j + U) / S), or is
// the prefix of caller-supplied counts, or j + 1 when the ESS rule decided not
// to resample.  A prefix value is the scan's tile-local value plus the offset
// of its tile.  The segment boundaries are found by a 64-ary search run by one
// wavefront; the test A_j + j < k is evaluated in FP64 and, next to equality, as
// N S_j + U < (k - j) S in 128-bit integers (no division).  Inside a segment
// the outputs find their sources without a search: each source with copies
// marks its first output, and a max-scan over the outputs carries the marks.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "../../include/smc.h"
#include "afun.hpp"
#include "common.hpp"
#include "det.hpp"
#include "kernels.hpp"
#include "segment.hpp"

namespace smc {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

template <int VEC>
struct VecT;
template <>
struct VecT<16> {
    typedef u32x4 T;
};
template <>
struct VecT<8> {
    typedef u32x2 T;
};
template <>
struct VecT<4> {
    typedef unsigned T;
};

// Which accesses at a segment's end go past the caches where the others do.
enum class Tail { kCached, kCachedLoad, kStream };

// Copies np rows [p0, p0 + np) of dst from rows sAnc[] of src, VEC bytes per
// lane access; consecutive lanes write consecutive addresses.  A thread's
// chunks are 256 apart, so its (row, column) moves by a constant step and one
// carry (a division per chunk, for rows that are no power of two, cost as much
// as the copy).
// kNtStore: the stores are non-temporal: a large new population is not read
// again by this call, and keeping it out of the caches spares the next
// resample the write-back of a cache full of dirty rows (about 5 us per call
// at N = 2^24 on MI355X).  One that the caches hold is written through them.
// kNtLoad: the source rows are read non-temporally too.  A segment whose
// outputs are mostly distinct sources reads each line about once; streaming
// those lines past the caches measured 48 us faster per call at N = 2^24,
// s = 0.5 (HBM read requests are whole 128-byte lines either way).  Where a
// few sources fill many outputs (heavy degeneracy) the cached reads are
// faster, the same lines serving the whole segment.
// kTail: what of that holds for the rows at the end of the segment, past the last
// whole round of loads (copy_streamed).
// kPow2: a row's chunks are a power of two up to 256, so a thread's column is
// fixed.
template <int VEC, bool kPow2, bool kNtLoad, bool kNtStore, Tail kTail>
__device__ inline void copy_chunks(const unsigned char *__restrict__ src,
                                   unsigned char *__restrict__ dst, int row_bytes, int cpr,
                                   const unsigned *sAnc, i64 p0, int total)
{
    typedef typename VecT<VEC>::T V;
    const int dr = kExpandThreads / cpr, dc = kExpandThreads - dr * cpr;
    int r = (int)threadIdx.x / cpr, col = (int)threadIdx.x - r * cpr;
    constexpr int U = VEC == 4 ? 8 : 4;  // loads in flight a thread
    V *d = reinterpret_cast<V *>(dst + p0 * (i64)row_bytes);
    auto load = [&](auto nt) {  // the chunk at (r, col), then on to the thread's next
        const V *sp = reinterpret_cast<const V *>(src + (i64)sAnc[r] * row_bytes) + col;
        const V v = decltype(nt)::value ? __builtin_nontemporal_load(sp) : *sp;
        r += dr;
        if (!kPow2) {
            col += dc;
            if (col >= cpr) {
                col -= cpr;
                ++r;
            }
        }
        return v;
    };
    auto store = [&](const V &v, int c, auto nt) {
        if (decltype(nt)::value) __builtin_nontemporal_store(v, d + c);
        else d[c] = v;
    };
    int c = threadIdx.x;
    for (; c + (U - 1) * kExpandThreads < total; c += U * kExpandThreads) {
        V v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = load(std::bool_constant<kNtLoad>());
#pragma unroll
        for (int u = 0; u < U; ++u)
            store(v[u], c + u * kExpandThreads, std::bool_constant<kNtStore>());
    }
    for (; c < total; c += kExpandThreads)
        store(load(std::bool_constant<kNtLoad && kTail == Tail::kStream>()), c,
              std::bool_constant<kNtStore && kTail != Tail::kCached>());
}

// Rows of at least 16 bytes whose size or address is no multiple of 16: 16-byte
// accesses at 4-byte alignment (which the memory pipeline takes), the last
// one of a row moved back to end with it, so that it repeats a few bytes of the
// one before.  Rows of 28 bytes then move in two accesses instead of seven (1000003
// of them, with their segments: 22 us before, 17 now).
typedef u32x4 u32x4_a4 __attribute__((aligned(4)));

template <bool kNtLoad, bool kNtStore>
__device__ inline void copy_ragged(const unsigned char *__restrict__ src,
                                   unsigned char *__restrict__ dst, int row_bytes,
                                   const unsigned *sAnc, i64 p0, int np)
{
    const int cpr = (row_bytes + 15) >> 4, total = np * cpr;
    const int dr = kExpandThreads / cpr, dc = kExpandThreads - dr * cpr;
    int r = (int)threadIdx.x / cpr, col = (int)threadIdx.x - r * cpr;
    constexpr int U = 4;
    unsigned char *d = dst + p0 * (i64)row_bytes;
    auto next = [&](int &row, int &off) {
        row = r;
        off = 16 * col < row_bytes - 16 ? 16 * col : row_bytes - 16;
        r += dr;
        col += dc;
        if (col >= cpr) {
            col -= cpr;
            ++r;
        }
    };
    auto load = [&](int row, int off) -> u32x4 {
        const u32x4_a4 *sp =
            reinterpret_cast<const u32x4_a4 *>(src + (i64)sAnc[row] * row_bytes + off);
        if (kNtLoad) return __builtin_nontemporal_load(sp);
        return *sp;
    };
    auto store = [&](const u32x4 &v, int row, int off) {
        u32x4_a4 *dp = reinterpret_cast<u32x4_a4 *>(d + (i64)row * row_bytes + off);
        if (kNtStore) __builtin_nontemporal_store(v, dp);
        else *dp = v;
    };
    int c = threadIdx.x;
    for (; c + (U - 1) * kExpandThreads < total; c += U * kExpandThreads) {
        u32x4 v[U];
        int row[U], off[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            next(row[u], off[u]);
            v[u] = load(row[u], off[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) store(v[u], row[u], off[u]);
    }
    for (; c < total; c += kExpandThreads) {
        int row, off;
        next(row, off);
        store(load(row, off), row, off);
    }
}

template <int VEC, bool kNtLoad, bool kNtStore, Tail kTail>
__device__ inline void copy_rows(const unsigned char *__restrict__ src,
                                 unsigned char *__restrict__ dst, int row_bytes,
                                 const unsigned *sAnc, i64 p0, int np)
{
    const int cpr = row_bytes / VEC;
    if ((cpr & (cpr - 1)) == 0 && cpr <= kExpandThreads)
        copy_chunks<VEC, true, kNtLoad, kNtStore, kTail>(src, dst, row_bytes, cpr, sAnc, p0,
                                                         np * cpr);
    else
        copy_chunks<VEC, false, kNtLoad, kNtStore, kTail>(src, dst, row_bytes, cpr, sAnc, p0,
                                                          np * cpr);
}

struct ExpandArgs {
    i64 n;
    const u64 *pref;
    const u64 *pref64;
    const u64 *tpre;
    const Ctrl *ctrl;
    int tsh, count_mode;
    const unsigned char *x;
    unsigned char *xo;
    int row_bytes;
    const unsigned char *aux;  // 8-byte side rows (a sampler's cached log-target), nullable
    unsigned char *auxo;
    i64 *nc_out;
    i64 *anc_out;
    ExpandMode mode;
    double *logw;       // a resampling iteration's weights, set to `reset` (nullable) ...
    double reset;
    unsigned *uniform;  // ... or marked uniform here instead (lazy reset, nullable)
    int stream;         // the new rows are written past the caches
};

// The rows at a segment's end lie in lines that the next segment's workgroup reads and
// writes at about the same time, so both go through the caches.  Streamed, they cost up
// to 9 % of a redistribution of rows of 32 to 96 bytes (rows of 32 bytes, s = 2,
// N = 2^23: 110 us streamed, 104 read through the caches, 103 written through them
// too).  That ends where such rows no longer share the 256 MB memory-side cache with the
// prefix and the counts and ancestors that the call writes.  From two fifths of it on
// (kTailStoreBytes) writing past the caches is faster (the same rows, no counts:
// N = 12 x 10^6 138 us both ways, 15 x 10^6 178 cached and 171 streamed, 2^24 203 and
// 190; with counts, N = 10^7: 164 and 150), and where they fill it (kTailLoadBytes)
// reading past them too (no counts, N = 2^25: 421 us and 413; resampling and rows of 64
// bytes with counts, N = 2^24: 454 and 442).
template <int VEC, int SEG>
__device__ inline void copy_streamed(const ExpandArgs &a, bool distinct, const unsigned *sAnc,
                                     i64 p0, int np)
{
    auto copy = [&](auto nt, auto tail) {
        copy_rows<VEC, decltype(nt)::value, true, decltype(tail)::value>(a.x, a.xo, a.row_bytes,
                                                                         sAnc, p0, np);
    };
    const std::bool_constant<true> yes;
    const std::bool_constant<false> no;
    const i64 kept = 8 * a.n * (1 + (a.nc_out ? 1 : 0) + (a.anc_out ? 1 : 0));
    if (SEG < kSegLen || kept < kTailStoreBytes) {
        if (distinct) copy(yes, std::integral_constant<Tail, Tail::kCached>());
        else copy(no, std::integral_constant<Tail, Tail::kCached>());
    } else if (!distinct) {
        copy(no, std::integral_constant<Tail, Tail::kCachedLoad>());
    } else if (kept < kTailLoadBytes) {
        copy(yes, std::integral_constant<Tail, Tail::kCachedLoad>());
    } else {
        copy(yes, std::integral_constant<Tail, Tail::kStream>());
    }
}

// Bound by HBM for large rows and populations (N = 2^24: 340 us for rows of 64
// bytes, 351 with A in 128-bit integers; 127 to 133 for rows of 8 with the weights'
// reset, 131 and 21 as two passes), below by the latency of its four phases (search,
// A, marks, copy; 5.8 us at N = 1000).
// SEG: merge steps of one workgroup.
// kRagged: rows for copy_ragged (VEC does not matter then).
template <int VEC, int SEG, bool kRagged>
__global__ __launch_bounds__(kExpandThreads) void k_expand(ExpandArgs a)
{
    __shared__ SegLds<SEG> s_seg;
    unsigned *const sAnc = s_seg.anc;
    const int tid = threadIdx.x;
    AFun f;
    if (!make_afun(a.ctrl, a.pref, a.tpre, a.tsh, a.n, a.count_mode, f,
                   blockIdx.x == 0 && tid == 0)) {
        // an iteration that found an error resamples nothing: its proposal
        // still has to reach the caller's array
        if (a.mode != ExpandMode::kForward) return;
        f.mode = 0;
    }
    if (a.mode == ExpandMode::kIfResampled && f.mode == 0) return;

    const Segment g = segment_cut<SEG>(f, a.pref64, s_seg);
    const i64 p0 = g.p0;
    const int ns = g.ns, np = g.np;

    // Alg 4 reset of the outputs this segment owns (a pass of its own took 21 us
    // and a launch at N = 2^24)
    if (f.mode == 1 && a.logw) {
        if (a.uniform) {
            if (blockIdx.x == 0 && tid == 0) *a.uniform = 1u;
        } else {
            for (int r = tid; r < np; r += kExpandThreads) a.logw[p0 + r] = a.reset;
        }
    }

    // the longest segments take several trips over their sources, each waiting for its
    // prefix values if they are requested one at a time (rows of 32 bytes, s = 0.5,
    // N = 2^23: 112 us, 107 now); the shorter ones, one or two trips, lose by it
    segment_map<SEG, SEG == kSegLen ? 4 : 1>(f, g, s_seg);
    if (a.nc_out)
        for (int i = tid; i < ns; i += kExpandThreads)
            a.nc_out[g.j0 + i] = (i64)s_seg.A[i + 1] - (i64)s_seg.A[i];
    if (a.anc_out)
        for (int r = tid; r < np; r += kExpandThreads) a.anc_out[p0 + r] = (i64)sAnc[r];
    const bool distinct = np < 2 * ns;  // fewer than two outputs per source in this segment
    if constexpr (kRagged) {
        if (a.stream && distinct)
            copy_ragged<true, true>(a.x, a.xo, a.row_bytes, sAnc, p0, np);
        else if (a.stream)
            copy_ragged<false, true>(a.x, a.xo, a.row_bytes, sAnc, p0, np);
        else
            copy_ragged<false, false>(a.x, a.xo, a.row_bytes, sAnc, p0, np);
    } else if (a.stream) {
        copy_streamed<VEC, SEG>(a, distinct, sAnc, p0, np);
    } else {
        copy_rows<VEC, false, false, Tail::kCached>(a.x, a.xo, a.row_bytes, sAnc, p0, np);
    }
    if (a.aux) copy_rows<8, false, false, Tail::kCached>(a.aux, a.auxo, 8, sAnc, p0, np);
}

template <int VEC, bool kRagged = false>
static void launch_expand_seg(int seg, int64_t n, hipStream_t s, const ExpandArgs &a)
{
    const dim3 g((unsigned)((2 * n + seg - 1) / seg)), b(kExpandThreads);
    switch (seg) {
    case 256: hipLaunchKernelGGL((k_expand<VEC, 256, kRagged>), g, b, 0, s, a); break;
    case 512: hipLaunchKernelGGL((k_expand<VEC, 512, kRagged>), g, b, 0, s, a); break;
    case 1024: hipLaunchKernelGGL((k_expand<VEC, 1024, kRagged>), g, b, 0, s, a); break;
    default: hipLaunchKernelGGL((k_expand<VEC, kSegLen, kRagged>), g, b, 0, s, a); break;
    }
}

hipError_t launch_expand(const Work &w, int64_t n, int count_mode, const void *x, void *x_out,
                         int row_bytes, hipStream_t s, const ExpandOut &o)
{
    ExpandArgs a;
    a.n = n;
    a.pref = w.pref;
    a.pref64 = w.pref64;
    a.tpre = w.tsum;
    a.ctrl = w.ctrl;
    a.tsh = w.tile_shift;
    a.count_mode = count_mode;
    a.x = reinterpret_cast<const unsigned char *>(x);
    a.xo = reinterpret_cast<unsigned char *>(x_out);
    a.row_bytes = row_bytes;
    a.aux = reinterpret_cast<const unsigned char *>(o.aux);
    a.auxo = reinterpret_cast<unsigned char *>(o.aux_out);
    a.nc_out = reinterpret_cast<i64 *>(o.ncopies);
    a.anc_out = reinterpret_cast<i64 *>(o.anc);
    a.mode = o.mode;
    a.logw = o.logw;
    a.reset = o.reset;
    a.uniform = o.uniform;
    a.stream = n * (int64_t)row_bytes >= kStreamBytes;
    const uintptr_t al = (uintptr_t)x | (uintptr_t)x_out | (uintptr_t)row_bytes;
    const int seg = expand_seg_len(n);
    if ((al & 15) == 0) launch_expand_seg<16>(seg, n, s, a);
    else if (row_bytes >= 16) launch_expand_seg<16, true>(seg, n, s, a);
    else if ((al & 7) == 0) launch_expand_seg<8>(seg, n, s, a);
    else launch_expand_seg<4>(seg, n, s, a);
    return hipGetLastError();
}

// ncopies_j = A_j - A_{j-1} for every source.  A thread takes four consecutive
// sources and the A before them from its neighbour lane; only the first lane
// of a wavefront evaluates that one itself (from the tile's offset where a
// tile begins).  16 bytes a source, prefix in and count out: bound by HBM.
// With one source a thread, A evaluated twice and in 128-bit integers each
// time, the pass took 79 us at N = 2^24; 48 now.
constexpr int kNcItems = 4;
typedef u64 u64x2_t __attribute__((ext_vector_type(2)));

__global__ __launch_bounds__(256) void k_ncopies(const Ctrl *ctrl, const u64 *pref,
                                                 const u64 *tpre, int tsh, i64 n, int count_mode,
                                                 int vec, i64 *nc)
{
    AFun f;
    if (!make_afun(ctrl, pref, tpre, tsh, n, count_mode, f, false)) return;
    const int lane = threadIdx.x & 63;
    const i64 step = (i64)gridDim.x * 256 * kNcItems;
    // the trip count is uniform over a wavefront (its lanes exchange A)
    for (i64 w0 = ((i64)blockIdx.x * 256 + (threadIdx.x - lane)) * kNcItems; w0 < n; w0 += step) {
        const i64 j0 = w0 + lane * kNcItems;
        u64 s[kNcItems];
        if (f.mode == 0) {
            for (int e = 0; e < kNcItems; ++e) s[e] = 0;
        } else {
            const u64 off = f.tpre[w0 >> f.tsh];  // a wavefront's run lies in one tile
            if (j0 + kNcItems <= n) {
#pragma unroll
                for (int e = 0; e < kNcItems; e += 2) {
                    const u64x2_t v = *reinterpret_cast<const u64x2_t *>(pref + j0 + e);
                    s[e] = v.x + off;
                    s[e + 1] = v.y + off;
                }
            } else {
#pragma unroll
                for (int e = 0; e < kNcItems; ++e) s[e] = j0 + e < n ? pref[j0 + e] + off : 0;
            }
        }
        unsigned a[kNcItems];
#pragma unroll
        for (int e = 0; e < kNcItems; ++e) a[e] = f.A_of(j0 + e, s[e]);
        unsigned prev = (unsigned)__shfl_up((int)a[kNcItems - 1], 1, 64);
        if (lane == 0) {
            prev = 0;
            if (w0 > 0) {
                u64 sp = 0;
                if (f.mode)
                    sp = f.tpre[w0 >> f.tsh] +
                         ((w0 & ((1ll << f.tsh) - 1)) ? pref[w0 - 1] : 0ull);
                prev = f.A_of(w0 - 1, sp);
            }
        }
        i64 c[kNcItems];
#pragma unroll
        for (int e = 0; e < kNcItems; ++e) {
            c[e] = (i64)a[e] - (i64)prev;
            prev = a[e];
        }
        if (vec && j0 + kNcItems <= n) {
#pragma unroll
            for (int e = 0; e < kNcItems; e += 2)
                __builtin_nontemporal_store(u64x2_t{(u64)c[e], (u64)c[e + 1]},
                                            reinterpret_cast<u64x2_t *>(nc + j0 + e));
        } else {
#pragma unroll
            for (int e = 0; e < kNcItems; ++e)
                if (j0 + e < n) nc[j0 + e] = c[e];
        }
    }
}
static_assert((1 << kTileShiftSmall) % (64 * kNcItems) == 0, "a wavefront's run lies in one tile");

hipError_t launch_ncopies(const Work &w, int64_t n, int count_mode, int64_t *ncopies,
                          hipStream_t s)
{
    int64_t blocks = (n + 256 * kNcItems - 1) / (256 * kNcItems);
    blocks = blocks > 4096 ? 4096 : blocks;
    hipLaunchKernelGGL(k_ncopies, dim3((unsigned)blocks), dim3(256), 0, s, w.ctrl, w.pref, w.tsum,
                       w.tile_shift, (i64)n, count_mode, ((uintptr_t)ncopies & 15) == 0,
                       reinterpret_cast<i64 *>(ncopies));
    return hipGetLastError();
}

}  // namespace smc
