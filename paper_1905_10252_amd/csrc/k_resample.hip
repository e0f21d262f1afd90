// Resampling kernels of Alg 4 (minimum variance resampling):
//   k_max          exact FP64 max of the log-weights (the stability shift of
//                  eq. normalise) and non-finite detection.
//   k_fold         combines the max slots, records the error of the call
//                  (used where no scan follows the max pass).
//   k_scan<true>   one pass over the log-weights: 64-bit fixed-point weights
//                  q_i = min(2^K, floor(2^K det_exp(l_i - m))), FP64 sums for
//                  log-sum-exp and ESS (eq. normalise, eq. neff), the exact
//                  sum of q_i^2, and the prefix sums of q within each tile of
//                  4096 or 1024 weights, plus the tile's total.
//   k_scan<false>  the same tile scan over caller-supplied int64 ncopies.
//   k_decide       the exclusive prefix of the tile totals (so that the
//                  inclusive prefix S_j of the Cumulative Sum of MVR is the
//                  tile-local value plus its tile's offset), the error of the
//                  call, the exact integer ESS decision (resample when
//                  ESS < N*, Alg 2), the systematic offset U = floor(r S / 2^64),
//                  log Z and the FP64 ESS from the tile partials; clears the
//                  other parity's max slots.
//   k_tile_prefix  the tile offsets alone, for caller-supplied counts.
// No tile waits on another: the scan is split into tile-local prefixes and
// one small scan over the tile totals, so no kernel here spins, and none uses
// a device-wide fence or a contended atomic.
// Every 64th tile-local prefix value is also written to a sample array, a
// coarse index for the merge-path searches of the expand kernel.
#include <hip/hip_runtime.h>

#include "../../include/smc.h"
#include "afun.hpp"
#include "common.hpp"
#include "decide.hpp"
#include "det.hpp"
#include "kernels.hpp"
#include "stats.hpp"
#include "reduce.hpp"

namespace smc {

// ------------------------------------------------------------- control init
__global__ void k_init_ctrl(Ctrl *ctrl, u64 *slots)
{
    u64 *p = reinterpret_cast<u64 *>(ctrl);
    for (int i = threadIdx.x; i < (int)(sizeof(Ctrl) / 8); i += blockDim.x) p[i] = 0;
    for (int i = threadIdx.x; i < kSlotWords; i += blockDim.x) slots[i] = 0;
}

hipError_t launch_init_ctrl(const Work &w, hipStream_t s)
{
    static_assert(sizeof(Ctrl) % 8 == 0, "ctrl size");
    hipLaunchKernelGGL(k_init_ctrl, dim3(1), dim3(256), 0, s, w.ctrl, w.slots);
    return hipGetLastError();
}

// ------------------------------------------------------------- exact max
// Grid-stride share per block, four 16-byte loads in flight per thread; each
// block publishes its max order key into the slots of this call's parity.
// The loads are non-temporal, here and in the scan: the weights are read once
// by each pass, and streaming them past the caches measured faster on MI355X
// than keeping them (N = 2^24: about 10 us less for the resample call).
typedef double f64x2_t __attribute__((ext_vector_type(2)));

__global__ __launch_bounds__(256) void k_max(const double *__restrict__ lw, i64 n, int vec2,
                                             u64 *slots_p)
{
    // two 16-byte loads in flight per thread: 1-2 us faster per call at
    // N = 2^24 than four or eight (and than one)
    constexpr int U = 2;
    const int tid = threadIdx.x;
    const i64 gtid = (i64)blockIdx.x * 256 + tid, gsz = (i64)gridDim.x * 256;

    u64 key = 0;
    unsigned bad = 0;
    const double ninf = -__builtin_huge_val();
    auto take = [&](double v) {
        bad |= (v != v) | (v == __builtin_huge_val());
        const u64 k = okey(v);
        key = k > key ? k : key;
    };
    if (vec2) {
        const i64 npair = n >> 1;
        const f64x2_t *lw2 = reinterpret_cast<const f64x2_t *>(lw);
        for (i64 i = gtid; i < npair; i += U * gsz) {
            f64x2_t v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const i64 j = i + u * gsz;
                v[u] = j < npair ? __builtin_nontemporal_load(lw2 + j) : f64x2_t{ninf, ninf};
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                take(v[u].x);
                take(v[u].y);
            }
        }
        if ((n & 1) && gtid == 0) take(lw[n - 1]);
    } else {
        for (i64 i = gtid; i < n; i += gsz) take(lw[i]);
    }
    const u64 bk = block_max_key(key, bad);
    slot_publish(slots_p, bk, bad);
}

hipError_t launch_max(const Work &w, const double *lw, int64_t n, int par, hipStream_t s)
{
    const int vec2 = ((uintptr_t)lw & 15) == 0;
    hipLaunchKernelGGL(k_max, dim3(max_blocks_of(n)), dim3(256), 0, s, lw, (i64)n, vec2,
                       w.slots + (par & 1) * kSlots * kSlotStride);
    return hipGetLastError();
}

// One wavefront: max over the 64 slots of parity par, the call's error
// (NaN or +inf seen: non-finite; max = -inf: every weight zero), and a clear
// of the other parity's slots for the next call.
__global__ __launch_bounds__(64) void k_fold(u64 *slots, int par, Ctrl *ctrl)
{
    const int lane = threadIdx.x;
    u64 *cur = slots + (par & 1) * kSlots * kSlotStride;
    u64 *nxt = slots + ((par & 1) ^ 1) * kSlots * kSlotStride;
    const u64 key = wave_max_u64(cur[lane * kSlotStride]);
    const unsigned bad = wave_or((unsigned)cur[lane * kSlotStride + 1]);
    nxt[lane * kSlotStride] = 0;
    nxt[lane * kSlotStride + 1] = 0;
    if (lane == 0) {
        unsigned err = 0;
        if (bad) err = kErrNonfinite;
        else if (key <= okey(-__builtin_huge_val())) err = kErrDegenerate;
        ctrl->mkey = key;
        ctrl->m = okey_inv(key);
        ctrl->err_call = err;
        if (err && !ctrl->err_latch) ctrl->err_latch = err;
        ctrl->pending = 0;
    }
}

hipError_t launch_fold(const Work &w, int par, hipStream_t s)
{
    hipLaunchKernelGGL(k_fold, dim3(1), dim3(64), 0, s, w.slots, par, w.ctrl);
    return hipGetLastError();
}

// ------------------------------------------------------------ tile scan
// Tile = kScanThreads threads x kItems items; tile t is workgroup t.
// Global loads and stores are coalesced 16-byte accesses over rows of
// 2 kScanThreads elements; an LDS transpose gives each thread kItems
// consecutive items for the sequential part of the scan.  Entry i of the
// transpose sits at slot (i ^ (i >> 5)) & 15 of its 16-entry block (a
// bijection): in both the striped and the per-thread accesses at most two
// lanes of a wave meet on a bank pair, the minimum for 8-byte accesses, with
// no pad words.
// The prefix written is local to the tile; the tile's total goes to tsum[t],
// which the following single-workgroup pass turns into tile offsets.  A
// chained scan (each tile waiting for its predecessors' totals) costs a
// round trip through the memory system per tile in flight; this split costs
// one small pass over 8 bytes per 4096 weights instead.
__host__ __device__ constexpr int kPad(int i) { return (i & ~15) | ((i ^ (i >> 5)) & 15); }
constexpr int kScanWaves = kScanThreads / 64;
constexpr int kScanRow = 2 * kScanThreads;  // elements per striped row

struct ScanArgs {
    const double *lw;   // quantise mode input
    const i64 *nc;      // count mode input
    i64 n;
    int K, vec2;
    Ctrl *ctrl;
    u64 *tsum;          // [n_tiles] tile totals
    TilePart *tpart;
    u64 *out;           // [n] tile-local inclusive prefix
    u64 *out64;         // [n / 64] every 64th tile-local prefix value
    const u64 *slots_p; // max slots of this call's parity (quantise mode)
    unsigned *uniform;  // lazy-reset flag to clear (nullable)
    StatsArgs st;
    int n_st;           // workgroups ahead of the tiles' that form st
};

// Bound by HBM at N = 2^24 (49 us; 62 with the weight quantised by ldexp, floor and
// a conversion, bound by vector issue then), by latency below 2^18 (4 to 5 us).
// Four waves per SIMD: the LDS of a 4096-element tile allows no more.
template <bool kQuant, int kItems, bool kStats = false>
__global__ __launch_bounds__(kScanThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_scan(
    ScanArgs a)
{
    static_assert(kItems % 4 == 0 && 64 % kItems == 0 && kItems <= 16, "scan tile shape");
    constexpr int kTile = kScanThreads * kItems;
    constexpr size_t kLds = kStats && sizeof(StatsLds) > 8 * kTile ? sizeof(StatsLds) : 8 * kTile;
    __shared__ u64 sq[kLds / 8];
    __shared__ u64 s_wsum[kScanWaves];
    __shared__ double s_z[kScanWaves], s_z2[kScanWaves];
    __shared__ u64 s_q2lo[kScanWaves], s_q2hi[kScanWaves];
    __shared__ unsigned s_bad[kScanWaves];

    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const i64 n = a.n;
    if constexpr (kStats) {  // the first workgroups, so that they end with the others
        if ((int)blockIdx.x < a.n_st) {
            if (a.st.cols)
                fold_columns<kScanThreads>(*reinterpret_cast<StatsLds *>(sq), a.st, blockIdx.x);
            else
                filter_stats<kScanThreads>(a.ctrl, a.st.is_part, a.st.nblk, a.st.d, a.st.rec_num,
                                           a.st.est,
                                           reinterpret_cast<smc_resample_info *>(a.st.info));
            return;
        }
    }
    const unsigned tile = blockIdx.x - (kStats ? a.n_st : 0);
    const i64 base = (i64)tile * kTile;
    const bool full = base + kTile <= n;

    double z = 0.0, z2 = 0.0;
    SqSum sq2;
    unsigned bad = 0;
    // striped: a thread's item 2r + h is element base + kScanRow r + 2 tid + h
    if (kQuant) {
        // every wave folds the 64 max slots itself (cached lines; no barrier)
        const double m = okey_inv(wave_max_u64(a.slots_p[lane * kSlotStride]));
        const int K = a.K;
        double v[kItems];
        if (full && a.vec2) {
#pragma unroll
            for (int r = 0; r < kItems / 2; ++r) {
                const f64x2_t t = __builtin_nontemporal_load(
                    reinterpret_cast<const f64x2_t *>(a.lw + base + r * kScanRow + 2 * tid));
                v[2 * r] = t.x;
                v[2 * r + 1] = t.y;
            }
        } else {
#pragma unroll
            for (int e = 0; e < kItems; ++e) {
                const i64 i = base + (e >> 1) * kScanRow + 2 * tid + (e & 1);
                v[e] = i < n ? a.lw[i] : -__builtin_huge_val();
            }
        }
#pragma unroll
        for (int e = 0; e < kItems; e += 4) {
            const double v4[4] = {v[e], v[e + 1], v[e + 2], v[e + 3]};
            u64 q4[4];
            quant_w<4>(v4, m, K, q4, z, z2, sq2);
#pragma unroll
            for (int w = 0; w < 4; ++w)
                sq[kPad(((e + w) >> 1) * kScanRow + 2 * tid + (w & 1))] = q4[w];
            // one group's registers at a time: nothing of it is left for later
            asm volatile("" : "+v"(sq2.ll), "+v"(sq2.hl), "+v"(sq2.hh), "+v"(z), "+v"(z2));
        }
    } else {
        i64 c[kItems];
#pragma unroll
        for (int e = 0; e < kItems; ++e) {
            const i64 i = base + (e >> 1) * kScanRow + 2 * tid + (e & 1);
            c[e] = i < n ? a.nc[i] : 0;
        }
#pragma unroll
        for (int e = 0; e < kItems; ++e) {
            const bool ok = c[e] >= 0 && c[e] <= n;
            bad |= ok ? 0u : 1u;
            sq[kPad((e >> 1) * kScanRow + 2 * tid + (e & 1))] = ok ? (u64)c[e] : 0ull;
        }
    }
    __syncthreads();

    // sequential inclusive scan of this thread's 16 consecutive items
    u64 loc[kItems];
    u64 run = 0;
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        run += sq[kPad(tid * kItems + j)];
        loc[j] = run;
    }
    const u64 incl = wave_incl_scan_u64(run);
    if (lane == 63) s_wsum[wid] = incl;
    // tile partial sums (fixed reduction order: reproducible)
    if (kQuant) {
        z = wave_sum_f64(z);
        z2 = wave_sum_f64(z2);
        const U128 q2 = wave_sum_u128(sq2.total());
        if (lane == 0) {
            s_z[wid] = z;
            s_z2[wid] = z2;
            s_q2lo[wid] = q2.lo;
            s_q2hi[wid] = q2.hi;
        }
    } else {
        bad = wave_or(bad);
        if (lane == 0) s_bad[wid] = bad;
    }
    __syncthreads();
    u64 wpre = 0, agg = 0;
#pragma unroll
    for (int i = 0; i < kScanWaves; ++i) {
        wpre += (i < wid) ? s_wsum[i] : 0;
        agg += s_wsum[i];
    }
    // each thread rewrites only the 16 entries it read above
    const u64 pre = wpre + incl - run;
#pragma unroll
    for (int j = 0; j < kItems; ++j) sq[kPad(tid * kItems + j)] = pre + loc[j];
    // every 64th prefix value (item 64g + 63 is the last item of its thread)
    if (((tid + 1) * kItems) % 64 == 0) {
        const i64 gi = base + tid * kItems + (kItems - 1);
        if (gi < n) a.out64[gi >> 6] = pre + loc[kItems - 1];
    }
    if (tid == 0) {
        if (a.uniform && tile == 0) *a.uniform = 0u;
        a.tsum[tile] = agg;
        if (kQuant) {
            TilePart p;
            double Z = s_z[0], Z2 = s_z2[0];
            U128 t{s_q2lo[0], s_q2hi[0]};
            for (int i = 1; i < kScanWaves; ++i) {
                Z += s_z[i];
                Z2 += s_z2[i];
                t = add128(t, U128{s_q2lo[i], s_q2hi[i]});
            }
            p.Z = Z;
            p.Z2 = Z2;
            p.q2lo = t.lo;
            p.q2hi = t.hi;
            a.tpart[tile] = p;
        } else {
            unsigned b = 0;
            for (int i = 0; i < kScanWaves; ++i) b |= s_bad[i];
            a.tpart[tile].q2lo = b;  // collected by k_tile_prefix
        }
    }
    __syncthreads();
    // the striped addresses are formed again here, not kept since the loads
    int tid2 = 2 * tid;
    asm volatile("" : "+v"(tid2));
    if (full) {
#pragma unroll
        for (int r = 0; r < kItems / 2; ++r) {
            const int s0 = r * kScanRow + tid2;
            ulonglong2 v;
            v.x = sq[kPad(s0)];
            v.y = sq[kPad(s0 + 1)];
            *reinterpret_cast<ulonglong2 *>(a.out + base + s0) = v;
        }
    } else {
#pragma unroll
        for (int e = 0; e < kItems; ++e) {
            const int s0 = (e >> 1) * kScanRow + tid2 + (e & 1);
            if (base + s0 < n) a.out[base + s0] = sq[kPad(s0)];
        }
    }
}

// Exclusive prefix of the tile totals, in place, by one workgroup of 1024
// threads (each a contiguous run of tiles), in two steps around a barrier: the
// thread's total and its scan in the wavefront, then the offsets; the second
// returns the grand total to every thread.  The thread's totals stay in
// registers in between (up to kRun of them).
struct TileOffsets {
    static constexpr int kRun = 4;  // tiles a thread at N = 2^24
    u64 v[kRun], run, incl;
    int per, t0;

    __device__ inline void begin(const u64 *tsum, int n_tiles, u64 *s_w)
    {
        const int tid = threadIdx.x;
        per = (n_tiles + 1023) / 1024;
        t0 = tid * per;
        run = 0;
        if (per <= kRun) {
#pragma unroll
            for (int i = 0; i < kRun; ++i) {
                v[i] = i < per && t0 + i < n_tiles ? tsum[t0 + i] : 0ull;
                run += v[i];
            }
        } else {
            for (int i = 0; i < per; ++i)
                if (t0 + i < n_tiles) run += tsum[t0 + i];
        }
        incl = wave_incl_scan_u64(run);
        if ((tid & 63) == 63) s_w[tid >> 6] = incl;
    }

    __device__ inline u64 finish(u64 *tsum, int n_tiles, const u64 *s_w) const
    {
        const int wid = threadIdx.x >> 6;
        u64 pre = 0, total = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            pre += (i < wid) ? s_w[i] : 0;
            total += s_w[i];
        }
        pre += incl - run;
        if (per <= kRun) {
#pragma unroll
            for (int i = 0; i < kRun; ++i) {
                if (i < per && t0 + i < n_tiles) tsum[t0 + i] = pre;
                pre += v[i];
            }
        } else {
            for (int i = 0; i < per; ++i)
                if (t0 + i < n_tiles) {
                    const u64 x = tsum[t0 + i];
                    tsum[t0 + i] = pre;
                    pre += x;
                }
        }
        return total;
    }
};

// Caller-supplied counts: tile offsets, their total (checked against N by the
// expand) and the tiles' flags for an invalid count; the call's other flags.
__global__ __launch_bounds__(1024) void k_tile_prefix(Ctrl *ctrl, u64 *tsum,
                                                      const TilePart *tpart, int n_tiles)
{
    __shared__ u64 s_w[16];
    TileOffsets to;
    to.begin(tsum, n_tiles, s_w);
    int bad = 0;
    for (int t = threadIdx.x; t < n_tiles; t += 1024) bad |= tpart[t].q2lo != 0;
    bad = __syncthreads_or(bad);
    const u64 total = to.finish(tsum, n_tiles, s_w);
    if (threadIdx.x == 0) {
        ctrl->ctotal = total;
        ctrl->ncopy_bad = bad ? 1u : 0u;
        ctrl->err_call = 0;
        ctrl->pending = 0;
    }
}

// ---------------------------------------------------------------- decision
// One workgroup: tile offsets; tile partials summed in a fixed order
// (reproducible FP64); exact integer decision and offset; with kStats also a
// sampler iteration's estimates, c_t and recycling from the columns folded beside
// the scan (folded here, by one compute unit, 66 columns of 1024 rows took this
// kernel from 5 to 14 us).  Bound by latency, so the
// independent chains (offsets, partials, max slots, columns, the
// state of the recycling) all start at once.
template <bool kStats>
__global__ __launch_bounds__(1024) void k_decide(Ctrl *ctrl, u64 *slots, int par,
                                                 const TilePart *tpart, u64 *tsum,
                                                 int n_tiles, i64 n, int K, u64 r, int mode,
                                                 int ess_num, int ess_den,
                                                 smc_resample_info *info, StatsArgs st)
{
    __shared__ double s_z[16], s_z2[16];
    __shared__ u64 s_lo[16], s_hi[16];
    __shared__ u64 s_w[16];
    __shared__ unsigned s_err;
    __shared__ double s_bc[3];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const RecState rec(ctrl);
    double rec_old = 0.0, sum = 0.0, weights = 1.0;
    if constexpr (kStats) {
        if (tid < 2 * st.d) {
            rec_old = st.rec_num[tid];
            sum = st.cols[2 + tid];
            weights = st.cols[1];
        }
    }
    u64 key = 0;
    unsigned badf = 0;
    if (wid == 0) {
        const u64 *cur = slots + (par & 1) * kSlots * kSlotStride;
        u64 *nxt = slots + ((par & 1) ^ 1) * kSlots * kSlotStride;
        key = cur[lane * kSlotStride];
        badf = (unsigned)cur[lane * kSlotStride + 1];
        nxt[lane * kSlotStride] = 0;
        nxt[lane * kSlotStride + 1] = 0;
    }
    double z = 0.0, z2 = 0.0;
    U128 q2{0, 0};
    constexpr int FU = 4;  // partials in flight per thread; summed in tile order
    for (int t0 = tid; t0 < n_tiles; t0 += 1024 * FU) {
        TilePart p[FU];
#pragma unroll
        for (int u = 0; u < FU; ++u) {
            const int t = t0 + 1024 * u;
            p[u] = t < n_tiles ? tpart[t] : TilePart{0.0, 0.0, 0ull, 0ull};
        }
#pragma unroll
        for (int u = 0; u < FU; ++u) {
            z += p[u].Z;
            z2 += p[u].Z2;
            q2 = add128(q2, U128{p[u].q2lo, p[u].q2hi});
        }
    }
    TileOffsets to;
    to.begin(tsum, n_tiles, s_w);
    z = wave_sum_f64(z);
    z2 = wave_sum_f64(z2);
    q2 = wave_sum_u128(q2);
    if (lane == 0) {
        s_z[wid] = z;
        s_z2[wid] = z2;
        s_lo[wid] = q2.lo;
        s_hi[wid] = q2.hi;
    }
    __syncthreads();
    const u64 S = to.finish(tsum, n_tiles, s_w);
    if (wid == 0) {
        // the 16 wavefronts' partials, one a lane (entries 16.. are the identity)
        const bool in = lane < 16;
        const double Z = wave_sum_f64(in ? s_z[lane & 15] : 0.0);
        const double Z2 = wave_sum_f64(in ? s_z2[lane & 15] : 0.0);
        const U128 Q2 = wave_sum_u128(in ? U128{s_lo[lane & 15], s_hi[lane & 15]} : U128{0, 0});
        key = wave_max_u64(key);
        badf = wave_or(badf);
        if (lane == 0) {
            const Decision dec = decide(key, badf, S, Z, Z2, Q2, n, r, mode, ess_num, ess_den);
            // an iteration whose decision found an error (NaN / +inf weight,
            // all weights zero) leaves c_t, the recycling sums and the
            // estimates as they were, as it stops at the resampling step
            double logc = 0.0;
            if constexpr (kStats) {
                if (!dec.err) {
                    double bc[3];
                    RecNext nx;
                    logc = recycle_step(rec, dec.logZ, bc, nx);
                    store_recycling(nx, logc, dec.logZ, dec.resample, ctrl);
                    for (int i = 0; i < 3; ++i) s_bc[i] = bc[i];
                }
            }
            store_decision(dec, K, logc, ctrl, info);
            s_err = dec.err;
        }
    }
    if constexpr (kStats) {
        __syncthreads();
        if (tid < 2 * st.d && !s_err)
            write_estimate(tid, st.d, sum, weights, rec_old, s_bc, st.rec_num, st.est);
    }
}

hipError_t launch_decide(const Work &w, int par, int64_t n, int K, uint64_t r, int mode,
                         int ess_num, int ess_den, void *info, hipStream_t s,
                         const StatsArgs &st)
{
    auto kern = st.is_part ? k_decide<true> : k_decide<false>;
    hipLaunchKernelGGL(kern, dim3(1), dim3(1024), 0, s, w.ctrl, w.slots, par, w.tpart, w.tsum,
                       w.n_tiles, (i64)n, K, (u64)r, mode, ess_num, ess_den,
                       reinterpret_cast<smc_resample_info *>(info), st);
    return hipGetLastError();
}

// ------------------------------------------------- one-workgroup resampling
// The whole of smc_resample for at most kSmallResample weights in one launch:
// max, fixed-point weights, their prefix, the sums, the decision and the copy
// counts.  Four launches of one or two workgroups each spent 12 us at
// N = 1000, nearly all of it launch and memory latency; here the weights stay
// in registers (kPer consecutive ones a thread, at most 1024 threads) and two
// barriers separate the three phases.  The same integers; the FP64 sums are
// taken in thread order.  The prefix is stored whole (every tile's offset 0)
// for the expand that may follow.  With that expand, N = 1000 of four FP64 values:
// 24.0 us before, 11.2 now.  The line at kSmallResample: the call takes 5.5 us at
// N = 1000, 8.9 at 4096, 12.4 at 6000 and 15.8 at 8192, the separate launches 14.1
// just above.
template <int kPer>
__global__ __launch_bounds__(1024) void k_small_resample(
    const double *__restrict__ lw, i64 n, int K, u64 r, int mode, int ess_num, int ess_den,
    Ctrl *ctrl, u64 *slots_other, u64 *tsum, int n_tiles, u64 *pref, u64 *pref64, i64 *nc,
    smc_resample_info *info)
{
    static_assert(kPer % 4 == 0, "weights in groups of four");
    __shared__ u64 s_key[16], s_wsum[16], s_lo[16], s_hi[16];
    __shared__ unsigned s_bad[16];
    __shared__ double s_z[16], s_z2[16];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, nw = blockDim.x >> 6;
    const int i0 = tid * kPer, ni = (int)n;
    const double ninf = -__builtin_huge_val();
    // the next call's max slots start clear, as after a decision
    if (slots_other && wid == nw - 1) {
        slots_other[lane * kSlotStride] = 0;
        slots_other[lane * kSlotStride + 1] = 0;
    }
    for (int t = tid; t < n_tiles; t += blockDim.x) tsum[t] = 0;
    double v[kPer];
    u64 key = 0;
    unsigned bad = 0;
#pragma unroll
    for (int e = 0; e < kPer; ++e) v[e] = i0 + e < ni ? lw[i0 + e] : ninf;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
        bad |= !(v[e] < __builtin_huge_val());
        const u64 k = okey(v[e]);
        key = k > key ? k : key;
    }
    key = wave_max_u64(key);
    bad = wave_or(bad);
    if (lane == 0) {
        s_key[wid] = key;
        s_bad[wid] = bad;
    }
    __syncthreads();
    key = s_key[0];
    bad = s_bad[0];
    for (int w = 1; w < nw; ++w) {
        key = s_key[w] > key ? s_key[w] : key;
        bad |= s_bad[w];
    }
    const double m = okey_inv(key);
    double z = 0.0, z2 = 0.0;
    SqSum sq;
    u64 loc[kPer], run = 0;
#pragma unroll
    for (int e = 0; e < kPer; e += 4) {
        const double v4[4] = {v[e], v[e + 1], v[e + 2], v[e + 3]};
        u64 q4[4];
        quant_w<4>(v4, m, K, q4, z, z2, sq);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            run += q4[w];
            loc[e + w] = run;
        }
    }
    const u64 incl = wave_incl_scan_u64(run);
    z = wave_sum_f64(z);
    z2 = wave_sum_f64(z2);
    const U128 q2 = wave_sum_u128(sq.total());
    if (lane == 63) s_wsum[wid] = incl;
    if (lane == 0) {
        s_z[wid] = z;
        s_z2[wid] = z2;
        s_lo[wid] = q2.lo;
        s_hi[wid] = q2.hi;
    }
    __syncthreads();
    u64 pre = incl - run, S = 0;
    for (int w = 0; w < nw; ++w) {
        pre += w < wid ? s_wsum[w] : 0ull;
        S += s_wsum[w];
    }
    // every wavefront forms the decision itself: no third barrier
    const bool in = lane < nw;
    const double Z = wave_sum_f64(in ? s_z[lane & 15] : 0.0);
    const double Z2 = wave_sum_f64(in ? s_z2[lane & 15] : 0.0);
    const U128 Q2 = wave_sum_u128(in ? U128{s_lo[lane & 15], s_hi[lane & 15]} : U128{0, 0});
    const Decision dec = decide(key, bad, S, Z, Z2, Q2, n, r, mode, ess_num, ess_den);
    if (tid == 0) store_decision(dec, K, 0.0, ctrl, info);
    AFun f;
    f.n = n;
    f.mode = 0;
    if (dec.resample) f.set_systematic(S, dec.U);
    unsigned prev = i0 > 0 ? f.A_of(i0 - 1, pre) : 0u;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
        if (i0 + e >= ni) break;
        const u64 s = pre + loc[e];
        pref[i0 + e] = s;
        if (((i0 + e) & 63) == 63) pref64[(i0 + e) >> 6] = s;
        if (nc && !dec.err) {
            const unsigned a = f.A_of(i0 + e, s);
            nc[i0 + e] = (i64)(a - prev);
            prev = a;
        }
    }
}

hipError_t launch_small_resample(const Work &w, const double *lw, int64_t n, int K, uint64_t r,
                                 int mode, int ess_num, int ess_den, int par, bool slots,
                                 int64_t *ncopies, void *info, hipStream_t s)
{
    auto kern = n <= 4096 ? k_small_resample<4> : k_small_resample<8>;
    const int64_t per = n <= 4096 ? 4 : 8;
    const int64_t waves = (n + 64 * per - 1) / (64 * per);
    hipLaunchKernelGGL(kern, dim3(1), dim3((unsigned)(64 * waves)), 0, s, lw, (i64)n, K, (u64)r,
                       mode, ess_num, ess_den, w.ctrl,
                       slots ? w.slots + ((par & 1) ^ 1) * kSlots * kSlotStride : (u64 *)nullptr,
                       w.tsum, w.n_tiles, w.pref, w.pref64, reinterpret_cast<i64 *>(ncopies),
                       reinterpret_cast<smc_resample_info *>(info));
    return hipGetLastError();
}

hipError_t launch_quant_scan(const Work &w, const double *lw, int64_t n, int K, int par,
                             hipStream_t s, bool clear_uniform, const StatsArgs &st)
{
    ScanArgs a;
    a.uniform = clear_uniform ? &w.ctrl->uniform : nullptr;
    a.lw = lw;
    a.nc = nullptr;
    a.n = n;
    a.K = K;
    a.vec2 = ((uintptr_t)lw & 15) == 0;
    a.ctrl = w.ctrl;
    a.tsum = w.tsum;
    a.tpart = w.tpart;
    a.out = w.pref;
    a.out64 = w.pref64;
    a.slots_p = w.slots + (par & 1) * kSlots * kSlotStride;
    a.st = st;
    a.n_st = !st.is_part ? 0 : (st.cols ? (1 + 2 * st.d + kScanWaves - 1) / kScanWaves : 1);
    const bool big = w.tile_shift == kTileShift;
    auto kern = a.n_st ? (big ? k_scan<true, 16, true> : k_scan<true, 4, true>)
                       : (big ? k_scan<true, 16> : k_scan<true, 4>);
    hipLaunchKernelGGL(kern, dim3(w.n_tiles + a.n_st), dim3(kScanThreads), 0, s, a);
    return hipGetLastError();
}

// eq. normalise: w_i = exp(l_i - m) / Z with the max and the FP64 sum of
// the last decision (nothing is written when that call found an error).
__global__ __launch_bounds__(256) void k_weights(const Ctrl *ctrl, const double *lw, i64 n,
                                                 double *w)
{
    if (ctrl->err_call) return;
    const double m = ctrl->m, Z = ctrl->Z;
    const i64 gtid = (i64)blockIdx.x * 256 + threadIdx.x, gsz = (i64)gridDim.x * 256;
    for (i64 i = gtid; i < n; i += gsz) {
        // the caller's array need not be the one of that decision: a value far above
        // m gives +inf, a NaN itself
        const double v = lw[i] - m;
        w[i] = (v <= 709.0 ? det_exp(v) : (v != v ? v : __builtin_huge_val())) / Z;
    }
}

hipError_t launch_weights(const Work &w, const double *lw, int64_t n, double *out, hipStream_t s)
{
    int64_t blocks = (n + 255) / 256;
    blocks = blocks > 8192 ? 8192 : blocks;
    hipLaunchKernelGGL(k_weights, dim3((unsigned)blocks), dim3(256), 0, s, w.ctrl, lw, (i64)n, out);
    return hipGetLastError();
}

hipError_t launch_count_scan(const Work &w, const int64_t *ncopies, int64_t n, hipStream_t s)
{
    ScanArgs a;
    a.uniform = nullptr;
    a.lw = nullptr;
    a.nc = reinterpret_cast<const i64 *>(ncopies);
    a.n = n;
    a.K = 0;
    a.vec2 = 0;
    a.ctrl = w.ctrl;
    a.tsum = w.tsum;
    a.tpart = w.tpart;
    a.out = w.pref;
    a.out64 = w.pref64;
    a.slots_p = nullptr;
    auto kern = w.tile_shift == kTileShift ? k_scan<false, 16> : k_scan<false, 4>;
    hipLaunchKernelGGL(kern, dim3(w.n_tiles), dim3(kScanThreads), 0, s, a);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    hipLaunchKernelGGL(k_tile_prefix, dim3(1), dim3(1024), 0, s, w.ctrl, w.tsum, w.tpart,
                       w.n_tiles);
    return hipGetLastError();
}

}  // namespace smc
