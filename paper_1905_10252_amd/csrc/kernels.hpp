// Host-side launchers of the libsmc kernels (one translation unit per kernel
// family).  Every launcher enqueues on `s` and returns the launch status.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"

namespace smc {

constexpr int kScanThreads = 256;
// Scan tiles: 4096 elements (16 a thread) for large populations; below
// kSmallTileN tiles of 1024, so that the tiles cover the chip (at N = 2^17, 32
// tiles of 4096 took 5.9 us, a chain of 16 exponentials a thread).
constexpr int kTileShift = 12, kTileShiftSmall = 10;
constexpr int64_t kSmallTileN = 1 << 20;
static_assert(kScanThreads * 16 == 1 << kTileShift && kScanThreads * 4 == 1 << kTileShiftSmall,
              "tile sizes");
inline int tile_shift_of(int64_t n) { return n < kSmallTileN ? kTileShiftSmall : kTileShift; }
constexpr int kMaxBlocks = 1024;                  // grid of the max / reweight passes
constexpr int kIsBlocks = 2048;                   // max grid of the sampler kernels
constexpr int kExpandThreads = 256;
constexpr int kSegLen = 2048;                     // most merge-path steps per expand workgroup
// Populations from this size on are written past the caches by the expand
// (half of the 256 MB memory-side cache).
constexpr int64_t kStreamBytes = 128ll << 20;
// What else the expand moves through that cache (its prefix, the counts and ancestors
// it writes) taking two fifths of it, or all of it (see copy_streamed).
constexpr int64_t kTailStoreBytes = 104ll << 20, kTailLoadBytes = 2 * kStreamBytes;
// Largest row of smc_redistribute: a segment's 32-bit chunk count
// (kSegLen rows of row_bytes / 4 chunks) then stays below 2^31.
constexpr int kMaxRowBytes = 1 << 20;
static_assert((long long)kSegLen * (kMaxRowBytes / 4) < (1ll << 31), "expand chunk count");
constexpr int kEstCols = 10;                      // 2 + 2 d sums of a filter row (d = 4)
constexpr int kLogregSplit = 8;                   // row blocks of the likelihood contraction

struct TilePart {
    double Z, Z2;
    u64 q2lo, q2hi;
};

// Device pointers into the caller's workspace.
struct Work {
    Ctrl *ctrl;
    u64 *slots;         // [2][64][16] max / non-finite slots, double-buffered by parity
    u64 *tsum;          // [n_tiles] tile totals, then their exclusive prefix
    TilePart *tpart;    // [n_tiles]
    u64 *pref;          // [n] tile-local inclusive prefix (of q, or of foreign counts)
    u64 *pref64;        // [n / 64 + 1] every 64th tile-local prefix value
    // sampler state (NULL when no target)
    double *lp;         // [n] cached log-target of the current particles
    double *x_scr;      // [n * d] redistribute destination
    double *lp_scr;     // [n]
    double *is_part;    // [kIsBlocks * (2 + 2d)] per-block estimate sums
    double *cols;       // [2 + 2d] the same, folded over the blocks
    double *rec_num;    // [2d] recycled estimate sums
    double *epart;      // particle filter: [kEstCols][filter_segments] row sums of the
                        // redistributed rows (NULL otherwise)
    // logistic regression (NULL otherwise)
    unsigned short *xs;   // [mpad][dp] bf16 X times (1 - 2 y), in MFMA operand order
    unsigned short *thb;  // [npad][dp] bf16 copy of the particles times log2 e
    double *csum;         // [dp] column sums of X (1 - 2 y) (of xs for BF16)
    double *xf;           // FP64: [mpad / 16][64][lr_ks(d)] X (1 - 2 y) in MFMA operand order
    double *etab;         // FP64: [kExpTabN] powers 2^(-j / kExpTabN)
    double *lpart;        // [kLogregSplit][n] partial log-likelihoods
    int64_t mpad, npad;
    int dp;
    int n_tiles, tile_shift;
    int is_grid;        // blocks of the sampler kernels (rows of is_part)
};

// FP64 likelihood: MFMA k-steps of four columns, one or an even number (a
// lane's operands of a tile are read 16 bytes at a time).
inline int lr_ks(int d) { return d <= 4 ? 1 : (d + 7) / 8 * 2; }
// Entries of the FP64 likelihood's table of powers of two.
constexpr int kExpTabN = 2048;
inline int n_tiles_of(int64_t n)
{
    const int sh = tile_shift_of(n);
    return (int)((n + (1ll << sh) - 1) >> sh);
}
inline int max_blocks_of(int64_t n)
{
    int64_t b = (n + 1023) / 1024;  // one round of loads a thread, up to kMaxBlocks
    return (int)(b < 1 ? 1 : (b > kMaxBlocks ? kMaxBlocks : b));
}


hipError_t launch_init_ctrl(const Work &w, hipStream_t s);
// Max pass into the slots of parity par, then the fold of those slots.
hipError_t launch_max(const Work &w, const double *lw, int64_t n, int par, hipStream_t s);
hipError_t launch_fold(const Work &w, int par, hipStream_t s);
// A sampler iteration's statistics from its blocks' sums (is_part NULL: none).
struct StatsArgs {
    const double *is_part = nullptr;
    int nblk = 0, d = 0;
    double *cols = nullptr;  // NULL: a filter iteration, whose decision has been made
    double *rec_num = nullptr, *est = nullptr;
    void *info = nullptr;    // a filter iteration's smc_resample_info
};

// Quantise + scan; reads the max slots of parity par.
// clear_uniform: also clears the lazy-reset flag (an iteration's scan runs
// after the kernels that read it).  st: statistics that workgroups of their own
// form beside the scan: the fold of this iteration's sums over the blocks, for the
// decision to finish, or all of the filter iteration before.
hipError_t launch_quant_scan(const Work &w, const double *lw, int64_t n, int K, int par,
                             hipStream_t s, bool clear_uniform = false,
                             const StatsArgs &st = StatsArgs());

// Error and decision of the call from the max slots of parity par and the
// scan; info is a device smc_resample_info (nullable).
hipError_t launch_decide(const Work &w, int par, int64_t n, int K, uint64_t r, int mode,
                         int ess_num, int ess_den, void *info, hipStream_t s,
                         const StatsArgs &st = StatsArgs());
// Normalised weights exp(l_i - m) / Z from the last decision.
hipError_t launch_weights(const Work &w, const double *lw, int64_t n, double *out, hipStream_t s);
// smc_resample in one launch, for n <= kSmallResample (one workgroup; above, the
// separate passes spread over the chip); slots: also clears the max slots of
// the parity after par.
constexpr int64_t kSmallResample = 6144;
hipError_t launch_small_resample(const Work &w, const double *lw, int64_t n, int K, uint64_t r,
                                 int mode, int ess_num, int ess_den, int par, bool slots,
                                 int64_t *ncopies, void *info, hipStream_t s);
hipError_t launch_count_scan(const Work &w, const int64_t *ncopies, int64_t n, hipStream_t s);
hipError_t launch_ncopies(const Work &w, int64_t n, int count_mode, int64_t *ncopies,
                          hipStream_t s);

// Merge-path steps of an expand workgroup: the shortest of 256 to kSegLen with which
// the workgroups are resident at once, eight a CU (with one and a half to two rounds
// of them, N = 400000 took 29.7 us for resampling and rows of 16 bytes, and 25.8 in
// one; N = 1000003 38.6 and 33.5).
inline int expand_seg_len(int64_t n)
{
    int seg = 256;
    while (seg < kSegLen && 2 * n > 2048ll * seg) seg <<= 1;
    return seg;
}
// The same for the filter's fused iteration, whose workgroups hold their CU longer:
// four per CU (N = 2^20: 34.4 us with 2048 steps, 38.6 with 1024; N = 2^19: 24.6,
// 22.7 with 1024, 25.3 with 512; N = 2^17: 13.0 with 512, 12.8 with 256).
inline int filter_seg_len(int64_t n)
{
    int seg = kSegLen;
    while (seg > 256 && 2 * n < 1024ll * seg) seg >>= 1;
    return seg;
}
inline int64_t filter_segments(int64_t n)
{
    const int seg = filter_seg_len(n);
    return (2 * n + seg - 1) / seg;
}

// What the expand does when the decision kept the weights: kCopy writes the
// identity; kIfResampled writes nothing; kForward (a sampler iteration whose
// proposal waits in the workspace copy) writes the identity, also when the
// iteration found an error.
enum class ExpandMode { kCopy, kIfResampled, kForward };

// The expand's optional outputs (all nullable).
struct ExpandOut {
    ExpandMode mode = ExpandMode::kCopy;
    int64_t *ncopies = nullptr, *anc = nullptr;
    const void *aux = nullptr;  // 8-byte side rows copied along
    void *aux_out = nullptr;
    double *logw = nullptr;     // weights set to `reset` where the decision resampled,
    double reset = 0.0;         //   or the flag `uniform` set instead (lazy reset)
    unsigned *uniform = nullptr;
};
hipError_t launch_expand(const Work &w, int64_t n, int count_mode, const void *x, void *x_out,
                         int row_bytes, hipStream_t s, const ExpandOut &o);

}  // namespace smc
