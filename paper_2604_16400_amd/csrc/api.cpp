// C ABI of the mixed-batch LoRA linear layer: context, validation, plan upload, launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "collm_lora.h"
#include "kernels.h"
#include "planner.h"

using namespace collm;

namespace collm {
thread_local LaunchEvents g_launch_events;
}

namespace {

thread_local std::string g_last_error;

int hip_fail(hipError_t e, const char *what)
{
    char buf[256];
    std::snprintf(buf, sizeof buf, "%s: %s", what, hipGetErrorString(e));
    g_last_error = buf;
    return COLLM_E_HIP;
}

#define HIP_TRY(expr)                                     \
    do {                                                  \
        hipError_t e_ = (expr);                           \
        if (e_ != hipSuccess) return hip_fail(e_, #expr); \
    } while (0)

constexpr int kSlots = 16;             // pinned staging ring: the host may run this many uploads ahead
constexpr uint64_t kWarmMaxBytes = (uint64_t)40 << 20;  // largest weight a rank-wide pass fetches ahead of its GEMM
constexpr size_t kRecordBytes = (size_t)64 << 20, kRecordBlock = (size_t)1 << 20;  // pinned plans of recorded calls, in all and at a time
constexpr int kMaxProfile = 16;
constexpr int64_t kDualMinBytes = (int64_t)192 << 20;  // training rows of dy from which dh and dB come from one pass (bwd_impl)

inline int round_up(int v, int m) { return (v + m - 1) / m * m; }
// whether n bytes at p and m bytes at q have none in common
inline bool apart(const void *p, int64_t n, const void *q, int64_t m) { return (uintptr_t)p + n <= (uintptr_t)q || (uintptr_t)q + m <= (uintptr_t)p; }
inline bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

}  // namespace

// pinned memory with plans of recorded calls, which replays read; ints
struct RecordBlock {
    int32_t *host = nullptr, *dev = nullptr;
    size_t size = 0, used = 0;
};

struct collm_ctx {
    int device = 0;
    bool static_scratch = false;  // the workspace is the library's static device array; plans travel as kernel arguments
    int max_tokens = 0, max_segments = 0, max_adapters = 0, max_rank = 0, max_d = 0;
    int rows_cap = 0;   // padded row capacity
    int rpad_cap = 0;   // max_rank rounded up to 16

    size_t plan_cap = 0;  // int32 units
    int32_t *h_stage[kSlots] = {};      // pinned, device-visible
    int32_t *h_stage_dev[kSlots] = {};  // the same memory as the GPU addresses it
    uint32_t stage_seq[kSlots] = {};    // sequence number of the upload that last used the slot (0: none)
    uint32_t seq = 0;                   // uploads issued so far
    uint32_t *h_done = nullptr;         // pinned words: sequence number of the last finished upload; what copies of recorded plans store, unread
    uint32_t *h_done_dev = nullptr;
    int *d_copy_counter = nullptr;
    void *d_zeros = nullptr;  // 256 bytes of zeros for masked 16-byte loads
    float *d_part = nullptr;  // sums of the K slices of a skinny pass  [slices][rows][rpad]
    size_t part_bytes = 0;
    int slot = 0;
    int32_t *d_plan = nullptr;

    void *d_hs = nullptr;     // scaled low-rank activations, forward row order  [rows][rpad]
    void *d_dhs = nullptr;    // dh in the element type, training row order      [rows][rpad]
    float *d_h32 = nullptr;   // recomputed h, training row order                [rows][rpad]
    float *d_dh32 = nullptr;  // dh in fp32, training row order                  [rows][rpad]
    int64_t workspace_bytes = 0;

    std::vector<int32_t> plan;
    PlanLayout L;
    bool plan_valid = false;
    // A call of this context has been recorded into a graph.  A replay puts the recorded call's plan on the device and nothing tells the host,
    // so from then on every eager call uploads all of its plan (the host's copy of a known batch is still reused), and so does the first
    // recorded call of a capture; the calls behind it in that capture follow it in every replay too, and find its plan.
    bool recorded = false;
    unsigned long long capture_id = 0;  // the capture that the last call was recorded in (0: it was eager)
    std::vector<RecordBlock> record_blocks;
    size_t record_bytes = 0;
    // what the cached plan was built from
    collm_shape key_shape{};
    int key_bm_all = 0, key_bm_train = 0;
    std::vector<int32_t> key_seg_start, key_seg_adapter, key_rank;
    std::vector<uint8_t> key_seg_train;
    std::vector<uint64_t> key_A, key_B;

    int tile_fwd = -1, tile_bwd = -1;  // forced GEMM tile shapes (-1 = choose)
    int wide_min_rows = -1;            // forced threshold of the tiled rank-wide pass (-1 = choose, 0 = never)
    int dual_pass = -1;                // dh and dB from one pass over dy: -1 = where it pays, 0 = never, 1 = wherever it applies
    int grad_streams = -1;             // adapter gradients: -1 = choose, 0 = on the caller's stream, 1 = on the second stream
    int gemm_split = -1;               // forced number of K slices of a GEMM with few rows (-1 = choose, 1 = never)
    int n_cus = 0;                     // compute units of the device
    int key_wide = 0, key_nsib = 0;
    int tile_steps_all = 0, tile_steps_train = 0;  // low-rank K-steps of a 128-row tile of the call's batch, about (count_steps)
    std::vector<int32_t> rows_of;      // ... its rows per adapter
    std::vector<int32_t> sum_rank;     // sibling calls: ranks summed over the siblings
    hipStream_t last_stream = nullptr;
    // the adapter gradients run beside dh and the dX GEMM on a second stream
    hipStream_t side = nullptr;
    hipEvent_t ev_fork = nullptr, ev_dh = nullptr, ev_join = nullptr;

    PlanPatch patch{};  // new table addresses that the call's first rank-wide pass puts in (blocks > 0)

    // host cost of the plan of the last compute call (collm_debug_plan_stats)
    float plan_build_us = 0.f, plan_upload_us = 0.f;
    int plan_mode = 0;       // 0: reused as it is, 1: built anew, 2: table addresses replaced, 3: gradient pointers only
    int plan_bytes_up = 0;   // bytes the call sent to the device

    // what the last compute call ran (collm_debug_last_call)
    int ran_grad_slices = 0, ran_mixed = 0, ran_pass_slices = 0;

    bool profile = false;
    int n_prof = 0;
    const char *prof_name[kMaxProfile] = {};
    hipEvent_t prof_ev[kMaxProfile][2] = {};
    int prof_launches[kMaxProfile] = {};  // kernels each entry timed (0: nothing ran, the events were not recorded)
    bool prof_ev_made = false;
};

namespace {

// How a GEMM's tiles are cut: `tile` for the first `big_tiles_m` row tiles (all of them when
// tail_tiles_m is 0), then 128x128 tiles for `tail_tiles_m` row tiles of 128 rows.  Or (tail_cols > 0, 256x256
// tiles, no row tail): the last tail_cols tile columns of all rows run as 128x128 tiles in a second launch.
struct Tiling {
    int tile;
    int big_tiles_m;
    int tail_tiles_m;
    int tail_cols = 0;
    int slices = 1;  // 256x256 tiles, no tail: K slices (large_slices)
};

constexpr int kSplitBlocks = 512;  // 128x128 tiles that run at once: two per CU

// can_split: the 128x128 tiles behind the large ones may have K cut into slices (see run_gemm), which lets a few
// such tiles use the whole GPU
// steps: low-rank K-steps of a 128-row tile, about
// one_round: the tiles between the two sizes exist for this GEMM (plain tiles, no siblings side by side, no SwiGLU)
Tiling pick_tiling(int rows, int cols, int K, bool can_split, bool one_round, int steps)
{
    // Two shapes are worth choosing between for whole rounds: 256x256 run by four waves (one block per CU, the most
    // efficient inner loop) and 128x128 (two blocks per CU, four times as many tiles).  The cost of
    // a choice is the time its tiles take over the 256 CUs in units of one full round of 256x256
    // tiles; the constants are read off measurements on 4096- to 13824-wide layers:
    //  - 256x256: a GPU that is not filled once clocks higher, but a tile's start, end and waits for memory stay
    //    (0.65 + 0.35 x: 64 tiles 0.70, 112 0.75, 144 0.84-0.94, 172 0.89); after whole rounds a last
    //    round that keeps a fraction f of the CUs busy costs 0.6 + 0.7 f, at most 1;
    //  - 128x128: a round of 512 tiles costs 0.65, one that leaves every CU a single block 0.39; from
    //    two rounds on the blocks' different speeds smooth the rounds out (0.62 per round, 0.3 for a
    //    nearly empty last one);
    //  - whole rounds of 256x256 tiles over the first rows and 128x128 tiles over the rest, as two
    //    launches: the sum of both plus 0.1 for the idle CUs at the boundary between them; at most 256
    //    small tiles with K in slices cost their share of a full round plus the kernel that adds the slices;
    //  - against more than two rounds of 128x128 tiles (the third is as long as a whole one unless nearly empty) up to 447 small
    //    tiles cost that share too, as they start on the CUs the large ones leave, and part of a first round 0.5 + 0.5 x.
    //    Forward calls with 128x128 tiles / large and small ones, us: 5427 rows 5192 -> 3920 344 / 281, 1325 rows 4256 -> 14656 235 / 197,
    //    1107 rows 17488 -> 16952 1113 / 864; up to two rounds the other way, 636 rows 6808 -> 24704 307 / 352.
    auto cost_large = [](double tiles) {
        const double x = tiles / 256.0, whole = std::floor(x), part = x - whole;
        if (x <= 1.0) return 0.65 + 0.35 * x;
        return whole + (part == 0.0 ? 0.0 : std::min(1.0, 0.6 + 0.7 * part));
    };
    auto cost_small = [](double tiles) {
        const double x = tiles / 512.0, whole = std::floor(x), part = x - whole;
        if (whole >= 2.0) return 0.62 * whole + (part == 0.0 ? 0.0 : (part <= 0.1 ? 0.3 : 0.62 * part + 0.1));
        if (whole == 0.0) return part <= 0.5 ? 0.39 : 0.65;
        return 0.65 + (part == 0.0 ? 0.0 : (part <= 0.1 ? 0.3 : 0.65));
    };
    const int rp = round_up(std::max(rows, 1), kRowPad);
    const int tm = rp / 256, tn = (cols + 255) / 256, tn128 = (cols + 127) / 128;
    const int rows128 = (std::max(rows, 1) + 127) / 128;
    const double cost256 = cost_large((double)tm * tn), cost128 = cost_small((double)rows128 * tn128);
    Tiling best = cost256 <= cost128 ? Tiling{kTile256x256, tm, 0} : Tiling{kTile128x128, rows128, 0};
    double best_cost = std::min(cost256, cost128);
    const int rounds = tm * tn / 256;
    if (rounds >= 1 && (tm * tn) % 256 != 0) {
        const int m = std::min(tm - 1, rounds * 256 / tn);
        const int tail = (std::max(rows, 1) - 256 * m + 127) / 128;
        if (m >= 1 && tail >= 1) {
            const double tail_tiles = (double)tail * tn128;
            const double tail_cost = (can_split && K >= 1024 && tail_tiles <= kSplitBlocks / 2) ? 0.65 * tail_tiles / 512.0 + 0.05
                                                                                 : cost_small(tail_tiles);
            const double cost = cost_large((double)m * tn) + tail_cost + 0.1;
            if (cost < best_cost) {
                best = Tiling{kTile256x256, m, tail};
                best_cost = cost;
            } else if (best.tile == kTile128x128 && (long)rows128 * tn128 > 2 * kSplitBlocks && can_split && K >= 1024 && tail_tiles < 448) {
                const double first = (double)m * tn / 256.0;
                const double share = (first < 1.0 ? 0.5 + 0.5 * first : first) + 0.65 * tail_tiles / 512.0 + 0.05 + 0.1;
                if (share < best_cost) best = Tiling{kTile256x256, m, tail};
            }
        }
    }
    // Tiles between the two sizes, where one block per CU holds the whole GEMM (see the ring in gemm_lora_kernel): a first round
    // that large tiles fill badly and small ones overfill.  x = blocks / 256.  GEMM alone, weights from memory, geometric means over
    // 12000 shapes (100 to 8192 rows, 1024 to 16384 wide), time against the choice between the two sizes: 128x192 0.88 .. 0.96,
    // 256x128 0.92 .. 0.95, 256x192 0.92 .. 0.93.  Whole forward calls, weights from memory, 60 shapes each (128 to 4096 rows): 128x192 (259 to 385
    // small tiles) 0.86 (0.68 .. 1.04), 256x128 (377 to 512) 0.89 (0.75 .. 1.02), 256x192 (518 to 744) 0.93 (0.86 .. 1.04).  Where the weight stands
    // in the last-level cache there is less to hide: 1003 rows 5120 -> 5120 117 / 86 us from memory, 79 / 78 from the cache.
    // Below 257 small tiles K slices or the ring on 128x128 tiles are better.
    // Not where the extension is long (`steps` of a 128-row tile): one block alone on its CU waits for every batch of tables (about 2 us a
    // batch, 472 rows of 93 adapters of rank 128, K = 10320, 125 -> 160 us; 935 rows of 31 of rank 32, K = 2304, 53 -> 67).
    // Nor up to 341 small tiles of K >= 16384, which are cut into three slices (733 rows 25448 -> 5408 386 / 451).
    const long small_tiles = (long)tn128 * rows128;
    if (one_round && small_tiles > kSplitBlocks / 2 && (int64_t)steps * 256 <= K && !(K >= 16384 && small_tiles <= 2 * kSplitBlocks / 3)) {
        const int tn192 = (cols + 191) / 192;
        auto consider = [&](int tile, int tiles_m, long tiles, double cost) {
            if (tiles > 256 || cost >= best_cost) return;
            best = Tiling{tile, tiles_m, 0};
            best_cost = cost;
        };
        const long t192 = (long)rows128 * tn192, t256 = (long)tm * tn128, t256w = (long)tm * tn192;
        consider(kTile128x192, rows128, t192, 0.43 + 0.11 * t192 / 256.0);
        consider(kTile256x128, tm, t256, 0.47 + 0.11 * t256 / 256.0);
        consider(kTile256x192, tm, t256w, 0.71 + 0.11 * t256w / 256.0);
        if (best.tile != kTile256x256 && best.tile != kTile128x128) return best;
    }
    // ... or whole rounds over the first tile columns and the last columns of all rows as at most one round of
    // 128x128 tiles (two per CU) in a second launch: a last round that fills part of the CUs with large tiles
    // costs most of a round, 512 small tiles cost 0.65.
    if (rounds >= 1 && (tm * tn) % 256 != 0) {
        const int c = tn - rounds * 256 / tm;  // tile columns that do not fit the whole rounds
        const int cols_tail = cols - 256 * (tn - c);
        const long small = (long)rows128 * ((cols_tail + 127) / 128);
        if (c >= 1 && c < tn && small <= 512) {
            const double cost = cost_large((double)tm * (tn - c)) + cost_small((double)small) + 0.05;
            if (cost < best_cost - 0.05) best = Tiling{kTile256x256, tm, 0, c};
        }
    }
    return best;
}

// Whether 128x128 tiles that are not cut run as one block per CU with the ring of four stages: all of them at once, and no long
// extension (as in slices_one_per_cu).  0.48 us a K tile instead of 0.85 with two stages, weights from memory.
bool ring_alone(const Tiling &t, int cols, int K, int steps)
{
    return t.tile == kTile128x128 && t.tail_tiles_m == 0 && (long)t.big_tiles_m * ((cols + 127) / 128) <= kSplitBlocks / 2 && (int64_t)steps * 64 <= K;
}

// Slices of K of a GEMM of few tiles run as at most one block per CU with the ring of four stages (three tiles of loads in flight per
// CU instead of two, half the partial sums), or 0 where `two` slices on two blocks per CU are better.  GEMM with the kernel
// that adds the slices against two blocks per CU with two stages, weights from memory, 10000 shapes (1 to 2048 rows, K =
// 1024 to 28672, 1 to 64 adapters of rank 16 to 64): up to 16 tiles 0.88 .. 0.91, up to 32 0.91, up to 64 0.92, up to 85 0.94.  From 86 to 128
// tiles (two slices) it would be 0.96 .. 1.3 for every contraction; where the comparison below takes it, whole forward calls of 150 shapes
// measured 0.94 (0.84 .. 1.03).  A slice keeps 192 K values (geometric mean 0.927; 256: 0.929, 512: 0.976).
//  - Also for dX beside the gradient kernels on the second stream, although a CU that holds such a block has no room for theirs: whole
//    backward calls, 950 shapes (64 to 1500 rows, 512 to 8192 <- 1024 to 16384): 0.979 (0.88 .. 1.18); level only where ranks up to 16 meet a
//    weight below 8 MB (65 shapes, 1.003), by no line that separates the shapes that lose (695 rows 2568 <- 2712 57 / 48 us) from those that gain
//    (948 rows 1472 <- 2080 39 / 44).
//  - A block alone on its CU takes 0.48 us a K tile, one of two 0.90; a slice's sums are written and read once more (about 8 TB/s).  The rule
//    compares these: a long contraction is better cut for the blocks that exist (714 rows, 72 tiles, K = 26112: three
//    slices on 216 CUs 124 us, seven on two blocks per CU 109).
//  - Not where the extension steps of a row tile outweigh K: they are spread over half as many blocks then (64 adapters of
//    rank 64 at K = 2048 1.2 .. 1.4).
long slices_one_per_cu(long tiles, int tiles_m, int K, int steps, long fit, long two)
{
    if (tiles > kSplitBlocks / 4 || (int64_t)steps / std::max(tiles_m, 1) * 64 > K) return 0;
    const long one = std::max(1L, std::min<long>({kSplitBlocks / 2 / tiles, K / 192, fit, 64L}));
    const double ktiles = K / 64.0, sums = tiles * 64.0 * 128.0 * 8.0 / 8e6;  // us (a row tile is mostly not full)
    return 0.48 * ktiles / one + sums * one <= 0.90 * ktiles / two + sums * two ? one : 0;
}

// Few tiles against a long contraction (decode-sized batches, or the small tiles behind whole rounds of large
// ones): too few blocks to fill the GPU, each walking all of K with one tile of loads in flight.  K is cut into
// slices so that up to two blocks per CU exist, as long as the fp32 partial sums fit the workspace; a second kernel adds the
// slices.  The slices share a row tile's extension steps too, and a step costs about as much as 32 K values (its table rows
// come one trip to memory later), so the rule counts K + 32 steps.  Forward calls with every number of slices, weights cold, in
// us; 818 shapes of 4 to 256 tiles, K = 256 to 28672, 8 to 96 steps: the rule is 1.2 % off the best on average, 18 % at worst.
//  - Up to one block per CU, where a block's chain is the time, a slice keeps 288: 8 tiles of K = 2048 (16 rows) 33 / 20 us with one slice / 8;
//    16 of K = 8192 143 / 45 with 16 (128 rows, 96 steps).
//  - Up to two blocks per CU it keeps 688: 64 tiles of K = 8192 52 / 45 with 4 / 7, but of K = 2048 (64 rows) 27.8 / 29.2.
//  - None below 1024: K = 512 and 32 tiles of 64 rows 22.1 / 21.8 with one / two, but with 96 steps 50 / 31 with 4.  With several row tiles
//    the sums weigh more, and none below 1408: 64 tiles (256 rows) of K = 1024 25.3 / 28.8, of K = 1536 31.2 / 30.3 with 4.
//  - 512 blocks in eight slices or more whose length is a power of two are slower than one slice less (the slices start in the
//    same memory channels): 64 tiles of K = 4096 35.1 / 32.0, 8192 50.4 / 44.9; K = 14336 72.7 / 87.2 ([N][K]: seven of 2048).
// Long contractions whose tiles fill one round only partly: three slices make nearly two whole rounds of up to 341 tiles,
// and a block's start and end no longer count.  With a power of two of row tiles one slice is slower for the same number of
// tiles, and slices pay earlier.  Whole forward call, 1 / 2 / 3 slices (row x column tiles): 8x36 of K = 8192 121 / 148 /
// 119, 11008 160 / 197 / 157, 14336 198 / 236 / 181; 4x84 of K = 14336 269 / 244 / 218; the GEMM alone, 3x110 of K = 14336
// 196 / 232 / 196, 16384 223 / 260 / 222, 28672 382 / 451 / 361; 2x129 of K = 14336 184 / 231 / 192.  Beyond, two slices: 8x44 tiles of K = 8192
// 161 / 153 and 148 / 155 ([N][K]), 14336 266 / 240 and 265 / 252; 4x86 of K = 20480 362 / 321 and 372 / 340, but 4x88 385 / 384
// and 372 / 399; not with other numbers of row tiles (6x64 of K = 20480 280 / 318, 3x115 304 / 373) or more tiles (8x48 367 / 377).
// steps: extension steps of all the row tiles.
// one_per_cu: null, or (plain tiles, the launch is the whole GEMM) whether the slices run as one block per CU (slices_one_per_cu).
long gemm_slices(int forced, int64_t part_bytes, int tiles_m, int cols, int K, bool b_kmajor, int steps, bool *one_per_cu)
{
    const long tiles = std::max((long)tiles_m * ((cols + 127) / 128), 1L);
    const long fit = (long)(part_bytes / std::max((int64_t)tiles_m * 128 * cols * 4, (int64_t)1));
    if (one_per_cu) *one_per_cu = false;
    if (forced > 1) return std::min<long>({forced, K / 64, fit, 64L});
    if (tiles > kSplitBlocks / 2) {
        const bool pow2 = tiles_m > 1 && (tiles_m & (tiles_m - 1)) == 0;
        long want = 1;
        if (tiles <= 2 * kSplitBlocks / 3) {
            if (K >= (pow2 && tiles >= 264 ? 11264 : 16384)) want = 3;
        } else if (pow2 && tiles <= 360) {
            if (tiles_m >= 8 ? K >= 11264 : (K >= 20480 && !b_kmajor)) want = 2;
        }
        return want <= fit ? want : 1;  // (all of them or none: fewer slices would be another round)
    }
    const int64_t len = K + (int64_t)32 * steps / std::max(tiles_m, 1);
    if (len < (tiles_m > 1 && tiles > 32 ? 1408 : 1024)) return 1;
    const long most = kSplitBlocks / tiles;
    long two = std::min<long>(most, len / 688);
    if (two == most && two >= 8 && two * tiles == kSplitBlocks) {
        const int slice = round_up((int)((K + two - 1) / two), 64);
        if ((slice & (slice - 1)) == 0) --two;
    }
    two = std::min<long>({std::max(two, std::min<long>(kSplitBlocks / 2 / tiles, len / 288)), (long)K / 64, fit, 64L});
    if (one_per_cu) {
        const long one = slices_one_per_cu(tiles, tiles_m, K, steps, fit, std::max(two, 1L));
        *one_per_cu = one > 0;
        if (one > 0) return one;
    }
    return two;
}

// K slices of 256x256 tiles, one block per CU in one round, or 0 where 128x128 tiles (at most 256 of them, in slices of their own on two
// blocks per CU) are the better ones.  For the same products a CU moves twice the bytes from L2 to LDS with two blocks of 128x128 tiles, and that
// path, not the matrix pipes, is their limit; but a block of 256x256 starts and ends longer, its slices are more and their sums too, and rows and
// columns that do not exist cost up to four times as much.  Times (us a K tile of a block, sums read and written per us, fixed) fitted to 63
// forward calls of 128 to 3600 rows, weights from memory; the margin is what separates all that lost from all that gained.
// GEMM with its sums inside whole calls, us, 128x128 / 256x256: 512 rows 22016 -> 5856 237 / 147 and 204 / 157 (backward), 1024 rows 4096 <- 22016 with the
// gradients beside it 214 / 165, 768 rows 9216 -> 4272 93 / 80, 2048 rows 22016 -> 1280 175 / 144, 256 rows 24832 -> 8792 199 / 144; outside the
// line 384 rows 15616 -> 10752 154 / 167, 599 rows 6912 -> 3840 56 / 66, 833 rows 12800 -> 1792 63 / 70, 896 rows 27136 -> 1024 level.
long large_slices(int64_t part_bytes, int rows, int cols, int K, bool b_kmajor, int steps)
{
    const int tiles_m = (rows + 127) / 128;
    const long tiles = (long)((rows + 255) / 256) * ((cols + 255) / 256), small_tiles = (long)tiles_m * ((cols + 127) / 128);
    const int64_t slice_bytes = (int64_t)rows * cols * 4;
    const long n = tiles > 0 ? std::min<long>({kSplitBlocks / 2 / tiles, (long)(part_bytes / slice_bytes), K / 512L}) : 0;
    // (not where the extension is long, as in slices_one_per_cu)
    if (n < 2 || small_tiles > kSplitBlocks / 2 || (int64_t)steps * 64 > K) return 0;
    bool alone = false;
    const long small = gemm_slices(-1, part_bytes, tiles_m, cols, K, b_kmajor, steps * tiles_m, &alone);
    if (alone) return 0;
    auto ktiles = [&](long slices) { return (double)((K + 64 * slices - 1) / (64 * slices)); };
    const double mb = slice_bytes / 1e6;
    const double large_us = 2.2 * ktiles(n) + 0.44 * mb * n + 8.0, small_us = 1.35 * ktiles(small) + 0.62 * mb * (small > 1 ? small : 0);
    return large_us < small_us ? n : 0;
}

// pick_tiling, or 256x256 tiles in slices of K (plain: no siblings side by side, no SwiGLU epilogue).
Tiling choose_tiling(int gemm_split, int64_t part_bytes, int rows, int cols, int K, bool b_kmajor, bool plain, bool can_split, bool one_round, int steps)
{
    Tiling t = pick_tiling(rows, cols, K, can_split, one_round, steps);
    if (!plain || !can_split || gemm_split >= 0 || t.tile != kTile128x128 || t.tail_tiles_m > 0) return t;
    const long n = large_slices(part_bytes, rows, cols, K, b_kmajor, steps);
    if (n >= 2) {
        t = Tiling{kTile256x256, (rows + 255) / 256, 0};
        t.slices = (int)n;
    }
    return t;
}
Tiling choose_tiling(const collm_ctx *c, int rows, int cols, int K, bool b_kmajor, bool plain, bool can_split, bool one_round, int steps)
{
    return choose_tiling(c->gemm_split, (int64_t)c->part_bytes, rows, cols, K, b_kmajor, plain, can_split, one_round, steps);
}

// Low-rank K-steps that a 128-row tile of the batch has on average, over all rows and over the training rows: an adapter reaches
// into about rows / 128 + 1 tiles.  (The tile choice needs it before the plan, whose steps depend on the tiles, is built.)
void count_steps(collm_ctx *c, const collm_shape *s, const int32_t *rank, const int32_t *seg_start, const int32_t *seg_adapter,
                 const uint8_t *seg_is_train)
{
    const int N = s->n_adapters;
    c->rows_of.assign((size_t)2 * std::max(N, 1), 0);
    int n_train = 0;
    for (int k = 0; k < s->n_segments; ++k) {
        const int a = seg_adapter[k], n = seg_start[k + 1] - seg_start[k];
        if (seg_is_train[k]) n_train += n;
        if (a < 0 || n == 0) continue;
        c->rows_of[2 * a] += n;
        if (seg_is_train[k]) c->rows_of[2 * a + 1] += n;
    }
    int64_t steps[2] = {0, 0};
    for (int a = 0; a < N; ++a)
        for (int o = 0; o < 2; ++o)
            if (c->rows_of[2 * a + o] > 0) steps[o] += (int64_t)((rank[a] + kKStep - 1) / kKStep) * (c->rows_of[2 * a + o] + 128);
    c->tile_steps_all = (int)(steps[0] / round_up(std::max(s->n_tokens, 1), 128));
    c->tile_steps_train = (int)(steps[1] / round_up(std::max(n_train, 1), 128));
}

int tile_steps(const collm_ctx *c, const RowOrderLayout &R) { return &R == &c->L.all ? c->tile_steps_all : c->tile_steps_train; }

// Extension steps of `tiles_m` row tiles of 128 rows from row tile `first` on, as the plan lists them.
int steps_of(const collm_ctx *c, const RowOrderLayout &R, int first, int tiles_m)
{
    const int32_t *off = c->plan.data() + (R.bm == 128 ? R.off_ext_off : R.off_ext_off_half) + first;
    return off[tiles_m] - off[0];
}

long gemm_slices(const collm_ctx *c, const RowOrderLayout &R, int first, int tiles_m, int cols, int K, bool b_kmajor, bool *one_per_cu)
{
    return gemm_slices(c->gemm_split, (int64_t)c->part_bytes, tiles_m, cols, K, b_kmajor, steps_of(c, R, first, tiles_m), one_per_cu);
}

// Whether the rank-wide pass in front of a GEMM should fetch the GEMM's weight into the last-level cache (run_skinny has
// the conditions on the pass itself).  Not where the GEMM is cut into slices and the weight is large: its 512 blocks
// keep enough loads in flight to stream the weight from memory at full rate, so the fetch only makes the pass longer
// (33 MB: 4-5 us, of which the GEMM gives back 1-3).  Measured, whole forward call in us with / without the fetch,
// 4096 -> 4096: 8 rows 32 / 29, 64 rows 36 / 32, 256 rows 47 / 44, 512 rows level, 1003 rows (one slice) 65 / 71;
// 1024 -> 1024 (2 MB): 22 / 24 and 26 / 28.
// grad_slices: 0, or the slices of a dX GEMM with the gradients in its launch, which has two blocks per CU whatever it would take alone.  Backward calls
// whose GEMM alone would be cut or in the ring, weights from memory: 90 shapes 1.06 times as fast with the fetch (1.00 .. 1.12; 79 tokens 5600 <- 824 26 / 23 us).
bool warm_pays(const collm_ctx *c, const RowOrderLayout &R, int rows, int cols, int K, bool b_kmajor, bool one_round, bool siblings, int grad_slices = 0)
{
    constexpr int64_t kWarmSlicedMaxBytes = (int64_t)8 << 20;
    if ((int64_t)cols * K * 2 <= kWarmSlicedMaxBytes) return true;
    if (grad_slices > 0) return grad_slices == 1;
    const bool can_split = c->gemm_split != 1;
    const Tiling t = choose_tiling(c, rows, cols, K, b_kmajor, !siblings, can_split, one_round, tile_steps(c, R));
    if (t.slices > 1) return false;
    if (t.tile != kTile256x256 && t.tile != kTile128x128) return false;
    bool alone = false;
    if (one_round && ring_alone(t, cols, K, tile_steps(c, R))) return false;
    return !(can_split && t.tile == kTile128x128 && t.tail_tiles_m == 0 && gemm_slices(c, R, 0, t.big_tiles_m, cols, K, b_kmajor, siblings ? nullptr : &alone) >= 2);
}

// Whether the adapter gradients of a backward call stay on the caller's stream.  On the second stream they run beside dh and
// the dX GEMM, but the three dependences between the streams cost 10 us on the GPU and more of host time per call.  The line
// lies where one stream stops saving time of a loop that the host keeps up with (forward + backward, wall) and starts to cost the
// GPU some (backward, queued ahead).  Two streams / one, us, by MiB of training rows of dy and x; wall and GPU:
//   rank 8, 16   0.4: 67 / 45 and 36 / 27;  1.9: 92 / 70 and 40 / 41;  3.8: 90 / 75 and 41 / 44 or 43 / 42;  6.0: 84 / 85 and 46 / 50;
//                7.5: 91 / 90 and 49 / 55
//   rank 32      0.4: 73 / 54 and 35 / 33;  1.9: 98 / 74 and 39 / 43;  3.0: 94 / 80 and 44 / 50;  6.0: 91 / 94 and 45 / 57
//   rank 64      0.8: 96 / 79 and 43 / 49;  3.0: 93 / 98 and 50 / 62: the gradient kernels themselves are too long
//   fp32         2.0: 69 / 56 and 35 / 31;  8.0: 100 / 98 and 54 / 55;  16: 156 / 169 and 91 / 105
// (the width of the gradient kernel's launch is the largest rank of the call's adapters, trained or not)
bool grads_alone(int n_train, int d_in, int d_out, bool f32, int rpad)
{
    const int64_t bytes = (int64_t)n_train * ((int64_t)d_in + d_out) * (f32 ? 4 : 2);
    const int64_t MiB = (int64_t)1 << 20;
    return bytes <= (f32 ? 8 * MiB : (rpad <= 16 ? 5 * MiB : (rpad <= 32 ? 2 * MiB : 0)));
}

// Whether dB starts behind the dh pass, with dA, instead of beside it: the caller's stream then has one point less at which it hands
// over to the second one (5 us of idle time each), and the dX GEMM alone has to cover both gradients.  So not where they are long against
// it: ranks above 32, a dimension so narrow that dX is short for its bytes, many columns of dy for few of x.  Backward call, beside
// the dh pass / behind it, us: 1792 rows 4096 -> 4096 rank 16 81.7 / 79.5, 7000 rows 240 / 216, 2048 rows 5120 -> 5120 126 / 118, 575 rows 8192 -> 6368
// rank 32 120 / 115, 3000 rows 8192 -> 16384 862 / 700; 30 shapes inside these limits 0.965 (geometric mean), 0.82 .. 1.03.  Outside: 230 rows
// 2568 -> 18432 rank 8 63 / 69, 4683 rows 1536 -> 4096 rank 16 90 / 92, 3500 rows 4096 -> 4096 rank 64 139 / 152, 276 rows 8448 -> 3328 rank 128 92 / 108.
bool fork_behind_dh(int rpad, int d_in, int d_out)
{
    return rpad <= 32 && (int64_t)d_in * d_out >= (int64_t)1700 * ((int64_t)d_in + d_out) && d_out <= 3 * (int64_t)d_in;
}

// ... nor where 256x256 tiles of dX make whole rounds (or all but a tenth of one): no CU is then free for the gradients before its end.
// 4096 rows 8192 -> 8192 rank 16 431 / 439 us, 4000 rows 4096 -> 4096 rank 32 147 / 152, 12000 rows rank 16 363 / 375.
bool whole_rounds(int rows, int cols, int slices)
{
    const int last = (int)((int64_t)(round_up(rows, 256) / 256) * ((cols + 255) / 256) * slices % 256);
    return last == 0 || last > 230;
}

// Whether the dX GEMM of a backward call may take the tiles that fill a CU's LDS and one round of CUs, uncut (pick_tiling, ring_alone):
// not where the gradient kernels run beside it on the second stream, as a CU that holds such a tile has no room for their blocks.  (K slices
// in the ring are shorter and take it all the same, slices_one_per_cu.)
// Backward call, us, with the two sizes only / all of them: 1792 rows 4096 -> 4096 86 / 88, 901 rows 4104 -> 11008 172 / 180.
bool dx_one_round(const collm_ctx *c, int n_train, int d_in, int d_out, bool f32, int rpad)
{
    return c->grad_streams >= 0 ? c->grad_streams == 0 : grads_alone(n_train, d_in, d_out, f32, rpad);
}

// Whether a call runs as the two kernels of kernels_decode.hip.
bool decode_sized(const collm_ctx *c, const collm_shape *s, const int32_t *rank, const int32_t *seg_start, const int32_t *seg_adapter, const uint8_t *seg_is_train,
                  int n_sib, bool swiglu)
{
    const int T = s->n_tokens;
    if (s->dtype != COLLM_BF16 || n_sib > 1 || swiglu || T < 1 || T > kDecodeRows) return false;
    if (c->tile_fwd >= 0 || c->gemm_split >= 0 || c->wide_min_rows >= 0) return false;
    // (64 rows of [N][K] weights are a quarter slower to read, which the longest contractions do not get back, us the general path / this: 28672 -> 4096 70.9 / 72.6,
    // 50 rows 24576 -> 6144 93.6 / 94.5, 20000 -> 4096 58.0 / 55.0)
    const bool tr = s->layout == COLLM_LAYOUT_OUT_IN;
    if (tr && T > 32 && s->d_in > 20480) return false;
    // (all rows on the base weight: the general path has no rank-wide pass then, and one kernel less where it does not cut K; us, it / this: 616 -> 13376
    // [N][K] 12.4 / 15.7, 12304 -> 6496 34 / 37, 13 drawn calls 0.88)
    bool adapters = false;
    for (int k = 0; k < s->n_segments; ++k) {
        if (seg_start[k + 1] == seg_start[k]) continue;
        if (seg_is_train[k]) return false;
        adapters = adapters || seg_adapter[k] >= 0;
    }
    if (!adapters) return false;
    int rmax = 1;
    for (int a = 0; a < s->n_adapters; ++a) {
        // (16-byte loads of parts of a table's rows: [rank] rows of B_a in one layout, 64 of more than 64 columns of A_a in the other)
        if (rank[a] % 8 != 0 && (tr || rank[a] > kDecodeRankCols)) return false;
        rmax = std::max(rmax, rank[a]);
    }
    // (at least one slice of each kind fits the workspace)
    return (int64_t)T * s->d_out + (int64_t)round_up(T, 16) * round_up(rmax, kKStep) <= (int64_t)c->part_bytes / 4;
}

// Gradients that run in blocks of the dX GEMM's launch (launch_gemm_grads).
struct GradsBeside {
    GradArgs dB, dA;
    int n_grad, rpad;
    int slices = 0;  // of K
    bool done = false;
};

// Slices of K of a dX GEMM with the gradients in its launch, or 0 where they have kernels of their own (serial: on the caller's stream).  One
// launch saves the two points at which the caller's stream hands over to the second one (5 us of idle time each), or two kernels in a
// chain, and the kernel that packs h; but the gradients' blocks are half as wide and share the CUs with the GEMM's.  A K tile of one of two
// GEMM blocks on a CU takes 0.9 us (0.48 of one alone, which leaves no place for a gradient), a chunk of 128 rows of a gradient block 1.2; the
// sums are written and read at 8 TB/s.
//  - GEMM of two blocks per CU beside the second stream: where the gradients end before its blocks in the places they leave.  Passes (forward and
//    backward), us: four layers 4096 -> 4096, 2048 tokens, rank 16 590 / 583; 740 tokens 5632 -> 2528 rank 32 448 / 406, 1148 tokens
//    6496 -> 3072 rank 64 700 / 660; 45 batches 1.009, none slower.  Where they miss it by up to 2.5 as many lose as gain (1096 -> 4864 rank 64
//    256 / 277, 13072 -> 2360 294 / 280).
//  - GEMM of one block per CU, or a call on one stream: the number of slices at which GEMM and gradients end first, if it is at most 8 (one
//    stream: 10) us behind the GEMM without them.  469 tokens 1056 -> 5496 rank 16 151 / 114, 733 tokens 1280 -> 2816 rank 64 357 / 289, 257 tokens
//    2992 -> 4096 rank 64 347 / 312; on one stream 271 tokens 3072 -> 1208 445 / 365, 401 tokens 1536 -> 2304 rank 8 114 / 98, 712 tokens 1280 -> 1280
//    rank 32 264 / 229; 36 batches 1.05 times as fast; at 10 us 1418 tokens 1792 -> 4136 rank 32 184 / 192, on one stream at 12 us 257
//    tokens 12544 -> 6488 728 / 750.
//  - Never where one block's rows take longer than all that: it walks the rows of its adapter in four waves, 1.3 us for 128 of them up to rank 16, 3.6
//    beyond (64 rank columns whatever the rank), while the kernels of their own have eight waves up to rank 32 and start beside the dh pass.  Backward calls,
//    two streams / one launch: one adapter of rank 32 with 6288 rows 784 <- 768 79 / 206, of rank 64 with 3381 rows 344 <- 536 92 / 124, of rank 16 with
//    5995 rows 768 <- 472 72 / 75.  780 drawn calls of 100 to 9000 rows: level at nine chunks of 128 rows (rank 16: 37), or where the GEMM covers them two and
//    a half times; 151 of them were more than 3 % slower in one launch, of the 573 inside this line 8 are (down to 0.885), those outside it 0.84.
int grads_in_gemm(const collm_ctx *c, int n_train, int d_in, int d_out, bool b_kmajor, int rpad, bool serial)
{
    if (c->grad_streams >= 0 || c->tile_bwd >= 0 || c->gemm_split >= 0 || rpad > kGemmGradRank || c->L.train.bm != 128) return 0;
    const Tiling t = choose_tiling(c, n_train, d_in, d_out, b_kmajor, true, true, false, c->tile_steps_train);
    if (t.tile != kTile128x128 || t.tail_tiles_m > 0) return 0;
    bool alone = false;
    const long n = std::max(1L, gemm_slices(c, c->L.train, 0, t.big_tiles_m, d_in, d_out, b_kmajor, &alone));
    const int chunks = (c->L.max_grad_rows + 127) / 128;
    const long tiles = (long)t.big_tiles_m * ((d_in + 127) / 128), grads = (long)c->L.n_grad * ((d_in + 63) / 64 + (d_out + 63) / 64);
    const double grad_us = grads * (5.0 + 1.2 * chunks);
    auto gemm_us = [&](long slices, double tile_us) { return tile_us * ((d_out + 64 * slices - 1) / (64 * slices)); };
    const double block_us = rpad <= 16 ? 5.0 + 1.3 * chunks : 8.0 + 3.6 * chunks;
    if (chunks > (rpad <= 16 ? 37 : 9) && block_us > 0.4 * gemm_us(n, 0.9)) return 0;
    if (!serial && !(n > 1 && alone)) return tiles * n < kSplitBlocks && grad_us <= gemm_us(n, 0.9) * (kSplitBlocks - tiles * n) ? (int)n : 0;
    // (wider ranks' blocks have more sums to write)
    const double grads_us = rpad <= 16 ? grad_us : grads * (8.0 + 1.8 * chunks);
    if (tiles > kSplitBlocks / 2) return 0;  // (on one stream the tiles between the two sizes are better)
    const double sum_us = (double)t.big_tiles_m * 128 * d_in * 8 / 8e6;
    double best_us = gemm_us(n, n == 1 || alone ? 0.48 : 0.9) + (n > 1 ? n * sum_us : 0.0) + (serial ? 10.0 : 8.0);
    int best = 0;
    for (long k = 1; k <= n && tiles * k < kSplitBlocks; ++k) {
        const double us = std::max(gemm_us(k, 0.9), grads_us / (kSplitBlocks - tiles * k)) + (k > 1 ? k * sum_us : 0.0);
        if (us < best_us) {
            best_us = us;
            best = (int)k;
        }
    }
    return best;
}

// One GEMM over the row order `R`: a single launch, or whole rounds of large tiles followed by
// small tiles over the remaining rows.
hipError_t run_gemm(collm_ctx *c, GemmArgs g, const RowOrderLayout &R, int rows, int cols, int forced_tile,
                    bool b_kmajor, bool one_round, hipStream_t st, bool swiglu = false, GradsBeside *beside = nullptr)
{
    // SwiGLU epilogue: `cols` counts gate and up columns; a tile holds half as many output columns as it is wide
    auto launch = [&](int tile) {
        g.tiles_n = (cols + gemm_tile_cols(tile) - 1) / gemm_tile_cols(tile);
        return swiglu ? launch_gemm_swiglu(g, tile, st) : launch_gemm(g, tile, b_kmajor, st);
    };
    const bool can_split = !swiglu && c->gemm_split != 1;
    // (the tiles between the two sizes are plain ones: a forced one stands for the size of the same height elsewhere)
    if (forced_tile >= 0 && (swiglu || g.n_sib > 1)) forced_tile = gemm_tile_rows(forced_tile) == 256 ? kTile256x256 : kTile128x128;
    const Tiling t = forced_tile >= 0 ? Tiling{forced_tile, R.n_rows_pad / gemm_tile_rows(forced_tile), 0}
                                      : choose_tiling(c, rows, cols, g.K, b_kmajor, !swiglu && g.n_sib <= 1, can_split, one_round, tile_steps(c, R));
    g.tile_m_base = 0;
    g.tiles_m = t.big_tiles_m;
    g.ext_off = c->d_plan + R.off_ext_off;
    g.ext = reinterpret_cast<const ExtStep *>(c->d_plan + R.off_ext);
    // few tiles against a long contraction: see gemm_slices.  Returns false if the launch should be a plain one.
    auto try_split = [&](int tiles_m, int row_base, int n_rows_here, hipError_t &err) -> bool {
        if (!can_split || forced_tile >= 0) return false;
        const int tiles_n = (cols + 127) / 128;
        const bool whole = !swiglu && g.n_sib <= 1 && row_base == 0 && t.tail_tiles_m == 0;
        bool alone = false;
        const bool with_grads = beside && whole;
        const long want = with_grads ? beside->slices : gemm_slices(c, R, row_base / 128, tiles_m, cols, g.K, b_kmajor, whole ? &alone : nullptr);
        if (want < 2) return false;
        GemmArgs gs = g;
        gs.tiles_m = tiles_m;
        gs.tiles_n = tiles_n;
        gs.k_per_split = round_up((int)((g.K + want - 1) / want), 64);
        const int n_split = (g.K + gs.k_per_split - 1) / gs.k_per_split;
        gs.part = c->d_part;
        gs.part_rows = tiles_m * 128;
        gs.part_ld = cols;
        gs.one_per_cu = alone;
        gs.row_base = row_base;
        gs.n_rows = n_rows_here;
        if (with_grads) {
            err = launch_gemm_grads(gs, n_split, b_kmajor, beside->dB, beside->dA, beside->n_grad, beside->rpad, st);
            beside->done = true;
        } else {
            err = launch_gemm_splitk(gs, kTile128x128, n_split, b_kmajor, st);
        }
        if (err == hipSuccess) err = launch_gemm_finish(gs, n_split, st);
        return true;
    };
    if (t.slices > 1) {
        GemmArgs gs = g;
        gs.tiles_n = (cols + 255) / 256;
        gs.k_per_split = round_up((g.K + t.slices - 1) / t.slices, 64);
        const int n_split = (g.K + gs.k_per_split - 1) / gs.k_per_split;
        gs.part = c->d_part;
        gs.part_rows = rows;
        gs.part_ld = cols;
        gs.row_base = 0;
        gs.n_rows = rows;
        if (R.bm != 256 || (int64_t)n_split * rows * cols * 4 > (int64_t)c->part_bytes) return hipErrorInvalidValue;
        const hipError_t err = launch_gemm_splitk(gs, kTile256x256, n_split, b_kmajor, st);
        return err == hipSuccess ? launch_gemm_finish(gs, n_split, st) : err;
    }
    hipError_t e = hipSuccess;
    if (t.tile == kTile128x128 && t.tail_tiles_m == 0 && try_split(t.big_tiles_m, 0, rows, e)) return e;
    // Whole rounds of large tiles over the first columns, small tiles over the other columns of all rows.  With the SwiGLU epilogue only
    // where the last round counts: after three rounds and a half the blocks' different speeds have smoothed the rounds out (training
    // rows also keep their pre-activations).  Forward call, one launch / two, by tiles / 256: 1.1 .. 1.5 0.85 .. 0.99, 2.1 .. 2.5 0.91 .. 0.99,
    // 3.1 .. 3.3 0.93 .. 1.01, 3.5 0.97 .. 1.03, beyond 0.95 .. 1.05 (4096 rows 4096 -> 2 x 2560, rank 64 232 / 209 us, -> 2 x 9216 586 / 599).
    const int big_tiles = t.big_tiles_m * ((cols + 255) / 256);
    if (t.tail_cols > 0 && (!swiglu || big_tiles < 256 * 7 / 2)) {
        const int tn_big = (cols + 255) / 256 - t.tail_cols;
        g.tiles_n = tn_big;
        e = swiglu ? launch_gemm_swiglu(g, kTile256x256, st) : launch_gemm(g, kTile256x256, b_kmajor, st);
        if (e != hipSuccess) return e;
        g.n_base = (swiglu ? 128 : 256) * tn_big;
        g.tiles_n = (cols - 256 * tn_big + 127) / 128;
        g.tiles_m = (rows + 127) / 128;
        g.ext_off = c->d_plan + R.off_ext_off_half;
        g.ext = reinterpret_cast<const ExtStep *>(c->d_plan + R.off_ext_half);
        return swiglu ? launch_gemm_swiglu(g, kTile128x128, st) : launch_gemm(g, kTile128x128, b_kmajor, st);
    }
    if (beside && t.tile == kTile128x128 && t.tail_tiles_m == 0) {
        g.tiles_n = (cols + 127) / 128;
        beside->done = true;
        return launch_gemm_grads(g, 1, b_kmajor, beside->dB, beside->dA, beside->n_grad, beside->rpad, st);
    }
    g.one_per_cu = one_round && forced_tile < 0 && ring_alone(t, cols, g.K, tile_steps(c, R));
    e = launch(t.tile);
    if (e != hipSuccess || t.tail_tiles_m == 0) return e;
    g.one_per_cu = 0;
    g.tile_m_base = 2 * t.big_tiles_m;
    g.tiles_m = t.tail_tiles_m;
    g.ext_off = c->d_plan + R.off_ext_off_half;
    g.ext = reinterpret_cast<const ExtStep *>(c->d_plan + R.off_ext_half);
    if (try_split(t.tail_tiles_m, 256 * t.big_tiles_m, rows - 256 * t.big_tiles_m, e)) return e;
    return launch(kTile128x128);
}

// Times the kernels launched while it lives (profile mode): from the start of the first to the end of the last,
// by the kernels' own time stamps (see LaunchEvents).
struct Prof {
    collm_ctx *c;
    int idx = -1;
    Prof(collm_ctx *c_, hipStream_t, const char *name) : c(c_)
    {
        if (name && c->profile && c->n_prof < kMaxProfile) {
            idx = c->n_prof++;
            c->prof_name[idx] = name;
            c->prof_launches[idx] = 0;
            g_launch_events = LaunchEvents{c->prof_ev[idx][0], c->prof_ev[idx][1], 0};
        }
    }
    ~Prof()
    {
        if (idx >= 0) {
            c->prof_launches[idx] = g_launch_events.launches;
            g_launch_events = LaunchEvents{};
        }
    }
    Prof(const Prof &) = delete;
    Prof &operator=(const Prof &) = delete;
};

int check_common(collm_ctx *ctx, const collm_shape *s, const void *x, const void *W,
                 const void *const *A, const void *const *B, const int32_t *rank,
                 const int32_t *seg_start, const int32_t *seg_adapter, const uint8_t *seg_is_train)
{
    if (!ctx || !s) return COLLM_E_NULL;
    if (s->dtype != COLLM_F32 && s->dtype != COLLM_BF16) return COLLM_E_DTYPE;
    const int q = s->dtype == COLLM_BF16 ? 8 : 4;
    if (s->d_in <= 0 || s->d_out <= 0 || s->d_in % q || s->d_out % q) return COLLM_E_SHAPE;
    if (s->layout != COLLM_LAYOUT_IN_OUT && s->layout != COLLM_LAYOUT_OUT_IN) return COLLM_E_SHAPE;
    if (s->d_in > ctx->max_d || s->d_out > ctx->max_d) return COLLM_E_SHAPE;
    if (s->n_tokens < 0 || s->n_tokens > ctx->max_tokens) return COLLM_E_SHAPE;
    {
        // the kernels address each operand tensor with 32-bit byte offsets below 2 GiB
        const int64_t lim = (int64_t)1 << 31, e = s->dtype == COLLM_BF16 ? 2 : 4;
        const int64_t dmax = std::max(s->d_in, s->d_out), dmin = std::min(s->d_in, s->d_out);
        if (((int64_t)s->n_tokens + 1) * dmax * e >= lim || (dmax + 128) * dmin * e >= lim) return COLLM_E_SHAPE;
    }
    if (s->n_segments < 0 || s->n_segments > ctx->max_segments) return COLLM_E_SHAPE;
    if (s->n_adapters < 0 || s->n_adapters > ctx->max_adapters) return COLLM_E_SHAPE;
    if (!seg_start) return COLLM_E_NULL;
    if (s->n_adapters > 0 && (!rank || !A || !B)) return COLLM_E_NULL;
    int rc = validate_batch(s, rank, seg_start, seg_adapter, seg_is_train, ctx->max_rank);
    if (rc != COLLM_OK) return rc;
    if (s->n_tokens > 0 && (!x || !W)) return COLLM_E_NULL;
    if (!aligned16(x) || !aligned16(W)) return COLLM_E_ALIGN;
    for (int k = 0; k < s->n_segments; ++k) {
        const int a = seg_adapter[k];
        if (a < 0 || seg_start[k + 1] == seg_start[k]) continue;
        if (!A[a] || !B[a]) return COLLM_E_ADAPTER;
        if (!aligned16(A[a]) || !aligned16(B[a])) return COLLM_E_ALIGN;
    }
    return COLLM_OK;
}

bool same_key(collm_ctx *c, const collm_shape *s, const void *const *A, const void *const *B,
              const int32_t *rank, const int32_t *seg_start, const int32_t *seg_adapter,
              const uint8_t *seg_is_train, int bm_all, int bm_train, int wide, bool fwd)
{
    if (!c->plan_valid) return false;
    const collm_shape &k = c->key_shape;
    if (k.d_in != s->d_in || k.d_out != s->d_out || k.n_tokens != s->n_tokens ||
        k.n_segments != s->n_segments || k.n_adapters != s->n_adapters || k.dtype != s->dtype)
        return false;
    // (a backward call runs over the training rows only: how the plan cuts all rows does not matter to it)
    if ((fwd && bm_all != c->key_bm_all) || bm_train != c->key_bm_train || wide != c->key_wide) return false;
    const int S = s->n_segments, N = s->n_adapters;
    if (std::memcmp(c->key_seg_start.data(), seg_start, sizeof(int32_t) * (S + 1))) return false;
    if (S && std::memcmp(c->key_seg_adapter.data(), seg_adapter, sizeof(int32_t) * S)) return false;
    if (S && std::memcmp(c->key_seg_train.data(), seg_is_train, S)) return false;
    if (N && std::memcmp(c->key_rank.data(), rank, sizeof(int32_t) * N)) return false;
    (void)A;
    (void)B;
    return true;
}

bool same_tables(collm_ctx *c, int N, const void *const *A, const void *const *B)
{
    for (int a = 0; a < N; ++a)
        if (c->key_A[a] != (uint64_t)(uintptr_t)A[a] || c->key_B[a] != (uint64_t)(uintptr_t)B[a]) return false;
    return true;
}

// Same batch, other adapter tables (another layer or projection of the model): the plan keeps its shape; the
// two pointer tables and the table address inside every extension step are replaced.
void patch_tables(collm_ctx *c, int N, const void *const *A, const void *const *B)
{
    PlanLayout &L = c->L;
    for (int a = 0; a < N; ++a) {
        const uint64_t va = (uint64_t)(uintptr_t)A[a], vb = (uint64_t)(uintptr_t)B[a];
        std::memcpy(c->plan.data() + L.off_A_ptr + 2 * a, &va, 8);
        std::memcpy(c->plan.data() + L.off_B_ptr + 2 * a, &vb, 8);
        c->key_A[a] = va;
        c->key_B[a] = vb;
    }
    auto patch = [&](int32_t off_ext, const std::vector<int32_t> &step_adapter, const void *const *tab) {
        ExtStep *ext = reinterpret_cast<ExtStep *>(c->plan.data() + off_ext);
        for (size_t k = 0; k < step_adapter.size(); ++k)
            if (step_adapter[k] >= 0) ext[k].tab = (uint64_t)(uintptr_t)tab[step_adapter[k]];  // (empty steps have no table)
    };
    patch(L.all.off_ext, L.all.ext_adapter, B);            // forward: expand tables
    patch(L.all.off_ext_half, L.all.ext_adapter_half, B);
    patch(L.train.off_ext, L.train.ext_adapter, A);        // backward: shrink tables
    patch(L.train.off_ext_half, L.train.ext_adapter_half, A);
}

// Takes the next pinned staging slot and a sequence number for it; waits until the GPU has copied what the slot held.
int take_slot(collm_ctx *c, int *slot, uint32_t *seq)
{
    const int sl = c->slot;
    c->slot = (c->slot + 1) % kSlots;
    if (c->stage_seq[sl] != 0) {
        // the slot is free once the upload that used it has been copied by the GPU
        const volatile uint32_t *done = c->h_done;
        int spins = 0;
        while ((int32_t)(*done - c->stage_seq[sl]) < 0) {
            if (++spins > 2000) {  // far behind: let the stream drain instead of spinning
                HIP_TRY(hipStreamSynchronize(c->last_stream));
                break;
            }
            std::this_thread::yield();
        }
    }
    *slot = sl;
    *seq = ++c->seq == 0 ? ++c->seq : c->seq;
    return COLLM_OK;
}

// Keeps `n` ints (a multiple of 4) of a plan for the replays of the call that is being recorded: their address as the device sees it, or null where
// the context's room for that is used up.  They stay until the context is destroyed (the library does not learn when a graph is).
const int32_t *keep_recorded(collm_ctx *c, const int32_t *src, size_t n)
{
    if (c->static_scratch) return nullptr;  // (allocates nothing)
    if (c->record_blocks.empty() || c->record_blocks.back().size - c->record_blocks.back().used < n) {
        const size_t bytes = std::max(n * sizeof(int32_t), kRecordBlock);
        if (c->record_bytes + bytes > kRecordBytes) return nullptr;
        RecordBlock b;
        b.size = bytes / sizeof(int32_t);
        c->record_blocks.reserve(c->record_blocks.size() + 1);
        // (the allocation is no part of what is being captured)
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) return nullptr;
        const bool ok = hipHostMalloc((void **)&b.host, bytes, hipHostMallocMapped) == hipSuccess &&
                        hipHostGetDevicePointer((void **)&b.dev, b.host, 0) == hipSuccess;
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (!ok) {
            (void)hipGetLastError();
            if (b.host) (void)hipHostFree(b.host);
            return nullptr;
        }
        c->record_blocks.push_back(b);
        c->record_bytes += bytes;
    }
    RecordBlock &b = c->record_blocks.back();
    std::memcpy(b.host + b.used, src, n * sizeof(int32_t));
    b.used += n;
    return b.dev + b.used - n;
}

// Copy ints [lo, hi) of the host plan to the device plan: through a pinned staging slot; for a call that is being recorded from pinned memory
// that no later upload overwrites; where there is none of either inside the arguments of a few small kernels.
int upload(collm_ctx *c, size_t lo, size_t hi, hipStream_t st, bool recording)
{
    if (hi <= lo) return COLLM_OK;
    const auto t0 = std::chrono::steady_clock::now();
    // rounded outwards to 16 bytes (the plan vector is padded to a multiple of 64 ints)
    const size_t lo4 = lo & ~(size_t)3, hi4 = std::min((hi + 3) & ~(size_t)3, c->plan.size());
    const int32_t *kept = recording ? keep_recorded(c, c->plan.data() + lo4, hi4 - lo4) : nullptr;
    if (kept) {
        HIP_TRY(launch_plan_copy(kept, c->d_plan + lo4, 0, hi4 - lo4, c->d_copy_counter, c->h_done_dev + 1, 0, st));
    } else if (c->static_scratch || recording) {
        HIP_TRY(launch_plan_words(c->plan.data() + lo4, c->d_plan + lo4, hi4 - lo4, st));
    } else {
        int sl = 0;
        uint32_t seq = 0;
        const int rc = take_slot(c, &sl, &seq);
        if (rc != COLLM_OK) return rc;
        std::memcpy(c->h_stage[sl] + lo4, c->plan.data() + lo4, (hi4 - lo4) * sizeof(int32_t));
        HIP_TRY(launch_plan_copy(c->h_stage_dev[sl], c->d_plan, lo4, hi4 - lo4, c->d_copy_counter, c->h_done_dev, seq, st));
        c->stage_seq[sl] = seq;
    }
    c->last_stream = st;
    c->plan_upload_us += std::chrono::duration<float, std::micro>(std::chrono::steady_clock::now() - t0).count();
    c->plan_bytes_up += (int)((hi4 - lo4) * sizeof(int32_t));
    return COLLM_OK;
}

// Leaves the plan's table addresses (patch_tables) to the call's first rank-wide pass (PlanPatch).  tab: the tables
// which that pass reads.
int stage_patch(collm_ctx *c, const void *const *tab, int n_adapters)
{
    const auto t0 = std::chrono::steady_clock::now();
    int sl = 0;
    uint32_t seq = 0;
    const int rc = take_slot(c, &sl, &seq);
    if (rc != COLLM_OK) return rc;
    const PlanLayout &L = c->L;
    PlanPatch &q = c->patch;
    int n16 = 0;
    auto part = [&](int i, int32_t off, size_t ints) {
        const size_t lo4 = (size_t)off & ~(size_t)3, hi4 = ints ? std::min(((size_t)off + ints + 3) & ~(size_t)3, c->plan.size()) : lo4;
        std::memcpy(c->h_stage[sl] + lo4, c->plan.data() + lo4, (hi4 - lo4) * sizeof(int32_t));
        q.lo[i] = (int32_t)(lo4 / 4);
        q.n[i] = (int32_t)((hi4 - lo4) / 4);
        n16 += q.n[i];
    };
    constexpr size_t kStepInts = sizeof(ExtStep) / sizeof(int32_t);
    part(0, L.off_A_ptr, (size_t)(L.off_dB_ptr - L.off_A_ptr) + 2 * (size_t)std::max(n_adapters, 1));
    part(1, L.all.off_ext, L.all.ext_adapter.size() * kStepInts);
    part(2, L.all.off_ext_half, L.all.ext_adapter_half.size() * kStepInts);
    part(3, L.train.off_ext, L.train.ext_adapter.size() * kStepInts);
    part(4, L.train.off_ext_half, L.train.ext_adapter_half.size() * kStepInts);
    q.src = c->h_stage_dev[sl];
    q.dst = c->d_plan;
    q.counter = c->d_copy_counter;
    q.done_host = c->h_done_dev;
    q.seq = seq;
    q.blocks = std::max(1, std::min(16, (n16 + 511) / 512));
    for (int a = 0; a < n_adapters; ++a) q.tab[a] = (uint64_t)(uintptr_t)tab[a];
    c->stage_seq[sl] = seq;
    c->plan_upload_us += std::chrono::duration<float, std::micro>(std::chrono::steady_clock::now() - t0).count();
    c->plan_bytes_up += n16 * 16;
    return COLLM_OK;
}

// Build (or reuse) the plan of this batch and put it on the device.
// pass_tab: null, or the call begins with a rank-wide pass over these tables, which can carry new addresses (run_skinny takes
// c->patch).  out_args: the call's kernels get the gradient buffers as arguments, not through the plan.
int prepare_plan(collm_ctx *c, const collm_shape *s, const void *const *A, const void *const *B,
                 const int32_t *rank, const int32_t *seg_start, const int32_t *seg_adapter,
                 const uint8_t *seg_is_train, float *const *dA, float *const *dB, bool allow_reuse,
                 hipStream_t st, bool fwd, const void *const *pass_tab, bool out_args, const int32_t *rank_ext_all = nullptr,
                 int n_sib = 1, bool swiglu = false, bool decode = false)
{
    const bool f32 = s->dtype == COLLM_F32;
    bool recording = false;
    unsigned long long capture_id = 0;
    if (st) {  // (the default stream cannot be recorded)
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        HIP_TRY(hipStreamIsCapturing(st, &capture));
        recording = capture != hipStreamCaptureStatusNone;
        if (recording) HIP_TRY(hipStreamGetCaptureInfo(st, &capture, &capture_id));
    }
    // whether the device holds the host's plan when this call's kernels run
    const bool known = recording ? capture_id != 0 && capture_id == c->capture_id : !c->recorded;
    c->recorded = c->recorded || recording;
    c->capture_id = capture_id;
    int n_train = 0;
    for (int k = 0; k < s->n_segments; ++k)
        if (seg_is_train[k]) n_train += seg_start[k + 1] - seg_start[k];
    const bool can_split = !f32 && c->gemm_split != 1, tr = s->layout == COLLM_LAYOUT_OUT_IN;
    count_steps(c, s, rank, seg_start, seg_adapter, seg_is_train);
    const int tile_fwd = c->tile_fwd >= 0 ? c->tile_fwd : choose_tiling(c, s->n_tokens, s->d_out, s->d_in, tr, !swiglu && n_sib <= 1, can_split && !swiglu, n_sib <= 1, c->tile_steps_all).tile;
    int rmax = 1;
    for (int a = 0; a < s->n_adapters; ++a) rmax = std::max(rmax, rank[a]);
    const bool one_round_dx = dx_one_round(c, n_train, s->d_in, s->d_out, f32, round_up(rmax, kKStep));
    const int tile_bwd = c->tile_bwd >= 0 ? c->tile_bwd : choose_tiling(c, n_train, s->d_in, s->d_out, !tr, true, can_split, one_round_dx, c->tile_steps_train).tile;
    const int bm_all = f32 ? 64 : gemm_tile_rows(tile_fwd);
    const int bm_train = f32 ? 64 : gemm_tile_rows(tile_bwd);
    // All rows of an adapter take the tiled rank-wide pass when ranks reach 64: there an adapter's table
    // outweighs 16 or 32 rows of activations several times, and the tiled pass fetches it once per 128 rows.
    // Narrow ranks waste its 128 columns of matrix work; measured, it still pays for the dh pass (tables
    // with K contiguous) from rank 32 up.  Encoded as all-rows threshold + 65536 * training-rows threshold.
    const int rpad_max = round_up(rmax, kKStep);
    const int wide_all = f32 || decode ? 0 : (c->wide_min_rows >= 0 ? c->wide_min_rows : (rpad_max >= 64 ? 1 : 0));
    const int wide_train = f32 ? 0 : (c->wide_min_rows >= 0 ? c->wide_min_rows : (rpad_max >= 32 ? 1 : 0));
    const int wide = wide_all + 65536 * wide_train;

    // A batch whose segment table, ranks, adapter tables and sizes equal those of the plan the device holds
    // reuses it (every layer and projection of a model sees the same batch): only a call on another stream
    // than the one the plan was uploaded on builds it again, since nothing orders the two streams.
    const bool reuse = allow_reuse && st == c->last_stream && n_sib == c->key_nsib &&
                       same_key(c, s, A, B, rank, seg_start, seg_adapter, seg_is_train, bm_all, bm_train, wide, fwd);
    bool new_tables = false;
    c->plan_build_us = c->plan_upload_us = 0.f;
    c->plan_mode = c->plan_bytes_up = 0;
    const auto t_plan = std::chrono::steady_clock::now();
    auto built = [&](int mode) {
        c->plan_mode = mode;
        c->plan_build_us = std::chrono::duration<float, std::micro>(std::chrono::steady_clock::now() - t_plan).count();
    };
    // (until what is new has been sent the device's plan is not the host's: a call that fails in between leaves no plan to reuse)
    c->plan_valid = false;
    if (reuse && !same_tables(c, s->n_adapters, A, B)) {
        patch_tables(c, s->n_adapters, A, B);
        new_tables = true;
        built(2);
    }
    if (!reuse) {
        PlanRequest rq;
        rq.shape = s;
        rq.rank = rank;
        rq.rank_ext_all = rank_ext_all;
        rq.seg_start = seg_start;
        rq.seg_adapter = seg_adapter;
        rq.seg_is_train = seg_is_train;
        rq.A = A;
        rq.B = B;
        rq.dA = dA;
        rq.dB = dB;
        rq.bm_all = bm_all;
        rq.bm_train = bm_train;
        rq.max_row_tiles = f32 ? 1 : skinny_max_row_tiles(round_up(rmax, kKStep));
        rq.wide_min_rows_all = wide_all;
        rq.wide_min_rows_train = wide_train;
        int rc = build_plan(rq, c->plan, c->L);
        if (rc != COLLM_OK) return rc;
        if ((size_t)c->L.total_ints > c->plan_cap) {
            g_last_error = "the plan of this batch is larger than the context's plan buffer";
            return COLLM_E_SHAPE;
        }
        built(1);
        rc = upload(c, 0, c->L.total_ints, st, recording);
        if (rc != COLLM_OK) return rc;
        // remember what this plan was built from
        const int S = s->n_segments, N = s->n_adapters;
        c->key_shape = *s;
        c->key_bm_all = bm_all;
        c->key_bm_train = bm_train;
        c->key_wide = wide;
        c->key_nsib = n_sib;
        c->key_seg_start.assign(seg_start, seg_start + S + 1);
        c->key_seg_adapter.assign(seg_adapter, seg_adapter + S);
        c->key_seg_train.assign(seg_is_train, seg_is_train + S);
        c->key_rank.assign(rank, rank + N);
        c->key_A.resize(N);
        c->key_B.resize(N);
        for (int a = 0; a < N; ++a) {
            c->key_A[a] = (uint64_t)(uintptr_t)A[a];
            c->key_B[a] = (uint64_t)(uintptr_t)B[a];
        }
    } else if (dA || dB || new_tables || !known) {
        // same batch as the host's plan: at most the pointer tables are new
        const int N = s->n_adapters;
        // (no row has an adapter: nothing runs)
        const RowOrderLayout &R = fwd ? c->L.all : c->L.train;
        const bool carry = new_tables && pass_tab && !f32 && !c->static_scratch && known && !recording && N <= kPatchTables && R.n_items + R.n_wide > 0;
        bool changed = false;
        for (int a = 0; a < (out_args ? 0 : N); ++a) {
            const uint64_t va = dA ? (uint64_t)(uintptr_t)dA[a] : 0, vb = dB ? (uint64_t)(uintptr_t)dB[a] : 0;
            changed |= std::memcmp(c->plan.data() + c->L.off_dA_ptr + 2 * a, &va, 8) != 0;
            changed |= std::memcmp(c->plan.data() + c->L.off_dB_ptr + 2 * a, &vb, 8) != 0;
            std::memcpy(c->plan.data() + c->L.off_dA_ptr + 2 * a, &va, 8);
            std::memcpy(c->plan.data() + c->L.off_dB_ptr + 2 * a, &vb, 8);
        }
        if (carry) {
            const int rc = stage_patch(c, pass_tab, N);
            if (rc != COLLM_OK) return rc;
        } else if (new_tables || !known) {
            int rc = upload(c, 0, c->L.total_ints, st, recording);
            if (rc != COLLM_OK) return rc;
        } else if (changed) {
            c->plan_mode = 3;
            int rc = upload(c, c->L.off_dA_ptr, (size_t)c->L.off_dB_ptr + 2 * (size_t)std::max(N, 1), st, recording);
            if (rc != COLLM_OK) return rc;
        }
    }
    c->plan_valid = true;
    c->last_stream = st;
    return COLLM_OK;
}

// A call that ends without having launched the pass that was to carry new addresses leaves a plan that is not whole.
struct PatchGuard {
    collm_ctx *c;
    ~PatchGuard()
    {
        if (c->patch.blocks > 0) c->plan_valid = false;
        c->patch.blocks = 0;
    }
};

// A rank-wide pass restricted to one of several sibling projections that lie side by side in the columns of
// dy and of the K-major tables: columns col0 .. col0 + K of rows of length ld.
struct SiblingPass {
    int n_sib = 0, sib = 0;
    int64_t ld = 0, col0 = 0;
    int rpad = 0;  // padded width of the widest single rank
};

// Partial sums of a rank-wide pass that another kernel has left in the layout of the pass's own K slices
// (part[(slice * part_rows + row) * part_ld + q]): run_skinny then only adds them up and stores.
struct SliceSums {
    float *part;
    int part_rows, part_ld, n_slices;
};

// One skinny pass over a row order.  beside (fp32): gradients that run in the same launch.
int run_skinny(collm_ctx *c, const collm_shape *s, const RowOrderLayout &R, const void *in, int K,
               int32_t off_tab, bool t_kmajor, float *f32_out, int64_t f32_ld, int f32_cols,
               int f32_by_token, float f32_mult, void *bf_out, float bf_mult, const char *name,
               hipStream_t st, const SiblingPass *sp = nullptr, const void *warm = nullptr, uint64_t warm_bytes = 0,
               const SliceSums *sums = nullptr, int bf_up = 0, const GradArgs *beside = nullptr)
{
    if (R.n_items == 0 && R.n_wide == 0) return COLLM_OK;
    // (taken by the call's first pass's first kernel; behind it the plan is whole)
    const PlanPatch *patch = c->patch.blocks > 0 ? &c->patch : nullptr;
    SkinnyArgs a{};
    // The weight of the GEMM that follows, fetched into the last-level cache by extra blocks of this pass (one per
    // compute unit) - if the weight is small (a GEMM of so few K tiles per block cannot hide the memory's latency:
    // 4096x4096 runs a fifth longer on a weight that comes from memory, 69 instead of 59 us) and this pass streams
    // less than the weight (it is then bound by latency and leaves the memory system idle; the fetch, about 12 us for
    // 33 MB, makes it 4 us longer).  Larger passes lose more than the GEMM gains (5120x5120, 8192 rows: +13 us / -11 us).
    const uint64_t pass_bytes = (uint64_t)R.n_rows * (uint64_t)K * (s->dtype == COLLM_BF16 ? 2 : 4);
    if (warm && warm_bytes <= kWarmMaxBytes && pass_bytes <= warm_bytes && c->n_cus > 0) {
        a.warm_base = warm;
        a.warm_bytes = warm_bytes;
        a.warm_blocks = c->n_cus;
    }
    const int64_t esz = s->dtype == COLLM_BF16 ? 2 : 4;
    a.in = in;
    a.ld_in = K;
    a.in_bytes = (uint32_t)((int64_t)s->n_tokens * K * esz);
    if (sp) {
        a.in = reinterpret_cast<const uint8_t *>(in) + sp->col0 * esz;
        a.ld_in = sp->ld;
        a.in_bytes = (uint32_t)((int64_t)s->n_tokens * sp->ld * esz - sp->col0 * esz);
        a.n_sib = sp->n_sib;
        a.sib = sp->sib;
        a.tab_ld = sp->ld;
        a.tab_off = sp->col0;
    }
    const int rpad = sp ? sp->rpad : c->L.rpad;
    a.K = K;
    a.tab = reinterpret_cast<const uint64_t *>(c->d_plan + off_tab);
    a.items = reinterpret_cast<const SkinnyItem *>(c->d_plan + R.off_items);
    a.row_tok = c->d_plan + R.off_row_tok;
    a.tok_train = c->d_plan + c->L.off_tok_train;
    a.f32_out = f32_out;
    a.f32_ld = f32_ld;
    a.f32_cols = f32_cols;
    a.f32_by_token = f32_by_token;
    a.f32_mult = f32_mult;
    a.bf_out = bf_out;
    a.bf_ld = c->L.rpad;
    a.bf_mult = bf_mult;
    a.bf_up = bf_up;
    // A wave keeps `depth` chunks of K in flight and so needs K / (waves * chunk * depth) round trips to memory; cutting K into
    // slices across blocks shortens that chain at the price of a second kernel that adds the slices (about 4 us with its launch).
    // Slices at all: as long as a wave keeps one chunk and the partial sums stay well below the bytes streamed (and inside the
    // workspace).
    //  - Chains of more than six round trips are cut where the items alone give fewer than 8 waves per CU (with more, the pass is
    //    bound by bandwidth and more, shorter blocks only scatter the stream), up to that many waves or down to about three trips.
    //  - Shorter ones, of blocks of eight waves (ranks to 32), are cut in four where that gives at most one block per CU, else in
    //    two on the same condition, if at least two round trips go away.  Forward call uncut / cut, us: rank 16, 128 rows
    //    5120 -> 5120 37.9 / 35.7, 500 rows 8192 -> 2048 [N][K] 52.1 / 45.0, 1003 rows 11008 -> 4096 142 / 136, 1003 rows
    //    8192 -> 4096 109.4 / 108.1; rank 24, 300 rows 7000 -> 504 40.2 / 31.1; forward and backward, 512 rows 5120 133.1 / 129.9,
    //    1200 rows 8192 292 / 287.  Outside: one trip less of three (1003 rows 5120, two slices) 76.7 / 77.3; 2048 -> 8192 49.6 /
    //    52; more blocks than CUs, 2000 rows 8192 207 / 211, 5120 rank 32 124.6 / 127; blocks of four waves, rank 40, 300 rows
    //    2560 -> 2560 77.0 / 80.8 with the backward.
    int n_split = 1;
    if (s->dtype == COLLM_BF16) {
        const int kw = skinny_waves(rpad);
        const int per_trip = kw * skinny_chunk(rpad) * skinny_depth(rpad, R.item_rows / kSkinnyRows);
        const long trips = (K + per_trip - 1) / per_trip;
        const long per_split = (long)c->rows_cap * c->rpad_cap * 4;
        long lim = std::min<long>(kSkinnyMaxSplit, (long)c->part_bytes / per_split);
        lim = std::min<long>(lim, K / (4L * rpad));
        lim = std::min<long>(lim, K / ((long)skinny_chunk(rpad) * kw));
        const long waves = (long)R.n_items * kw;
        if (trips > 6 && waves > 0 && waves < 2048) {
            n_split = (int)std::max<long>(1, std::min<long>({lim, (2048 + waves - 1) / waves, (trips + 2) / 3}));
        } else if (kw == 8) {
            const long n = std::min<long>(waves <= 512 ? 4 : (waves <= 1024 ? 2 : 1), lim);
            if (n > 1 && trips - (trips + n - 1) / n >= 2) n_split = (int)n;
        }
    }
    a.part = c->d_part;
    a.part_rows = c->rows_cap;
    a.part_ld = c->rpad_cap;
    if (sums) {
        // the slices are there already: only the kernel that adds them and does this pass's stores
        if (R.n_wide > 0 || s->dtype != COLLM_BF16) return COLLM_E_SHAPE;
        a.part = sums->part;
        a.part_rows = sums->part_rows;
        a.part_ld = sums->part_ld;
        HIP_TRY(launch_skinny_finish(a, nullptr, 0, 0, R.n_items, R.item_rows / kSkinnyRows, sums->n_slices, st));
        return COLLM_OK;
    }
    Prof prof(c, st, name);
    if (s->dtype == COLLM_F32) {
        a.n_items = R.n_items;
        HIP_TRY(beside ? launch_dh_dB_f32(a, *beside, rpad, t_kmajor, st) : launch_skinny_f32(a, R.n_items, t_kmajor, st));
        return COLLM_OK;
    }
    int n_wsplit = 1;
    // Both kinds of items in one launch where the 16-row items are narrow (ranks that are no multiples of 8 beside wide ones): each kind is
    // a short chain on a part of the CUs, and one behind the other they are two.  A block fills a CU; all of them run at once, with room for those
    // that put in new table addresses (112 blocks of 16-row items and 96, 144 tiled ones, 1367 rows of 11008 values: 17.7 / 25.7 us).  Half
    // of the places go to the 16-row items at most, cut until two round trips are left.  Passes with their sums, two launches / one, us: 1367 rows of
    // 11008 values, ranks 12, 20 and 64 29 / 23, 901 training rows of them 25 / 17, of 4104 values with [K][r] tables 29 / 15; whole passes of 30
    // batches of such ranks 1.12 (1.00 .. 1.34) times as fast.
    constexpr long kMixedPlaces = 224;
    const int rp_items = round_up(R.item_rank, kKStep);  // (their own ranks)
    bool mixed = R.n_wide > 0 && R.n_items > 0 && !sp && R.item_rows == kSkinnyRows && rp_items <= kMixedRank;
    if (mixed) {
        const long per_trip = 8L * skinny_chunk(rp_items) * skinny_depth(rp_items, 1);
        const long n = std::max<long>(1, std::min<long>({(K + 2 * per_trip - 1) / (2 * per_trip), kMixedPlaces / 2 / R.n_items, (long)kSkinnyMaxSplit,
                                                         (long)c->part_bytes / ((long)c->rows_cap * c->rpad_cap * 4)}));
        // (many items of a long contraction: slices in more than one round of smaller blocks are better, 27136 values of 1781 rows 1174 / 1191 us)
        mixed = (K + n * per_trip - 1) / (n * per_trip) <= 6;
        if (mixed) n_split = (int)n;
    }
    c->ran_mixed += mixed;
    if (R.n_items > 0) c->ran_pass_slices = std::max(c->ran_pass_slices, n_split);
    if (R.n_wide > 0) {
        // Long runs: 128-row tiles through the GEMM machinery.  A block fills a CU (four LDS stages), so K is cut
        // so that at most one block per CU exists, as long as a slice keeps 512 K values and the partial sums fit
        // the workspace; the small kernel that adds the slices also does this pass's stores.
        GemmArgs g{};
        g.a = a.in;
        g.lda = a.ld_in;
        g.K = K;
        g.a_bytes = a.in_bytes;
        g.row_tok = a.row_tok;
        g.items = reinterpret_cast<const SkinnyItem *>(c->d_plan + R.off_wide);
        g.tab = a.tab;
        g.part = a.part;
        g.part_rows = a.part_rows;
        g.part_ld = a.part_ld;
        g.part_n_sib = a.n_sib;
        g.tab_ld = a.tab_ld;
        g.tab_off = a.tab_off;
        // (the warm-up rides with the tiled pass when there is one, else with the 16-row items)
        g.warm_base = a.warm_base;
        g.warm_bytes = a.warm_bytes;
        g.warm_blocks = a.warm_blocks;
        a.warm_blocks = 0;
        const long blocks = (long)R.n_wide * ((rpad + 127) / 128);
        const long per_split = (long)c->rows_cap * c->rpad_cap * 4;
        // (one block per CU with K-major tables, two with tables as they lie in memory: see launch_wide)
        const long places = mixed ? kMixedPlaces - std::min<long>((long)R.n_items * n_split, kMixedPlaces / 2) : (t_kmajor ? 256 : 512);
        long ns = std::min<long>({places / blocks, std::max(1, K / 512), (long)c->part_bytes / per_split, (long)kSkinnyMaxSplit});
        ns = std::max<long>(ns, 1);
        g.k_per_split = round_up((int)((K + ns - 1) / ns), 64);
        n_wsplit = (K + g.k_per_split - 1) / g.k_per_split;
        a.n_items = R.n_items;
        HIP_TRY(launch_wide(g, R.n_wide, rpad, n_wsplit, t_kmajor, st, patch, mixed ? &a : nullptr, rp_items, n_split));
        c->patch.blocks = 0;
        patch = nullptr;
    }
    if (R.n_items > 0 && !mixed) {
        HIP_TRY(launch_skinny(a, R.n_items, rpad, R.item_rows / kSkinnyRows, n_split, t_kmajor, st, patch));
        c->patch.blocks = 0;
    }
    // (the sums of the two kinds of items lie in different rows of the workspace)
    HIP_TRY(launch_skinny_finish(a, reinterpret_cast<const SkinnyItem *>(c->d_plan + R.off_wide), R.n_wide, n_wsplit,
                                 mixed || n_split > 1 ? R.n_items : 0, R.item_rows / kSkinnyRows, n_split, st));
    return COLLM_OK;
}


// How the first kernel of a decode-sized call is cut: slices of K of each of the weight's strips, and of each of the shrink's `items`.  A block fills
// a CU, and the two kinds share the CUs.  Both numbers are taken by estimate (us):
//  - a round of 256 values takes 1 .. 2.5 by the number of rows, a third more with [N][K] weights, and no less than the memory needs for what the
//    blocks that run at once ask for (1.4 with a few, 2.7 with 256: 9656 -> 14256 in 112 blocks 84 us, in 224 55); a block 2 beside its rounds.
//  - one round of blocks, or up to two where one would leave a quarter of the CUs idle (18312 -> 18120, 142 strips, 148 uncut, 126 in three slices: the
//    second, partial round reads from memory beside the first); a slice keeps 192 values.
//  - a block of the shrink 2 and a chunk of its 64 values 0.4 for ranks up to 16, else 1.3.
//  - the second kernel: 0.8 a trip to memory (decode_sum_trips, of the largest item), or the sums' bytes (15104 -> 768, 34 rows: 31 us in 24 slices, 26 in ten).
// No places are kept for the blocks that put in new table addresses (up to 16, short): four layers of 64 rows 4096 -> 11008 with tables of their own 167
// us either way, and a call's sums must not depend on whether its tables are new.
// 386 drawn calls of 1 to 64 rows, weights from memory: 0.98 of the best of the cuts tried; 260 others 1.32 times as fast as the general path (0.90 at
// the least), 1.04 times as with slices for one round by chains and bytes alone.
struct DecodeCut {
    int n_slices, k_per_slice, h_slices;
};
DecodeCut decode_cut(int T, int N, int K, bool kmajor, int rpad, int items, int item_rows, int cus, int64_t room)
{
    const int strips = (N + kDecodeCols - 1) / kDecodeCols;
    const int64_t rows_h = (int64_t)round_up(T, 16) * rpad, rows_y = (int64_t)T * N;  // floats of a slice
    const double round_us = (T <= 16 ? 1.0 : (T <= 32 ? 1.6 : 2.5)) * (kmajor ? 1.3 : 1.0), chunk_us = rpad <= 16 ? 0.4 : 1.3;
    DecodeCut best{1, 0, 1};
    double best_us = 1e30, shrink[9];
    long most[9];
    int h_most = 0;
    for (int h = 1; h <= 8 && (h == 1 || (items > 0 && h * 512 <= K && h * items < cus && h * rows_h + rows_y <= room)); h_most = h++) {
        const long one = std::max(0L, (cus - (long)h * items) / strips);  // slices in one round
        const long places = one * strips < cus * 3 / 4 ? 2L * cus / strips : one;
        most[h] = std::max(1L, std::min<long>({places, (long)K / 192, (long)((room - h * rows_h) / rows_y)}));
        shrink[h] = items > 0 ? 2.0 + chunk_us * ((K + 256 * h - 1) / (256 * h)) : 0.0;
    }
    for (long n = 1; n <= most[1]; n += n < 16 ? 1 : 4) {  // (the fewer slices of the shrink, the more there may be of the strips)
        const long blocks = strips * n, rounds = (round_up((int)((K + n - 1) / n), 64) + 255) / 256;
        auto at_once = [&](long b) { return b > 0 ? rounds * std::max(round_us, 1.4 + 0.005 * b) + 2.0 : 0.0; };
        const double base = (blocks / cus) * at_once(cus) + at_once(blocks % cus);
        const double sums = std::max((double)n * rows_y * 8 / 4.0e6, 0.8 * decode_sum_trips(item_rows, (int)n));
        for (int h = 1; h <= h_most; ++h) {
            const double us = (blocks + (long)h * items <= cus ? std::max(base, shrink[h]) : base + 0.7 * shrink[h]) + sums;
            if (n <= most[h] && us < best_us) {
                best = {(int)n, 0, h};
                best_us = us;
            }
        }
    }
    best.k_per_slice = round_up((K + best.n_slices - 1) / best.n_slices, 64);
    best.n_slices = (K + best.k_per_slice - 1) / best.k_per_slice;
    return best;
}

// The two kernels of a decode-sized inference call.
int run_decode(collm_ctx *c, const collm_shape *s, const void *x, const void *W, const void *const *B, void *y, hipStream_t st)
{
    const PlanLayout &L = c->L;
    const RowOrderLayout &R = L.all;
    const bool tr = s->layout == COLLM_LAYOUT_OUT_IN;
    const int T = s->n_tokens, N = s->d_out, K = s->d_in;
    const int strips = (N + kDecodeCols - 1) / kDecodeCols, rows_h = round_up(T, 16);
    const int h_cols = L.rpad <= 16 ? 1 : (L.rpad + kDecodeRankCols - 1) / kDecodeRankCols;
    const SkinnyItem *items = reinterpret_cast<const SkinnyItem *>(c->plan.data() + R.off_items);
    int item_rows = std::min(R.n_base, 16);
    for (int i = 0; i < R.n_items; ++i) item_rows = std::max(item_rows, items[i].n_rows);
    const DecodeCut cut = decode_cut(T, N, K, tr, L.rpad, R.n_items * h_cols, item_rows, std::max(c->n_cus, 1), (int64_t)c->part_bytes / 4);
    const int n_slices = cut.n_slices;
    SkinnyArgs a{};
    a.in = x;
    a.ld_in = s->d_in;
    a.in_bytes = (uint32_t)((int64_t)s->n_tokens * s->d_in * 2);
    a.K = s->d_in;
    a.tab = reinterpret_cast<const uint64_t *>(c->d_plan + L.off_A_ptr);
    a.items = reinterpret_cast<const SkinnyItem *>(c->d_plan + R.off_items);
    a.n_items = R.n_items;
    a.row_tok = c->d_plan + R.off_row_tok;
    DecodeFinishArgs d;
    d.w = W;
    d.ldw = tr ? s->d_in : s->d_out;
    d.w_bytes = (uint32_t)((int64_t)s->d_in * s->d_out * 2);
    d.N = s->d_out;
    d.y = y;
    d.n_rows = s->n_tokens;
    d.part = c->d_part;
    d.strips = strips;
    d.n_slices = n_slices;
    d.k_per_slice = cut.k_per_slice;
    d.h_slices = cut.h_slices;
    d.h_cols = h_cols;
    d.scale = s->scale;
    d.n_base = R.n_base;
    for (int i = 0; i < R.n_items; ++i)
        d.items[i] = {(uint32_t)items[i].row_lo | (uint32_t)items[i].n_rows << 16, (uint32_t)items[i].rank, (uint64_t)(uintptr_t)B[items[i].adapter]};
    // the shrink's sums behind those of the slices
    a.part = c->d_part + (int64_t)n_slices * T * N;
    a.part_rows = rows_h;
    a.part_ld = L.rpad;
    Prof prof(c, st, "decode");
    HIP_TRY(launch_decode_base(a, d, L.rpad, tr, st, c->patch.blocks > 0 ? &c->patch : nullptr));
    c->patch.blocks = 0;
    HIP_TRY(launch_decode_finish(a, d, tr, st));
    return COLLM_OK;
}

// Sibling projections (several projections of the same x side by side in the columns of W, y and dy).  Checks
// the description and fills c->sum_rank with the ranks summed over the siblings, which is what the rank-wide
// passes over all siblings, the plan and the context's limits see.
int prepare_siblings(collm_ctx *c, const collm_shape *s, const collm_siblings *sib, const int32_t *rank)
{
    if (!c || !s || !sib) return COLLM_E_NULL;
    if (s->dtype != COLLM_BF16) return COLLM_E_DTYPE;
    if (s->layout != COLLM_LAYOUT_IN_OUT) return COLLM_E_SHAPE;
    const bool swiglu = sib->activation == COLLM_ACT_SWIGLU;
    if (sib->activation != COLLM_ACT_NONE && !swiglu) return COLLM_E_SHAPE;
    const int P = sib->n_siblings;
    if (P < 1 || P > COLLM_MAX_SIBLINGS) return COLLM_E_SHAPE;
    if (swiglu && (P != 2 || sib->d_out[0] != sib->d_out[1])) return COLLM_E_SHAPE;
    if (!aligned16(sib->pre_act)) return COLLM_E_ALIGN;
    int64_t sum = 0;
    for (int j = 0; j < P; ++j) {
        if (sib->d_out[j] <= 0 || sib->d_out[j] % 8) return COLLM_E_SHAPE;
        if (j + 1 < P && sib->d_out[j] % 256) return COLLM_E_SHAPE;  // a column tile belongs to one sibling
        sum += sib->d_out[j];
    }
    if (sum != s->d_out) return COLLM_E_SHAPE;
    if (s->n_adapters < 0 || s->n_adapters > c->max_adapters) return COLLM_E_SHAPE;
    if (s->n_adapters > 0 && !rank) return COLLM_E_NULL;
    c->sum_rank.resize((size_t)std::max(s->n_adapters, 1));
    for (int a = 0; a < s->n_adapters; ++a) {
        if (rank[a] < 1 || rank[a] > c->max_rank || (P > 1 && rank[a] % 8) || (swiglu && rank[a] % 16))
            return COLLM_E_RANK;
        c->sum_rank[a] = rank[a] * P;
    }
    return COLLM_OK;
}

}  // namespace

// -----------------------------------------------------------------------------------------
// Workspace of collm_lora_linear_fwd_noalloc: one array per GPU the library is loaded on, held until the
// process ends.  The name is a host-side stand-in, not a device address: the address on a device comes from
// hipGetSymbolAddress with that device current, once per device, and is what the kernels receive.
namespace {
constexpr size_t kScratchBytes = (size_t)16 << 20;
constexpr int kScratchMaxTokens = 2048, kScratchMaxSegments = 2048, kScratchMaxAdapters = 64, kScratchMaxRank = 64,
              kScratchMaxD = 16384;
constexpr size_t kScratchZerosOff = 0, kScratchPlanOff = 4096, kScratchPlanBytes = (size_t)256 << 10,
                 kScratchHsOff = kScratchPlanOff + kScratchPlanBytes,
                 kScratchHsBytes = (size_t)kScratchMaxTokens * kScratchMaxRank * 4,
                 kScratchPartOff = kScratchHsOff + kScratchHsBytes, kScratchPartBytes = kScratchBytes - kScratchPartOff;
static_assert(kScratchMaxTokens % kRowPad == 0 && kScratchMaxRank % kKStep == 0, "limits are padded sizes already");
static_assert(kScratchPartOff % 256 == 0 && kScratchHsOff % 256 == 0, "every region is 256-byte aligned");
constexpr int kMaxDevices = 64;
}  // namespace
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
namespace {
std::mutex g_scratch_mutex;
collm_ctx *g_scratch_ctx[kMaxDevices] = {};

// The per-device context of the entry point that allocates nothing: host bookkeeping only, every device pointer
// lies inside that device's copy of `scratch`.  Set up at the first call on the device.
int scratch_context(int device, hipStream_t st, collm_ctx **out)
{
    if (device < 0 || device >= kMaxDevices) return COLLM_E_SHAPE;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ctx[device]) {
        HIP_TRY(hipSetDevice(device));
        unsigned char *ptr = nullptr;
        HIP_TRY(hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch)));
        if (!ptr || ((uintptr_t)ptr & 255u)) {
            g_last_error = "address of the static scratch array is null or misaligned";
            return COLLM_E_HIP;
        }
        collm_ctx *c = new (std::nothrow) collm_ctx();
        if (!c) return COLLM_E_NOMEM;
        c->device = device;
        c->static_scratch = true;
        c->max_tokens = kScratchMaxTokens;
        c->max_segments = kScratchMaxSegments;
        c->max_adapters = kScratchMaxAdapters;
        c->max_rank = kScratchMaxRank;
        c->max_d = kScratchMaxD;
        c->rows_cap = kScratchMaxTokens;
        c->rpad_cap = kScratchMaxRank;
        c->plan_cap = kScratchPlanBytes / sizeof(int32_t);
        c->d_zeros = ptr + kScratchZerosOff;
        c->d_plan = reinterpret_cast<int32_t *>(ptr + kScratchPlanOff);
        c->d_hs = ptr + kScratchHsOff;
        c->d_part = reinterpret_cast<float *>(ptr + kScratchPartOff);
        c->part_bytes = kScratchPartBytes;
        if (hipDeviceGetAttribute(&c->n_cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) c->n_cus = 0;
        c->workspace_bytes = (int64_t)kScratchBytes;
        // host vectors at their largest size, so that later calls do not grow them
        c->plan.reserve(c->plan_cap);
        c->rows_of.reserve(2 * kScratchMaxAdapters);
        c->key_seg_start.reserve(kScratchMaxSegments + 1);
        c->key_seg_adapter.reserve(kScratchMaxSegments);
        c->key_seg_train.reserve(kScratchMaxSegments);
        c->key_rank.reserve(kScratchMaxAdapters);
        c->key_A.reserve(kScratchMaxAdapters);
        c->key_B.reserve(kScratchMaxAdapters);
        // the block of zeros that masked 16-byte loads read (a small fill kernel, in stream order before any use)
        hipError_t e = launch_fill_zero(c->d_zeros, 256, st);
        if (e != hipSuccess) {
            delete c;
            return hip_fail(e, "launch_fill_zero");
        }
        g_scratch_ctx[device] = c;
    }
    *out = g_scratch_ctx[device];
    return COLLM_OK;
}
}  // namespace

// -----------------------------------------------------------------------------------------
extern "C" {

const char *collm_status_string(int status)
{
    switch (status) {
    case COLLM_OK: return "ok";
    case COLLM_E_NULL: return "a required pointer is NULL";
    case COLLM_E_SHAPE: return "unsupported size, or beyond what the context was created for";
    case COLLM_E_SEGMENTS: return "bad segment table";
    case COLLM_E_ADAPTER: return "bad adapter index or missing adapter table";
    case COLLM_E_RANK: return "rank out of range";
    case COLLM_E_DTYPE: return "unknown element type";
    case COLLM_E_ALIGN: return "device pointer not 16-byte aligned";
    case COLLM_E_HIP: return "HIP call failed";
    case COLLM_E_NOMEM: return "allocation failed";
    default: return "unknown status";
    }
}

const char *collm_last_error(void) { return g_last_error.c_str(); }

int collm_token_map(const collm_shape *shape, const int32_t *seg_start, const int32_t *seg_adapter,
                    const uint8_t *seg_is_train, int32_t *tok_segment, int32_t *tok_adapter,
                    uint8_t *tok_is_train)
{
    if (!shape || !seg_start) return COLLM_E_NULL;
    int rc = validate_batch(shape, nullptr, seg_start, seg_adapter, seg_is_train, kMaxRank);
    if (rc != COLLM_OK) return rc;
    if (shape->n_tokens > 0 && (!tok_segment || !tok_adapter || !tok_is_train)) return COLLM_E_NULL;
    token_map(shape, seg_start, seg_adapter, seg_is_train, tok_segment, tok_adapter, tok_is_train);
    return COLLM_OK;
}

int collm_ctx_create(collm_ctx **out, int device, int32_t max_tokens, int32_t max_segments,
                     int32_t max_adapters, int32_t max_rank, int32_t max_d)
{
    if (!out) return COLLM_E_NULL;
    *out = nullptr;
    if (max_tokens < 1 || max_segments < 1 || max_adapters < 0 || max_d < 1) return COLLM_E_SHAPE;
    if (max_rank < 1 || max_rank > kMaxRank) return COLLM_E_RANK;
    HIP_TRY(hipSetDevice(device));
    collm_ctx *c = new (std::nothrow) collm_ctx();
    if (!c) return COLLM_E_NOMEM;
    c->device = device;
    c->max_tokens = max_tokens;
    c->max_segments = max_segments;
    c->max_adapters = max_adapters;
    c->max_rank = max_rank;
    c->max_d = max_d;
    c->rows_cap = round_up(max_tokens, kRowPad);
    c->rpad_cap = round_up(max_rank, kKStep);
    c->plan_cap = plan_ints_upper_bound(max_tokens, max_segments, max_adapters, max_rank);
    if (hipDeviceGetAttribute(&c->n_cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) c->n_cus = 0;

    auto fail = [&](int rc) {
        collm_ctx_destroy(c);
        return rc;
    };
    int64_t ws = 0;
    auto dev_alloc = [&](void **p, size_t bytes) -> hipError_t {
        ws += (int64_t)bytes;
        return hipMalloc(p, bytes);
    };
    for (int i = 0; i < kSlots; ++i) {
        if (hipHostMalloc((void **)&c->h_stage[i], c->plan_cap * sizeof(int32_t), hipHostMallocMapped) != hipSuccess)
            return fail(COLLM_E_NOMEM);
        if (hipHostGetDevicePointer((void **)&c->h_stage_dev[i], c->h_stage[i], 0) != hipSuccess) return fail(COLLM_E_HIP);
    }
    if (hipHostMalloc((void **)&c->h_done, 64, hipHostMallocMapped) != hipSuccess) return fail(COLLM_E_NOMEM);
    *c->h_done = 0;
    if (hipHostGetDevicePointer((void **)&c->h_done_dev, c->h_done, 0) != hipSuccess) return fail(COLLM_E_HIP);
    const size_t act = (size_t)c->rows_cap * c->rpad_cap;
    // partial sums of the K slices: room for kSkinnyMaxSplit slices, but no more than 64 MiB (at least one)
    c->part_bytes = std::max(act * 4, std::min(act * 4 * kSkinnyMaxSplit, (size_t)64 << 20));
    // ... and of a GEMM with few rows: up to 8 slices of 512 rows of the widest output
    c->part_bytes = std::max(c->part_bytes, std::min((size_t)std::min(c->rows_cap, 512) * (size_t)max_d * 4 * 8, (size_t)64 << 20));
    if (dev_alloc((void **)&c->d_plan, c->plan_cap * sizeof(int32_t)) != hipSuccess ||
        dev_alloc(&c->d_hs, act * 4) != hipSuccess || dev_alloc(&c->d_dhs, act * 4) != hipSuccess ||
        dev_alloc((void **)&c->d_h32, act * 4) != hipSuccess ||
        dev_alloc((void **)&c->d_dh32, act * 4) != hipSuccess ||
        dev_alloc((void **)&c->d_copy_counter, 64) != hipSuccess || dev_alloc(&c->d_zeros, 256) != hipSuccess ||
        dev_alloc((void **)&c->d_part, c->part_bytes) != hipSuccess)
        return fail(COLLM_E_NOMEM);
    if (hipMemset(c->d_copy_counter, 0, 64) != hipSuccess) return fail(COLLM_E_HIP);
    if (hipMemset(c->d_zeros, 0, 256) != hipSuccess) return fail(COLLM_E_HIP);
    // the events order the two streams of this GPU and nothing else: no system-scope cache flush when they are recorded
    // (the gaps they leave on the caller's stream shrink from 6-7 to 4-5 us; whoever waits for the caller's stream
    // gets that flush from the wait)
    constexpr unsigned kOrderOnly = hipEventDisableTiming | hipEventDisableSystemFence;
    if (hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_fork, kOrderOnly) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_dh, kOrderOnly) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_join, kOrderOnly) != hipSuccess)
        return fail(COLLM_E_HIP);
    if (hipDeviceSynchronize() != hipSuccess) return fail(COLLM_E_HIP);
    c->workspace_bytes = ws;
    *out = c;
    return COLLM_OK;
}

int collm_ctx_destroy(collm_ctx *c)
{
    if (!c) return COLLM_OK;
    (void)hipSetDevice(c->device);
    (void)hipDeviceSynchronize();
    for (int i = 0; i < kSlots; ++i) {
        if (c->h_stage[i]) (void)hipHostFree(c->h_stage[i]);
    }
    for (const RecordBlock &b : c->record_blocks) (void)hipHostFree(b.host);
    if (c->h_done) (void)hipHostFree(c->h_done);
    if (c->side) (void)hipStreamDestroy(c->side);
    for (hipEvent_t e : {c->ev_fork, c->ev_dh, c->ev_join})
        if (e) (void)hipEventDestroy(e);
    if (c->prof_ev_made)
        for (int i = 0; i < kMaxProfile; ++i) {
            (void)hipEventDestroy(c->prof_ev[i][0]);
            (void)hipEventDestroy(c->prof_ev[i][1]);
        }
    void *bufs[] = {c->d_plan, c->d_hs, c->d_dhs, c->d_h32, c->d_dh32, c->d_copy_counter, c->d_zeros, c->d_part};
    for (void *b : bufs)
        if (b) (void)hipFree(b);
    delete c;
    return COLLM_OK;
}

int64_t collm_ctx_workspace_bytes(const collm_ctx *c) { return c ? c->workspace_bytes : 0; }

int collm_debug_host_tile_order(int tile_rows, int tiles_m, int tiles_n, int K, int band, int32_t *band_used,
                                int32_t *tile_m, int32_t *tile_n)
{
    if (!band_used || !tile_m || !tile_n) return COLLM_E_NULL;
    if (tiles_m <= 0 || tiles_n <= 0 || K <= 0 || (tile_rows != 128 && tile_rows != 256) ||
        (int64_t)tiles_m * tiles_n > (1 << 24) || (band >= 0 && band % 8 != 0))
        return COLLM_E_SHAPE;
    *band_used = band >= 0 ? band : gemm_band_rows(tile_rows, K, tiles_m);
    host_tile_order(tiles_m, tiles_n, *band_used, tile_m, tile_n);
    return COLLM_OK;
}

int collm_debug_host_shared_order(int tiles_m, int tiles_n, int n_slices, int K, int grad_blocks, int32_t *slice, int32_t *tile_m,
                                  int32_t *tile_n, int32_t *grad)
{
    if (!slice || !tile_m || !tile_n || !grad) return COLLM_E_NULL;
    if (tiles_m <= 0 || tiles_n <= 0 || n_slices < 1 || K <= 0 || grad_blocks < 0 ||
        (int64_t)tiles_m * tiles_n * n_slices + grad_blocks > (1 << 24))
        return COLLM_E_SHAPE;
    return host_shared_order(tiles_m, tiles_n, n_slices, K, grad_blocks, slice, tile_m, tile_n, grad);
}

int collm_debug_host_tiling(int rows, int cols, int K, int can_split, int32_t *tile, int32_t *big_tiles_m,
                            int32_t *tail_tiles_m, int32_t *tail_cols)
{
    if (!tile || !big_tiles_m || !tail_tiles_m || !tail_cols) return COLLM_E_NULL;
    if (rows < 0 || cols <= 0 || K <= 0) return COLLM_E_SHAPE;
    const Tiling t = pick_tiling(rows, cols, K, can_split != 0, false, 0);
    *tile = t.tile;
    *big_tiles_m = t.big_tiles_m;
    *tail_tiles_m = t.tail_tiles_m;
    *tail_cols = t.tail_cols;
    return COLLM_OK;
}

int collm_debug_host_gemm_slices(int tiles_m, int cols, int K, int b_kmajor, int steps, int64_t workspace_bytes, int32_t *slices)
{
    if (!slices) return COLLM_E_NULL;
    if (tiles_m <= 0 || cols <= 0 || K <= 0 || steps < 0 || workspace_bytes < 0) return COLLM_E_SHAPE;
    *slices = (int32_t)std::max(1L, gemm_slices(-1, workspace_bytes, tiles_m, cols, K, b_kmajor != 0, steps, nullptr));
    return COLLM_OK;
}

int collm_debug_host_plain_gemm(int rows, int cols, int K, int b_kmajor, int steps, int64_t workspace_bytes, int32_t *tile, int32_t *slices,
                                int32_t *one_per_cu)
{
    if (!tile || !slices || !one_per_cu) return COLLM_E_NULL;
    if (rows <= 0 || cols <= 0 || K <= 0 || steps < 0 || workspace_bytes < 0) return COLLM_E_SHAPE;
    const Tiling t = choose_tiling(-1, workspace_bytes, rows, cols, K, b_kmajor != 0, true, true, true, (int)((steps + (rows + 127) / 128 - 1) / ((rows + 127) / 128)));
    *tile = t.tile;
    *slices = t.slices;
    *one_per_cu = t.slices > 1;
    if (t.tile == kTile128x128 && t.tail_tiles_m == 0) {
        bool alone = false;
        *slices = (int32_t)std::max(1L, gemm_slices(-1, workspace_bytes, t.big_tiles_m, cols, K, b_kmajor != 0, steps, &alone));
        *one_per_cu = *slices > 1 ? alone : ring_alone(t, cols, K, steps / t.big_tiles_m);
    }
    return COLLM_OK;
}

int collm_debug_host_grad_lds(int rank, int beside_gemm, int32_t *bytes)
{
    if (!bytes) return COLLM_E_NULL;
    if (rank < 1 || rank > kMaxRank) return COLLM_E_RANK;
    *bytes = grad_lds(round_up(rank, kKStep), beside_gemm != 0);
    return COLLM_OK;
}

int collm_debug_host_grad_streams(int n_train, int d_in, int d_out, int dtype, int max_rank, int32_t *streams)
{
    if (!streams) return COLLM_E_NULL;
    if (n_train < 0 || d_in <= 0 || d_out <= 0) return COLLM_E_SHAPE;
    if (dtype != COLLM_F32 && dtype != COLLM_BF16) return COLLM_E_DTYPE;
    if (max_rank < 1 || max_rank > kMaxRank) return COLLM_E_RANK;
    *streams = grads_alone(n_train, d_in, d_out, dtype == COLLM_F32, round_up(max_rank, kKStep)) ? 1 : 2;
    return COLLM_OK;
}

int collm_debug_host_row_order(const collm_shape *s, const int32_t *rank, const int32_t *seg_start,
                               const int32_t *seg_adapter, const uint8_t *seg_is_train, int tile_rows,
                               int training_rows_only, int32_t *row_tok, int32_t *tile_steps)
{
    if (!s || !seg_start || !row_tok || !tile_steps) return COLLM_E_NULL;
    if (tile_rows != 64 && tile_rows != 128 && tile_rows != 256) return COLLM_E_SHAPE;
    int rc = validate_batch(s, rank, seg_start, seg_adapter, seg_is_train, 256);
    if (rc != COLLM_OK) return rc;
    PlanRequest rq;
    rq.shape = s;
    rq.rank = rank;
    rq.seg_start = seg_start;
    rq.seg_adapter = seg_adapter;
    rq.seg_is_train = seg_is_train;
    rq.bm_all = rq.bm_train = tile_rows;
    std::vector<int32_t> plan;
    PlanLayout L;
    rc = build_plan(rq, plan, L);
    if (rc != COLLM_OK) return rc;
    const RowOrderLayout &R = training_rows_only ? L.train : L.all;
    for (int i = 0; i < R.n_rows; ++i) row_tok[i] = plan[R.off_row_tok + i];
    const int n_tiles = (R.n_rows + tile_rows - 1) / tile_rows;
    for (int t = 0; t < n_tiles; ++t) tile_steps[t] = plan[R.off_ext_off + t + 1] - plan[R.off_ext_off + t];
    return R.n_rows;
}

int collm_debug_set_tiles(collm_ctx *c, int fwd_tile, int bwd_tile)
{
    if (!c) return COLLM_E_NULL;
    auto ok = [](int t) { return t >= -1 && t <= kTile256x192; };
    if (!ok(fwd_tile) || !ok(bwd_tile)) return COLLM_E_SHAPE;
    c->tile_fwd = fwd_tile;
    c->tile_bwd = bwd_tile;
    return COLLM_OK;
}

int collm_debug_set_gemm_split(collm_ctx *c, int n_slices)
{
    if (!c) return COLLM_E_NULL;
    if (n_slices < -1 || n_slices == 0 || n_slices > 64) return COLLM_E_SHAPE;
    c->gemm_split = n_slices;
    return COLLM_OK;
}

int collm_debug_set_dual_pass(collm_ctx *c, int mode)
{
    if (!c) return COLLM_E_NULL;
    if (mode < -1 || mode > 1) return COLLM_E_SHAPE;
    c->dual_pass = mode;
    return COLLM_OK;
}

int collm_debug_set_grad_streams(collm_ctx *c, int mode)
{
    if (!c) return COLLM_E_NULL;
    if (mode < -1 || mode > 1) return COLLM_E_SHAPE;
    c->grad_streams = mode;
    return COLLM_OK;
}

int collm_debug_set_wide_pass(collm_ctx *c, int min_rows)
{
    if (!c) return COLLM_E_NULL;
    if (min_rows < -1 || min_rows > 65535) return COLLM_E_SHAPE;
    c->wide_min_rows = min_rows;
    return COLLM_OK;
}

int collm_device_info(int device, int32_t *compute_units, int32_t *clock_khz, int32_t *memory_clock_khz,
                      int32_t *memory_bus_bits, int64_t *l2_bytes)
{
    if (!compute_units || !clock_khz || !memory_clock_khz || !memory_bus_bits || !l2_bytes) return COLLM_E_NULL;
    hipDeviceProp_t pr;
    HIP_TRY(hipGetDeviceProperties(&pr, device));
    *compute_units = pr.multiProcessorCount;
    *clock_khz = pr.clockRate;
    *memory_clock_khz = pr.memoryClockRate;
    *memory_bus_bits = pr.memoryBusWidth;
    *l2_bytes = pr.l2CacheSize;
    return COLLM_OK;
}

int collm_debug_plan_stats(const collm_ctx *c, float *build_us, float *upload_us, int32_t *bytes, int32_t *mode)
{
    if (!c || !build_us || !upload_us || !bytes || !mode) return COLLM_E_NULL;
    *build_us = c->plan_build_us;
    *upload_us = c->plan_upload_us;
    *bytes = c->plan_bytes_up;
    *mode = c->plan_mode;
    return COLLM_OK;
}

int collm_debug_last_call(const collm_ctx *c, int32_t *grad_slices, int32_t *mixed_passes, int32_t *pass_slices)
{
    if (!c || !grad_slices || !mixed_passes || !pass_slices) return COLLM_E_NULL;
    *grad_slices = c->ran_grad_slices;
    *mixed_passes = c->ran_mixed;
    *pass_slices = c->ran_pass_slices;
    return COLLM_OK;
}

int collm_profile_enable(collm_ctx *c, int enable)
{
    if (!c) return COLLM_E_NULL;
    if (enable && !c->prof_ev_made) {
        for (int i = 0; i < kMaxProfile; ++i) {
            HIP_TRY(hipEventCreate(&c->prof_ev[i][0]));
            HIP_TRY(hipEventCreate(&c->prof_ev[i][1]));
        }
        c->prof_ev_made = true;
    }
    c->profile = enable != 0;
    c->n_prof = 0;
    return COLLM_OK;
}

int collm_profile_read(collm_ctx *c, const char **names, float *ms, int cap)
{
    if (!c || !names || !ms) return COLLM_E_NULL;
    const int n = std::min(c->n_prof, cap);
    for (int i = 0; i < n; ++i) {
        names[i] = c->prof_name[i];
        ms[i] = 0.f;
        if (c->prof_launches[i] == 0) continue;
        HIP_TRY(hipEventSynchronize(c->prof_ev[i][1]));
        HIP_TRY(hipEventElapsedTime(&ms[i], c->prof_ev[i][0], c->prof_ev[i][1]));
    }
    return n;
}

static int fwd_impl(collm_ctx *c, const collm_shape *s, const collm_siblings *sib, const void *x, const void *W,
                    const void *const *A, const void *const *B, const int32_t *rank1,
                    const int32_t *seg_start, const int32_t *seg_adapter,
                    const uint8_t *seg_is_train, void *y, float *h_save, void *stream)
{
    // with siblings, `rank` is the sum over the siblings and rank1 the adapter's own
    const int P = sib ? sib->n_siblings : 1;
    int rc = sib ? prepare_siblings(c, s, sib, rank1) : COLLM_OK;
    if (rc != COLLM_OK) return rc;
    const int32_t *rank = P > 1 ? c->sum_rank.data() : rank1;
    const bool swiglu = sib && sib->activation == COLLM_ACT_SWIGLU;
    rc = check_common(c, s, x, W, A, B, rank, seg_start, seg_adapter, seg_is_train);
    if (rc != COLLM_OK) return rc;
    if (s->n_tokens > 0 && !y) return COLLM_E_NULL;
    if (!aligned16(y) || !aligned16(h_save)) return COLLM_E_ALIGN;
    if (s->n_tokens == 0) return COLLM_OK;
    hipStream_t st = (hipStream_t)stream;
    HIP_TRY(hipSetDevice(c->device));
    c->n_prof = 0;
    c->ran_grad_slices = c->ran_mixed = c->ran_pass_slices = 0;
    const PatchGuard guard{c};
    const bool decode = decode_sized(c, s, rank, seg_start, seg_adapter, seg_is_train, P, swiglu);
    {
        Prof prof(c, st, "plan_copy");
        rc = prepare_plan(c, s, A, B, rank, seg_start, seg_adapter, seg_is_train, nullptr, nullptr, true, st, true, A, false,
                          P > 1 ? rank1 : nullptr, P, swiglu, decode);
    }
    if (rc != COLLM_OK) return rc;
    const PlanLayout &L = c->L;
    const bool f32 = s->dtype == COLLM_F32;
    if (decode) return run_decode(c, s, x, W, B, y, st);

    // shrink: h = x A_a (fp32), kept as s*h in the element type for the GEMM's extra K-steps
    // COLLM_LAYOUT_OUT_IN: every table is the transpose, so each pass takes the kernel variant its
    // counterpart in the other direction uses
    const bool tr = s->layout == COLLM_LAYOUT_OUT_IN;
    rc = run_skinny(c, s, L.all, x, s->d_in, L.off_A_ptr, tr, h_save, c->max_rank, c->max_rank, 1, 1.0f,
                    c->d_hs, s->scale, "shrink", st, nullptr, !f32 && (swiglu || warm_pays(c, L.all, s->n_tokens, s->d_out, s->d_in, tr, P <= 1, P > 1)) ? W : nullptr,
                    (uint64_t)s->d_in * s->d_out * 2, nullptr, swiglu ? L.rpad / 2 : 0);
    if (rc != COLLM_OK) return rc;

    GemmArgs g{};
    g.a = x;
    g.lda = s->d_in;
    g.b = W;
    g.ldb = tr ? s->d_in : s->d_out;
    g.out = y;
    g.ldo = s->d_out;
    g.N = s->d_out;
    g.K = s->d_in;
    g.a_bytes = (uint32_t)((int64_t)s->n_tokens * s->d_in * 2);
    g.b_bytes = (uint32_t)((int64_t)s->d_in * s->d_out * 2);
    g.tiles_m = L.all.n_tiles_m;
    g.row_tok = c->d_plan + L.all.off_row_tok;
    g.ext_off = c->d_plan + L.all.off_ext_off;
    g.ext = reinterpret_cast<const ExtStep *>(c->d_plan + L.all.off_ext);
    g.hs = c->d_hs;
    g.hs_ld = L.rpad;
    g.hs_bytes = (uint32_t)((size_t)c->rows_cap * c->rpad_cap * 4);
    g.ext_ld = tr ? 0 : s->d_out;
    g.zeros = c->d_zeros;
    g.n_sib = swiglu ? 0 : P;
    for (int j = 0, col = 0; j + 1 < P; ++j) g.sib_col[j] = (col += sib->d_out[j]);
    if (swiglu) {
        // y is [T, d_ff]; W and the expand tables keep their 2 d_ff columns
        g.N = g.ldo = g.act_col = sib->d_out[0];
        g.pre_act = sib->pre_act;
        g.pre_ld = s->d_out;
        g.tok_train = c->d_plan + L.off_tok_train;
    }
    {
        Prof prof(c, st, "gemm_fwd");
        if (f32) {
            g.n_rows = s->n_tokens;
            g.tile_steps = L.all.n_ext / ((L.all.n_rows + 63) / 64);
            HIP_TRY(launch_gemm_f32(g, tr, st));
        } else {
            HIP_TRY(run_gemm(c, g, L.all, s->n_tokens, s->d_out, c->tile_fwd, tr, P <= 1, st, swiglu));
        }
    }
    return COLLM_OK;
}

int collm_lora_linear_fwd(collm_ctx *c, const collm_shape *s, const void *x, const void *W,
                          const void *const *A, const void *const *B, const int32_t *rank,
                          const int32_t *seg_start, const int32_t *seg_adapter,
                          const uint8_t *seg_is_train, void *y, float *h_save, void *stream)
{
    return fwd_impl(c, s, nullptr, x, W, A, B, rank, seg_start, seg_adapter, seg_is_train, y, h_save, stream);
}

int collm_lora_linear_fwd_noalloc(int device, const collm_shape *s, const void *x, const void *W,
                                  const void *const *A, const void *const *B, const int32_t *rank,
                                  const int32_t *seg_start, const int32_t *seg_adapter,
                                  const uint8_t *seg_is_train, void *y, float *h_save, void *stream)
{
    if (!s) return COLLM_E_NULL;
    if (s->n_tokens > kScratchMaxTokens || s->n_segments > kScratchMaxSegments || s->n_adapters > kScratchMaxAdapters ||
        s->d_in > kScratchMaxD || s->d_out > kScratchMaxD) {
        char buf[200];
        std::snprintf(buf, sizeof buf,
                      "collm_lora_linear_fwd_noalloc serves at most %d tokens, %d segments, %d adapters of rank <= %d and "
                      "d_in, d_out <= %d (static workspace of %zu MiB)",
                      kScratchMaxTokens, kScratchMaxSegments, kScratchMaxAdapters, kScratchMaxRank, kScratchMaxD,
                      kScratchBytes >> 20);
        g_last_error = buf;
        return COLLM_E_SHAPE;
    }
    collm_ctx *c = nullptr;
    int rc = scratch_context(device, (hipStream_t)stream, &c);
    if (rc != COLLM_OK) return rc;
    rc = fwd_impl(c, s, nullptr, x, W, A, B, rank, seg_start, seg_adapter, seg_is_train, y, h_save, stream);
    if (rc == COLLM_E_RANK)
        g_last_error = "collm_lora_linear_fwd_noalloc: a rank is outside 1..64 (the static workspace's limit)";
    return rc;
}

int collm_lora_siblings_fwd(collm_ctx *c, const collm_shape *s, const collm_siblings *sib, const void *x,
                            const void *W, const void *const *A, const void *const *B, const int32_t *rank,
                            const int32_t *seg_start, const int32_t *seg_adapter, const uint8_t *seg_is_train,
                            void *y, float *h_save, void *stream)
{
    if (!sib) return COLLM_E_NULL;
    return fwd_impl(c, s, sib, x, W, A, B, rank, seg_start, seg_adapter, seg_is_train, y, h_save, stream);
}

static int bwd_impl(collm_ctx *c, const collm_shape *s, const collm_siblings *sib, const void *x, const void *W,
                    const void *const *A, const void *const *B, const int32_t *rank1,
                    const int32_t *seg_start, const int32_t *seg_adapter,
                    const uint8_t *seg_is_train, const void *dy, const float *h_save, void *dx,
                    float *const *dA, float *const *dB, int accumulate, void *stream)
{
    const int P = sib ? sib->n_siblings : 1;
    int rc = sib ? prepare_siblings(c, s, sib, rank1) : COLLM_OK;
    if (rc != COLLM_OK) return rc;
    const int32_t *rank = P > 1 ? c->sum_rank.data() : rank1;
    rc = check_common(c, s, x, W, A, B, rank, seg_start, seg_adapter, seg_is_train);
    if (rc != COLLM_OK) return rc;
    if ((dA == nullptr) != (dB == nullptr)) return COLLM_E_NULL;
    int n_train = 0, n_trained = 0;  // (trained adapters are counted up to kGradOuts + 1)
    int32_t trained[kGradOuts];
    for (int k = 0; k < s->n_segments; ++k) {
        if (!seg_is_train[k] || seg_start[k + 1] == seg_start[k]) continue;
        n_train += seg_start[k + 1] - seg_start[k];
        const int a = seg_adapter[k];
        if (n_trained <= kGradOuts && std::find(trained, trained + n_trained, a) == trained + n_trained) {
            if (n_trained < kGradOuts) trained[n_trained] = a;
            ++n_trained;
        }
        if (dA) {
            if (!dA[a] || !dB[a]) return COLLM_E_ADAPTER;
            if (!aligned16(dA[a]) || !aligned16(dB[a])) return COLLM_E_ALIGN;
        }
    }
    if (n_train > 0 && !dy) return COLLM_E_NULL;
    if (!aligned16(dy) || !aligned16(dx) || !aligned16(h_save)) return COLLM_E_ALIGN;
    if (n_train == 0) return COLLM_OK;
    hipStream_t st = (hipStream_t)stream;
    HIP_TRY(hipSetDevice(c->device));
    c->n_prof = 0;
    c->ran_grad_slices = c->ran_mixed = c->ran_pass_slices = 0;
    // Few gradient buffers travel as arguments of the gradient kernels, which then need nothing that an upload of this call puts into
    // the plan (the pass over dy that gives dh and dB at once, for narrow ranks, looks them up there): new adapter tables
    // ride on the rank-wide pass that the call begins with, beside dB on the second stream.  Four 4096 -> 4096 projections, 2048 tokens, 1792 of
    // them training, forward and backward: 634 us with the backward calls' upload in front, 610 without.
    const bool may_dual = P == 1 && s->layout == COLLM_LAYOUT_IN_OUT && c->dual_pass != 0 && (c->dual_pass == 1 || (int64_t)n_train * s->d_out * 2 >= kDualMinBytes);
    const bool out_args = dA && s->dtype == COLLM_BF16 && n_trained <= kGradOuts && !may_dual;
    const PatchGuard guard{c};
    {
        Prof prof(c, st, "plan_copy");
        rc = prepare_plan(c, s, A, B, rank, seg_start, seg_adapter, seg_is_train, dA, dB, true, st, false, dA && !out_args ? nullptr : (!h_save && dA ? A : B), out_args,
                          P > 1 ? rank1 : nullptr, P);
    }
    if (rc != COLLM_OK) return rc;
    // siblings: widest single rank, padded, for the passes that take one sibling at a time
    int rpad1 = c->L.rpad;
    if (P > 1) {
        int r1 = 1;
        for (int a = 0; a < s->n_adapters; ++a) r1 = std::max(r1, rank1[a]);
        rpad1 = round_up(r1, kKStep);
    }
    const PlanLayout &L = c->L;
    const bool f32 = s->dtype == COLLM_F32;
    const bool tr = s->layout == COLLM_LAYOUT_OUT_IN;

    // h of the training rows, if the forward call did not keep it
    if (!h_save && dA) {
        rc = run_skinny(c, s, L.train, x, s->d_in, L.off_A_ptr, tr, c->d_h32, L.rpad, L.rpad, 0, 1.0f,
                        c->d_hs, s->scale, "shrink_recompute", st);
        if (rc != COLLM_OK) return rc;
    }
    // The adapter gradients depend on little (dB_a: h and dy; dA_a: dh and x) and are bound by memory
    // latency, as is dh: they run on a second stream beside dh and the dX GEMM, which joins the
    // caller's stream again before the call returns.  (Serial when kernels are being timed.)
    // Small batches stay on the caller's stream (see grads_alone).
    const bool alone = c->grad_streams >= 0 ? c->grad_streams == 0 : grads_alone(n_train, s->d_in, s->d_out, f32, L.rpad);
    // Or in the dX GEMM's launch, where that leaves places free (grads_in_gemm).  Not where a buffer that the launch writes lies in one that another part
    // of it reads: a dx in the place of what the gradients read, a dA in that of h, which are behind them otherwise.
    const int64_t T = s->n_tokens, esz = f32 ? 4 : 2;
    bool own = dA && dx && apart(dx, T * s->d_in * esz, x, T * s->d_in * esz);
    const bool dx_behind_dA = own;  // (fp32)
    own = own && apart(dx, T * s->d_in * esz, dy, T * s->d_out * esz) && apart(dx, T * s->d_in * esz, h_save, h_save ? T * c->max_rank * 4 : 0);
    for (int k = 0; own && h_save && k < s->n_segments; ++k)
        if (seg_is_train[k] && seg_start[k + 1] > seg_start[k])
            own = apart(dA[seg_adapter[k]], (int64_t)s->d_in * rank[seg_adapter[k]] * 4, h_save, T * c->max_rank * 4);
    const bool may_fuse = own && !c->profile && !f32 && P == 1 && !may_dual && L.n_grad > 0;
    GradsBeside beside{};
    beside.slices = may_fuse ? grads_in_gemm(c, n_train, s->d_in, s->d_out, !tr, L.rpad, alone) : 0;
    const bool fused = beside.slices > 0;
    const bool overlap = dA && !alone && !fused && !c->profile;
    const bool one_round = dx_one_round(c, n_train, s->d_in, s->d_out, f32, L.rpad);
    // fp32 on one stream: dB beside dh, dA beside dX
    const bool pair = f32 && dA && alone && !c->profile && pair_f32(L.rpad, s->d_in, s->d_out);
    hipStream_t gs = overlap ? c->side : st;
    GradArgs ga{};
    ga.row_tok = c->d_plan + L.train.off_row_tok;
    ga.items = reinterpret_cast<const GradItem *>(c->d_plan + L.off_grad);
    ga.n_items = L.n_grad;
    ga.accumulate = accumulate ? 1 : 0;
    auto set_outs = [&](float *const *g) {
        if (!out_args || L.n_grad > kGradOuts) return;
        ga.n_out = L.n_grad;
        const GradItem *items = reinterpret_cast<const GradItem *>(c->plan.data() + L.off_grad);
        for (int k = 0; k < L.n_grad; ++k) ga.out[k] = (uint64_t)(uintptr_t)g[items[k].adapter];
    };
    bool dx_even = false;  // the dX GEMM leaves no CU free
    if (overlap && dx && !f32) {
        const Tiling t = c->tile_bwd >= 0 ? Tiling{c->tile_bwd, 0, 0}
                                          : choose_tiling(c, n_train, s->d_in, s->d_out, !tr, true, c->gemm_split != 1, one_round, c->tile_steps_train);
        ga.beside_gemm = t.tile == kTile128x128 ? 1 : 0;
        dx_even = t.tile == kTile256x256 && whole_rounds(n_train, s->d_in, t.slices);
    }

    // Narrow ranks (all at most 16), tables as [rank][d_out]: dh and dB_a both come from ONE pass over the training
    // rows of dy (kernels.h, DualArgs), which is the largest operand of the backward pass beside W.  The rows of
    // every trained adapter are cut into pieces so that two blocks per CU exist (pieces of 512 rows down to 64), as
    // long as the per-group slices of dh and the per-piece sums of dB fit the workspace of partial sums.  It pays where
    // the training rows of dy do not fit the last-level cache (256 MB): 8192 rows of 28672 columns (470 MB) take 153 us
    // against 94 + 122 for the two passes and the step is 1 % shorter; 8192 x 8192 (134 MB) 65 against 31 + 43 with
    // no gain for the step (the two passes run side by side on two streams and the second reader finds dy in the
    // cache); on 8192 x 1024 (34 against 10 + 15) and 1792 x 4096 (28 against 14 + 10) the partial sums and the two
    // kernels that add them cost more than the second read.
    DualArgs du{};
    bool dual = false;
    if (!f32 && !tr && P == 1 && dA && c->dual_pass != 0 && L.rpad == kKStep && L.train.n_wide == 0 && L.n_grad > 0 &&
        (c->dual_pass == 1 || (int64_t)L.train.n_rows * s->d_out * 2 >= kDualMinBytes)) {
        const int groups = (s->d_out + kDualCols - 1) / kDualCols;
        auto pieces_of = [&](int rows) { return (L.max_grad_rows + rows - 1) / rows; };
        auto fits = [&](int rows) {
            const size_t dh_floats = (size_t)round_up(groups * L.train.n_rows_pad * kKStep, 64);
            // (pieces are the grid's second dimension, with the rows of blocks that fetch the weight behind them)
            return (long)L.n_grad * pieces_of(rows) + c->n_cus < 65536 &&
                   (dh_floats + (size_t)L.n_grad * pieces_of(rows) * kKStep * s->d_out) * 4 <= c->part_bytes;
        };
        int rows = kDualMaxPieceRows;
        while (rows > 64 && (long)groups * L.n_grad * pieces_of(rows) < 2L * std::max(c->n_cus, 1)) rows >>= 1;
        while (rows < kDualMaxPieceRows && !fits(rows)) rows <<= 1;
        if (fits(rows)) {
            dual = true;
            du.dy = dy;
            du.ld_dy = s->d_out;
            du.dy_bytes = (uint32_t)((int64_t)s->n_tokens * s->d_out * 2);
            du.N = s->d_out;
            du.hs = c->d_hs;
            du.ld_hs = L.rpad;
            du.hs_bytes = (uint32_t)((size_t)L.train.n_rows_pad * L.rpad * 2);
            du.row_tok = ga.row_tok;
            du.items = ga.items;
            du.n_grad = L.n_grad;
            du.tab_b = reinterpret_cast<const uint64_t *>(c->d_plan + L.off_B_ptr);
            du.out_tab = reinterpret_cast<const uint64_t *>(c->d_plan + L.off_dB_ptr);
            du.accumulate = ga.accumulate;
            du.piece_rows = rows;
            du.max_pieces = pieces_of(rows);
            du.part_dh = c->d_part;
            du.part_rows = L.train.n_rows_pad;
            du.part_ld = kKStep;
            du.part_dB = c->d_part + round_up(groups * L.train.n_rows_pad * kKStep, 64);
            // (the weight of the dX GEMM, as the dh pass would fetch it: see run_skinny)
            const uint64_t w_bytes = (uint64_t)s->d_in * s->d_out * 2;
            if (dx && w_bytes <= kWarmMaxBytes && (uint64_t)L.train.n_rows * s->d_out * 2 <= w_bytes && c->n_cus > 0) {
                du.warm_base = W;
                du.warm_bytes = w_bytes;
                du.warm_rows = (c->n_cus + groups - 1) / groups;
            }
        }
    }
    if (dual) {
        Prof prof(c, st, "dh_dB");
        // s h as bf16 in training row order: left by the recomputing pass, or packed from h_save here
        if (h_save)
            HIP_TRY(launch_pack_rows(h_save, c->max_rank, c->max_rank, c->d_plan + L.train.off_row_tok, L.train.n_rows,
                                     s->scale, c->d_hs, L.rpad, st));
        HIP_TRY(launch_dual(du, st));
        const SliceSums sums{du.part_dh, du.part_rows, du.part_ld, (s->d_out + kDualCols - 1) / kDualCols};
        rc = run_skinny(c, s, L.train, dy, s->d_out, L.off_B_ptr, true, c->d_dh32, L.rpad, L.rpad, 0, s->scale, c->d_dhs,
                        s->scale, nullptr, st, nullptr, nullptr, 0, &sums);
        if (rc != COLLM_OK) return rc;
        HIP_TRY(launch_dual_sum(du, st));
    }
    // dB_a = s h^T dy
    const bool late = overlap && !dual && dx && P == 1 && !dx_even && fork_behind_dh(L.rpad, s->d_in, s->d_out);
    auto launch_dB = [&]() -> int {
        if (overlap && !late) {
            HIP_TRY(hipEventRecord(c->ev_fork, st));
            HIP_TRY(hipStreamWaitEvent(c->side, c->ev_fork, 0));
        }
        ga.big = dy;
        ga.ld_big = s->d_out;
        ga.big_bytes = (uint32_t)((int64_t)s->n_tokens * s->d_out * esz);
        ga.N = s->d_out;
        if (h_save) {
            ga.small_ = h_save;
            ga.ld_small = c->max_rank;
            ga.small_by_token = 1;
        } else {
            ga.small_ = c->d_h32;
            ga.ld_small = L.rpad;
            ga.small_by_token = 0;
        }
        ga.small_mult = s->scale;
        if (!f32) {
            // the small operand as a scaled bf16 copy in training row order (half the bytes of the fp32 one, no
            // conversion in the kernel): left by the recomputing pass, or packed from h_save here.  The forward
            // call's copy of s h (all rows) in the same buffer is dead once that call's GEMM has run.
            // (small batches skip the packing kernel: their gradient kernel converts as it reads)
            const bool pack = h_save && !((alone || fused) && P == 1);
            if (pack)
                HIP_TRY(launch_pack_rows(h_save, c->max_rank, c->max_rank, c->d_plan + L.train.off_row_tok,
                                         L.train.n_rows, s->scale, c->d_hs, L.rpad, gs));
            if (pack || !h_save) {
                ga.small_bf = c->d_hs;
                ga.ld_small_bf = L.rpad;
            }
        }
        ga.out_tab = reinterpret_cast<const uint64_t *>(c->d_plan + L.off_dB_ptr);
        set_outs(dB);
        ga.out_transposed = tr ? 1 : 0;
        if (fused) {
            beside.dB = ga;
            ga.small_bf = nullptr;
        } else if (!pair) {
            Prof prof(c, gs, "grad_dB");
            if (f32) {
                HIP_TRY(launch_grad_f32(ga, L.n_grad, L.rpad, gs));
            } else if (P == 1) {
                HIP_TRY(launch_grad(ga, L.n_grad, L.rpad, gs));
            } else {
                // one launch per sibling: its columns of dy against its columns of s h
                for (int j = 0, col = 0; j < P; col += sib->d_out[j], ++j) {
                    GradArgs gj = ga;
                    gj.big = reinterpret_cast<const uint8_t *>(dy) + (int64_t)col * 2;
                    gj.big_bytes = ga.big_bytes - (uint32_t)col * 2u;
                    gj.N = sib->d_out[j];
                    gj.n_sib = P;
                    gj.sib = j;
                    gj.ld_out = s->d_out;
                    gj.out_off = col;
                    HIP_TRY(launch_grad(gj, L.n_grad, rpad1, gs));
                }
            }
        }
        return COLLM_OK;
    };
    if (dA && !dual && !late) {
        rc = launch_dB();
        if (rc != COLLM_OK) return rc;
    }

    // dh = s dy B_a^T: fp32 for dA, element type for the dX GEMM's extra K-steps
    if (dual) {
        // dh came out of the pass over dy above, together with dB
    } else if (P == 1) {
        rc = run_skinny(c, s, L.train, dy, s->d_out, L.off_B_ptr, !tr, c->d_dh32, L.rpad, L.rpad, 0, s->scale,
                        c->d_dhs, s->scale, "dh", st, nullptr, !f32 && dx && warm_pays(c, L.train, n_train, s->d_in, s->d_out, !tr, one_round, false, beside.slices) ? W : nullptr,
                        (uint64_t)s->d_in * s->d_out * 2, nullptr, 0, pair ? &ga : nullptr);
        if (rc != COLLM_OK) return rc;
    } else {
        // one pass per sibling over its columns of dy and of the tables, each writing its columns of dh
        for (int j = 0, col = 0; j < P; col += sib->d_out[j], ++j) {
            SiblingPass sp;
            sp.n_sib = P;
            sp.sib = j;
            sp.ld = s->d_out;
            sp.col0 = col;
            sp.rpad = rpad1;
            rc = run_skinny(c, s, L.train, dy, sib->d_out[j], L.off_B_ptr, true, c->d_dh32, L.rpad, L.rpad, 0,
                            s->scale, c->d_dhs, s->scale, "dh", st, &sp);
            if (rc != COLLM_OK) return rc;
        }
    }

    if (dA) {
        if (overlap) {
            HIP_TRY(hipEventRecord(c->ev_dh, st));
            HIP_TRY(hipStreamWaitEvent(c->side, c->ev_dh, 0));
        }
        if (late) {
            rc = launch_dB();
            if (rc != COLLM_OK) return rc;
        }
        // dA_a = x^T dh
        ga.big = x;
        ga.ld_big = s->d_in;
        ga.big_bytes = (uint32_t)((int64_t)s->n_tokens * s->d_in * esz);
        ga.N = s->d_in;
        ga.small_ = c->d_dh32;
        ga.ld_small = L.rpad;
        ga.small_by_token = 0;
        ga.small_mult = 1.0f;
        if (!f32) {
            ga.small_bf = c->d_dhs;  // dh in the element type, as the dh pass left it for the dX GEMM
            ga.ld_small_bf = L.rpad;
        }
        ga.out_tab = reinterpret_cast<const uint64_t *>(c->d_plan + L.off_dA_ptr);
        set_outs(dA);
        ga.out_transposed = tr ? 0 : 1;
        if (fused) {
            beside.dA = ga;
            beside.n_grad = L.n_grad;
            beside.rpad = L.rpad;
        } else if (!pair) {
            Prof prof(c, gs, "grad_dA");
            if (f32) HIP_TRY(launch_grad_f32(ga, L.n_grad, L.rpad, gs));
            else HIP_TRY(launch_grad(ga, L.n_grad, L.rpad, gs));
        }
        if (overlap) HIP_TRY(hipEventRecord(c->ev_join, c->side));
    }

    if (dx) {
        GemmArgs g{};
        g.a = dy;
        g.lda = s->d_out;
        g.b = W;
        g.ldb = tr ? s->d_in : s->d_out;
        g.out = dx;
        g.ldo = s->d_in;
        g.N = s->d_in;
        g.K = s->d_out;
        g.a_bytes = (uint32_t)((int64_t)s->n_tokens * s->d_out * 2);
        g.b_bytes = (uint32_t)((int64_t)s->d_in * s->d_out * 2);
        g.tiles_m = L.train.n_tiles_m;
        g.row_tok = c->d_plan + L.train.off_row_tok;
        g.ext_off = c->d_plan + L.train.off_ext_off;
        g.ext = reinterpret_cast<const ExtStep *>(c->d_plan + L.train.off_ext);
        g.hs = c->d_dhs;
        g.hs_ld = L.rpad;
        g.hs_bytes = (uint32_t)((size_t)c->rows_cap * c->rpad_cap * 4);
        g.ext_ld = tr ? s->d_in : 0;
        g.zeros = c->d_zeros;
        Prof prof(c, st, "gemm_dx");
        if (f32) {
            g.n_rows = n_train;
            g.tile_steps = L.train.n_ext / ((L.train.n_rows + 63) / 64);
            // (a caller's dx in the place of its x, or part of it: dA reads x first)
            if (pair && dx_behind_dA && gemm_f32_with_dA(g, !tr)) {
                HIP_TRY(launch_dx_dA_f32(g, ga, L.rpad, !tr, st));
            } else {
                if (pair) HIP_TRY(launch_grad_f32(ga, L.n_grad, L.rpad, st));
                HIP_TRY(launch_gemm_f32(g, !tr, st));
            }
        } else {
            HIP_TRY(run_gemm(c, g, L.train, n_train, s->d_in, c->tile_bwd, !tr, one_round && !fused, st, false, fused ? &beside : nullptr));
            if (fused && beside.done) c->ran_grad_slices = beside.slices;
            if (fused && !beside.done) {
                HIP_TRY(launch_grad(beside.dB, L.n_grad, L.rpad, st));
                HIP_TRY(launch_grad(beside.dA, L.n_grad, L.rpad, st));
            }
        }
    }
    if (pair && !dx) HIP_TRY(launch_grad_f32(ga, L.n_grad, L.rpad, st));
    if (overlap) HIP_TRY(hipStreamWaitEvent(st, c->ev_join, 0));
    return COLLM_OK;
}

int collm_lora_linear_bwd(collm_ctx *c, const collm_shape *s, const void *x, const void *W,
                          const void *const *A, const void *const *B, const int32_t *rank,
                          const int32_t *seg_start, const int32_t *seg_adapter,
                          const uint8_t *seg_is_train, const void *dy, const float *h_save, void *dx,
                          float *const *dA, float *const *dB, int accumulate, void *stream)
{
    return bwd_impl(c, s, nullptr, x, W, A, B, rank, seg_start, seg_adapter, seg_is_train, dy, h_save, dx, dA, dB,
                    accumulate, stream);
}

int collm_lora_siblings_bwd(collm_ctx *c, const collm_shape *s, const collm_siblings *sib, const void *x,
                            const void *W, const void *const *A, const void *const *B, const int32_t *rank,
                            const int32_t *seg_start, const int32_t *seg_adapter, const uint8_t *seg_is_train,
                            const void *dy, const float *h_save, void *dx, float *const *dA, float *const *dB,
                            int accumulate, void *stream)
{
    if (!sib) return COLLM_E_NULL;
    return bwd_impl(c, s, sib, x, W, A, B, rank, seg_start, seg_adapter, seg_is_train, dy, h_save, dx, dA, dB,
                    accumulate, stream);
}

int collm_swiglu_bwd(int device, int32_t n_tokens, int32_t d_ff, int32_t n_segments, const int32_t *seg_start,
                     const uint8_t *seg_is_train, const void *pre_act, const void *dout, void *dy, void *stream)
{
    if (n_tokens < 0 || n_segments < 0 || d_ff <= 0 || d_ff % 8) return COLLM_E_SHAPE;
    if (n_segments > 0 && (!seg_start || !seg_is_train)) return COLLM_E_NULL;
    if (n_segments > 0 && seg_start[0] != 0) return COLLM_E_SEGMENTS;
    bool any = false;
    for (int k = 0; k < n_segments; ++k) {
        if (seg_start[k + 1] < seg_start[k]) return COLLM_E_SEGMENTS;
        any = any || (seg_is_train[k] && seg_start[k + 1] > seg_start[k]);
    }
    if (n_segments > 0 && seg_start[n_segments] != n_tokens) return COLLM_E_SEGMENTS;
    if (!any) return COLLM_OK;
    if (!pre_act || !dout || !dy) return COLLM_E_NULL;
    if (!aligned16(pre_act) || !aligned16(dout) || !aligned16(dy)) return COLLM_E_ALIGN;
    HIP_TRY(hipSetDevice(device));
    SwigluBwdArgs a{};
    a.pre = pre_act;
    a.dout = dout;
    a.dy = dy;
    a.d_ff = d_ff;
    a.ld_pre = a.ld_dy = 2 * (int64_t)d_ff;
    a.ld_dout = d_ff;
    for (int k = 0; k < n_segments; ++k) {
        const int n = seg_start[k + 1] - seg_start[k];
        if (seg_is_train[k] && n > 0) {
            a.tok0[a.n_seg] = seg_start[k];
            a.row0[a.n_seg + 1] = a.row0[a.n_seg] + n;
            ++a.n_seg;
        }
        if (a.n_seg == kSwigluSegs || (k + 1 == n_segments && a.n_seg > 0)) {
            HIP_TRY(launch_swiglu_bwd(a, (hipStream_t)stream));
            a.n_seg = 0;
        }
    }
    return COLLM_OK;
}

int collm_adapter_fedavg(int device, collm_dtype dtype, int32_t n_copies, const void *const *src, void *dst,
                         int64_t n_elems, void *stream)
{
    if (dtype != COLLM_F32 && dtype != COLLM_BF16) return COLLM_E_DTYPE;
    if (n_copies < 1 || n_copies > kMaxFedAvgCopies || n_elems < 0) return COLLM_E_SHAPE;
    if (!src || (n_elems > 0 && !dst)) return COLLM_E_NULL;
    if (!aligned16(dst)) return COLLM_E_ALIGN;
    FedAvgArgs a{};
    for (int k = 0; k < n_copies; ++k) {
        if (n_elems > 0 && !src[k]) return COLLM_E_NULL;
        if (!aligned16(src[k])) return COLLM_E_ALIGN;
        a.src[k] = src[k];
    }
    if (n_elems == 0) return COLLM_OK;
    a.dst = dst;
    a.n = n_elems;
    a.n_copies = n_copies;
    HIP_TRY(hipSetDevice(device));
    HIP_TRY(launch_fedavg(a, dtype == COLLM_BF16, (hipStream_t)stream));
    return COLLM_OK;
}

int collm_adapter_adamw(int device, collm_dtype dtype, void *param, float *master, const float *grad,
                        float *m, float *v, int64_t n_elems, const collm_adamw *hp, void *stream)
{
    if (dtype != COLLM_F32 && dtype != COLLM_BF16) return COLLM_E_DTYPE;
    if (!hp) return COLLM_E_NULL;
    if (n_elems < 0 || hp->step < 1) return COLLM_E_SHAPE;
    if (n_elems == 0) return COLLM_OK;
    if (!param || !grad || !m || !v) return COLLM_E_NULL;
    if (!aligned16(param) || !aligned16(master) || !aligned16(grad) || !aligned16(m) || !aligned16(v)) return COLLM_E_ALIGN;
    AdamWArgs a{};
    a.param = param;
    a.master = master;
    a.grad = grad;
    a.m = m;
    a.v = v;
    a.n = n_elems;
    a.lr = hp->lr;
    a.beta1 = hp->beta1;
    a.beta2 = hp->beta2;
    a.eps = hp->eps;
    a.weight_decay = hp->weight_decay;
    a.bias1 = (float)(1.0 - std::pow((double)hp->beta1, (double)hp->step));
    a.rsqrt_bias2 = (float)(1.0 / std::sqrt(1.0 - std::pow((double)hp->beta2, (double)hp->step)));
    HIP_TRY(hipSetDevice(device));
    HIP_TRY(launch_adamw(a, dtype == COLLM_BF16, (hipStream_t)stream));
    return COLLM_OK;
}

int collm_debug_device_token_map(collm_ctx *c, int32_t *tok_segment, int32_t *tok_adapter,
                                 uint8_t *tok_is_train)
{
    if (!c) return COLLM_E_NULL;
    if (!c->plan_valid) return COLLM_E_SHAPE;
    const PlanLayout &L = c->L;
    if (L.n_tokens > 0 && (!tok_segment || !tok_adapter || !tok_is_train)) return COLLM_E_NULL;
    HIP_TRY(hipSetDevice(c->device));
    HIP_TRY(hipStreamSynchronize(c->last_stream));
    std::vector<int32_t> dev((size_t)L.total_ints);
    HIP_TRY(hipMemcpy(dev.data(), c->d_plan, dev.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
    // Undo the adapter grouping: row r of the forward row order is token row_tok[r] and was
    // given adapter row_adapter[r]; segment and training flag come from the per-token arrays
    // the kernels read.
    for (int t = 0; t < L.n_tokens; ++t) tok_adapter[t] = -2;
    for (int r = 0; r < L.all.n_rows_pad; ++r) {
        const int tok = dev[L.all.off_row_tok + r];
        if (tok < 0) continue;
        if (tok >= L.n_tokens) return COLLM_E_SHAPE;
        tok_adapter[tok] = dev[L.all.off_row_adapter + r];
    }
    for (int t = 0; t < L.n_tokens; ++t) {
        tok_segment[t] = dev[L.off_tok_segment + t];
        tok_is_train[t] = (uint8_t)dev[L.off_tok_train + t];
        // the per-token adapter array must agree with the row order
        if (dev[L.off_tok_adapter + t] != tok_adapter[t]) tok_adapter[t] = -3;
    }
    // training rows must be exactly the training tokens
    std::vector<uint8_t> seen((size_t)std::max(L.n_tokens, 1), 0);
    for (int r = 0; r < L.train.n_rows_pad; ++r) {
        const int tok = dev[L.train.off_row_tok + r];
        if (tok >= 0 && tok < L.n_tokens) seen[tok] = 1;
    }
    for (int t = 0; t < L.n_tokens; ++t)
        if (seen[t] != tok_is_train[t]) tok_is_train[t] = 0xEE;
    return COLLM_OK;
}

}  // extern "C"
