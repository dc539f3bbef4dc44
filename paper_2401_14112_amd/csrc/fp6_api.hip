// C ABI of the library (see include/fp6.h): argument checks on the host, kernel
// selection, launches on the caller's stream.  No allocation, no synchronization.
#include "../../include/fp6.h"
#include "../../include/fp6_bench.h"

#include <atomic>
#include <cmath>
#include <initializer_list>

#include "fp6_device.hpp"
#include "linear_stream.hpp"
#include "linear_block.hpp"
#include "linear_tiled.hpp"
#include "pack_unpack.hpp"

namespace {

using namespace fp6;

constexpr int kLayoutVersion = 4;  // 4: 3-bit tiles of 512 columns (6-, 5-, 4-bit streams as in 3)
// Configurations of the streaming kernel: {token tiles per wave, row tiles per block, groups of k-tiles per block (one wave
// each), weight tiles in flight per wave, tokens of a token tile that are staged}.
struct StreamCfg {
    int nt, wm, wk, depth, xr;
};
// Packed weights.  First of each kind the one that the tuning hook for the split factor pins and that layers with more row
// blocks than CUs take.
constexpr StreamCfg kStreamCfg[] = {{1, 8, 1, 2, 2},  {1, 4, 2, 2, 2},  {1, 2, 4, 2, 2},  {1, 1, 8, 2, 2},
                                    {1, 8, 1, 2, 8},  {1, 4, 2, 2, 8},  {1, 2, 4, 2, 8},  {1, 1, 8, 2, 8},
                                    {1, 8, 1, 2, 16}, {1, 4, 2, 2, 16}, {1, 2, 4, 2, 16}, {1, 1, 8, 2, 16},
                                    {2, 8, 1, 2, 16}, {2, 6, 1, 2, 16}, {2, 4, 2, 2, 16}, {2, 2, 4, 2, 16},
                                    {3, 8, 1, 2, 16}, {3, 6, 1, 2, 16}, {3, 4, 2, 2, 16},
                                    {4, 8, 1, 2, 16}, {4, 6, 1, 2, 16}, {4, 4, 2, 2, 16}};
// fp16 weights (staged through LDS, 8 KB per tile in flight): blocks that fit the LDS of a CU beside the activation stages.
// Four tiles per wave instead of two in the block of four row tiles: 655 drawn calls that take it, weights from memory, median
// time 0.94 with two of that with four, lowest 0.80, largest 1.01 (the kernel's waits leave one request out at any depth).
constexpr StreamCfg kStreamCfgFp16[] = {{1, 8, 1, 2, 16}, {1, 4, 1, 2, 16}, {1, 4, 2, 2, 16}, {1, 1, 4, 2, 16},
                                        {2, 8, 1, 2, 16}, {2, 6, 1, 2, 16}, {2, 2, 2, 2, 16},
                                        {3, 4, 1, 2, 16}, {3, 6, 1, 2, 16},
                                        {4, 4, 1, 2, 16}, {4, 6, 1, 2, 16}};
constexpr int kStreamCfgs = sizeof(kStreamCfg) / sizeof(kStreamCfg[0]), kStreamCfgsFp16 = sizeof(kStreamCfgFp16) / sizeof(kStreamCfgFp16[0]);
template <bool PACKED, int C>
struct StreamShapeOf {
    static constexpr StreamCfg c = PACKED ? kStreamCfg[C] : kStreamCfgFp16[C];
    typedef StreamShape<c.nt, c.wm, c.wk, c.depth, c.xr> type;
};
constexpr int kMaxLds = 160 * 1024;
constexpr int stream_lds_bytes(const StreamCfg &c, int tile_cols, int lds_tile)
{
    return 2 * c.wk * c.nt * (tile_cols / 32) * c.xr / 16 * 1024 + c.wm * c.wk * c.depth * lds_tile;
}
constexpr int kStreamMaxN = 64;  // token counts up to this use the streaming kernel
constexpr int kCus = kXcds * kCusPerXcd;

std::atomic<int> g_forced_split{0};

// The kernels address the activations of up to 64 tokens, and the 16 rows of an fp16 weight tile, with 32-bit
// byte offsets: 64 * K * 2 must stay below 2^31.
constexpr int64_t kMaxK = 1ll << 24;
bool shape_ok(int64_t M, int64_t K) { return M > 0 && K > 0 && M % kTileRows == 0 && K % kTileK == 0 && M < (1ll << 31) && K < kMaxK; }
// Packed weights: tiles are stored k-tile major and a wave addresses the tiles of its row tile with 32-bit
// offsets that step by one k-tile's worth of all row tiles; the pipelines request up to 64 tiles past the end
// of a slice (out of range: they read as zeros), and those offsets must not wrap either.  Priced at the 6-bit
// tile size for every width.
bool packed_shape_ok(int64_t M, int64_t K)
{
    return shape_ok(M, K) && (K / kTileK + 64) * (M / kTileRows) <= ((1ll << 31) - 1) / kTileBytes;
}
bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Where a launch keeps its split-K state: arrival counters (zero before and after every launch) and the
// partial tiles.  Both kinds of buffer hold the counters in a region of fixed size at their start, whatever the
// plan, so that the partial tiles of one launch can never be read as counters by another: the launches of one call
// (a call cut into chunks plans each of them for itself) and calls of other shapes and weights that share a workspace.
// Every automatic plan with k slices has at most 128 blocks of at most eight waves, and one counter per wave or row
// tile: 4 KB hold them.  Only a forced split factor needs more.
constexpr size_t kCounterBytes = 4 * 1024;
constexpr size_t kStaticCounterBytes = 64 * 1024;  // the library's static buffer (fp6_linear_static)

struct SplitBuffers {
    int *counters;
    uint8_t *partials;
};

// Distance, in counters, of the arrival counters of a prompt-sized launch: as far apart as the region allows, up to 128
// bytes.  Arrivals at one cache line queue up: with 12 slices and 16 counters per line the queue costs 1.2 us
// (256 x 12544, N = 96, 6 bits 16.7 -> 15.2 us, 1232 x 7168, N = 80 14.5 -> 13.1; fp16, 816 x 5632, N = 418 31.1 -> 18.7);
// spread, no 64 bytes see more than 64 of them, where they could see 256.
int counter_step(size_t counters)
{
    int step = 1;
    while (step < 32 && counters * (size_t)step * 2 * sizeof(int) <= kCounterBytes)
        step *= 2;
    return step;
}

size_t counter_bytes_of(size_t counters, int step) { return (counters * (size_t)step * sizeof(int) + 255) / 256 * 256; }

struct WorkspaceRef {
    void *base;
    size_t bytes;
    size_t counter_region;  // its first bytes: kStaticCounterBytes or counter_region_bytes()
    bool own = false;       // the library's buffer
    // the buffers of a launch whose plan needs counter_bytes + partial_bytes; FP6_OK when they fit
    fp6_status view(size_t counter_bytes, size_t partial_bytes, SplitBuffers &out) const
    {
        out.counters = nullptr;
        out.partials = nullptr;
        if (partial_bytes == 0)
            return FP6_OK;  // no split-K: nothing is touched
        if (!base || counter_bytes > counter_region || bytes < counter_region || bytes - counter_region < partial_bytes)
            return FP6_ERR_WORKSPACE;
        if (!aligned16(base))
            return FP6_ERR_ALIGN;
        out.counters = static_cast<int *>(base);
        out.partials = static_cast<uint8_t *>(base) + counter_region;
        return FP6_OK;
    }
};

// The weights a launch reads, as the plan sees them.
struct StreamWeights {
    bool packed, grouped;
    int bits;       // per weight
    int tile_cols;  // columns of a weight tile in the streaming kernel
    int lds_tile;   // bytes of LDS that a tile in flight takes
};
// Configurations that exist for a format: those that fit the LDS.
constexpr bool stream_cfg_built(const StreamCfg &c, const StreamWeights &w)
{
    return stream_lds_bytes(c, w.tile_cols, w.lds_tile) <= kMaxLds;
}
template <class Src>  // the source of a format, as the entry points name it
constexpr StreamWeights stream_weights_of()
{
    typedef typename Src::StreamSource S;
    return {S::kPackedConfigs, std::is_same_v<S, PackedFp6GroupSource>, S::kBits, S::kTileCols, S::kLdsTileBytes};
}

struct StreamPlan {
    int cfg;         // index into kStreamCfg / kStreamCfgFp16
    int split;       // split-K factor
    int row_blocks;  // blocks along M
    size_t counter_bytes, partial_bytes;  // 0 without k slices
    // What the call asks its caller for.  A call is refused without the workspace that the size query names, and the query
    // does not depend on the block chosen: a shape whose blocks of eight row tiles would take k slices asks for those also
    // where its block needs none.
    size_t required_counters, required_partials;
};

// k slices and token tiles of the blocks of eight (four) row tiles for whose partial sums a caller's workspace is sized.
struct StreamSlices {
    int64_t split, nt;
};
StreamSlices stream_slices_of_shape(int64_t M, int64_t N, int64_t KT, bool packed)
{
    const int64_t row_tiles = M / kTileRows, max_split = KT >= 4 ? KT / 2 : 1;
    const bool four = !packed && N > 32;
    StreamSlices best{1, N <= 16 ? 1 : N <= 32 ? 2 : 4};
    int64_t best_blocks = -1;
    for (int waves = N <= 16 || four ? 4 : 8; waves <= (four ? 4 : 8); waves += 4) {
        const int64_t rb = (row_tiles + waves - 1) / waves;
        int64_t s = kCus / rb;
        s = s > max_split ? max_split : s;
        s = s > 64 ? 64 : s < 1 ? 1 : s;
        while (s > 1 && (uint64_t)s * (uint64_t)row_tiles * (uint64_t)best.nt * 1024u >= (1ull << 31))
            s /= 2;
        while (s > 1 && (uint64_t)(KT + 20 * s) * (uint64_t)row_tiles * kTileBytes >= (1ull << 31))
            s /= 2;
        const int64_t blocks = rb * s;
        const bool single = blocks <= kCus;
        if (best_blocks < 0
            || (single ? best_blocks > kCus || blocks > best_blocks || (blocks == best_blocks && s > best.split)
                       : best_blocks > kCus && blocks < best_blocks)) {
            best.split = s;
            best_blocks = blocks;
        }
    }
    return best;
}

// The launch's buffers in a caller's workspace, which is refused unless it holds what the call asks for; the library's own
// buffer has no such promise to keep.
fp6_status stream_buffers(const StreamPlan &p, const WorkspaceRef &workspace, SplitBuffers &buf)
{
    return workspace.own ? workspace.view(p.counter_bytes, p.partial_bytes, buf) : workspace.view(p.required_counters, p.required_partials, buf);
}

// Estimated time of a launch, us.  A stage (one k-tile per wave) of a block takes 0.38 us and 5 ns per KB of weights,
// 9.5 ns per KB of activations and from three token tiles on 80 ns for each, on a CU that does not wait for memory; the
// launch as a whole is no faster than 6.9 TB/s, and then half of the activation time still shows; a launch with k slices
// hands them over, one with groups of k-tiles adds them up in LDS.
// The chosen block against the best of all, each pinned in turn (9900 calls of 512 to 32768 rows and 1024 to 28672 columns, weights
// from memory): by format and token count 1.6 to 2.8 % slower on average, 4.9 % for 3 bits and 17 to 32 tokens.
double stream_cost(const StreamCfg &c, int64_t M, int64_t K, int64_t s, const StreamWeights &w)
{
    const int64_t KT = (K + w.tile_cols - 1) / w.tile_cols;
    const double blocks = (double)((M / kTileRows + c.wm - 1) / c.wm * s), rounds = blocks > kCus ? blocks / kCus : 1.0;
    const double stages = rounds * (double)(((KT + s - 1) / s + c.wk - 1) / c.wk);
    const double tile_kb = w.tile_cols / 512.0;  // of one bit per weight
    const double weight_kb = tile_kb * c.wm * c.wk * w.bits, x_kb = tile_kb * 16.0 * c.wk * c.nt * c.xr / 16.0;
    const double x_us = 0.0095 * x_kb + (c.nt > 2 ? 0.08 * c.nt * w.tile_cols / kTileK : 0.0);
    const double handover = s > 1 ? 0.5 + (double)s * (0.17 + 0.15 * c.nt) : 0.0;
    // (group scales at 9 to 16 tokens: with 0.05 layers of 9 to 12 k-tiles take 2 x 4 blocks, which the scales make slower than 1 x 8; 2746
    // drawn calls whose block that decides, median time 0.90, largest 1.10 at 304 rows)
    const double per_group = w.grouped && c.nt == 1 && c.xr == 16 ? 0.045 : 0.05, groups = c.wk > 1 ? 0.1 + per_group * c.wk * c.nt : 0.0;
    const double alone = stages * (0.38 + (w.packed ? 0.005 : 0.016) * weight_kb + x_us) + handover;
    const double memory = (double)M * (double)K * w.bits / 8.0 / (w.packed ? 6.9e6 : 5.4e6) + stages * 0.5 * x_us + 0.3 * handover;
    return (alone > memory ? alone : memory) + groups;
}

// The block and the split-K factor with the least estimated time, with no more partial sums than the caller's workspace
// holds.  Few row tiles: fewer of them per block and more groups of k-tiles, so that the chip is full without k slices
// (4096 x 4096, N = 1 8.4 us with S = 8 and eight row tiles, 4.7 with one; 2048 x 16384, N = 1 13.2 -> 7.8; 8192 x 8192,
// N = 1 11.6 -> 10.2); more tokens: more row tiles, which share the copies of the activations (8192 x 22016, N = 16 23.0 us
// with eight, 26.0 with two).  Six row tiles where eight leave CUs idle (12288 x 12288, N = 45 28.4 -> 25.6).
StreamPlan plan_stream(int64_t M, int64_t N, int64_t K, const StreamWeights &w)
{
    const StreamCfg *table = w.packed ? kStreamCfg : kStreamCfgFp16;
    const int64_t row_tiles = M / kTileRows;
    const int64_t KT = (K + w.tile_cols - 1) / w.tile_cols;  // steps of the streaming kernel for this source
    const int64_t forced = g_forced_split.load(std::memory_order_relaxed);
    const int64_t max_split = KT >= 4 ? KT / 2 : 1;  // at least two k-tiles per slice
    const int nt = (int)((N + 15) / 16), xr = !w.packed || N > 8 ? 16 : N > 2 ? 8 : 2;
    const StreamSlices shape = stream_slices_of_shape(M, N, KT, w.packed);
    StreamPlan p{-1, 1, 0, 0, 0, 0, 0};
    double best = 0.0;
    for (int i = 0; i < (w.packed ? kStreamCfgs : kStreamCfgsFp16); ++i) {
        const StreamCfg &c = table[i];
        if (c.nt != nt || c.xr != xr || !stream_cfg_built(c, w))
            continue;
        const int64_t rb = (row_tiles + c.wm - 1) / c.wm;
        if (p.cfg >= 0 && rb > kCus)
            continue;  // a second round, most of it idle: one row of blocks more than CUs costs up to half as much again
        int64_t s = forced > 0 ? forced : kCus / rb;
        s = s > max_split ? max_split : s;
        if (forced <= 0 && s * nt > shape.split * shape.nt)
            s = shape.split * shape.nt / nt;
        s = s > 64 ? 64 : s < 1 ? 1 : s;
        // the kernel addresses the partial tiles with 32-bit byte offsets
        while (s > 1 && (uint64_t)s * (uint64_t)row_tiles * (uint64_t)nt * 1024u >= (1ull << 31))
            s /= 2;
        // ... and, with the k-tiles dealt to slices and groups, the weights with 32-bit offsets that step by s * wk k-tiles
        // and run up to five such steps past the end of a slice (look-ahead of the pipeline; those read as zeros)
        while (s > 1 && (uint64_t)(KT + (c.wk > 4 ? 5 * c.wk : 20) * s) * (uint64_t)row_tiles * kTileBytes >= (1ull << 31))
            s /= 2;
        for (;; s /= 2) {  // the most slices, then halves
            // Six row tiles with four token tiles (3 bits: with two as well) and no k slices take as many stages as the plan without them and
            // copy the activations more often.  Median time without them over that with them, drawn calls, weights from memory: 6 bits 0.91, 5 and
            // 4 bits 0.95, 3 bits 0.91 and 0.96 (5165 calls, largest 1.02), group scales 0.85 up to 128 row blocks of eight (1862 calls, largest
            // 0.96) but up to 1.06 beyond, where they keep them.  (With slices six row tiles take 0.97 to 1.05 of the time of eight.)
            if (w.packed && c.wm == 6 && (nt == 4 || (nt == 2 && w.bits == 3)) && s == 1 && !(w.grouped && row_tiles > 8 * 128))
                break;
            const double cost = stream_cost(c, M, K, s, w);
            // fp16 weights at the memory's rate: where the estimate is the same for two blocks, the one that fills more CUs (5424 x
            // 20992, N = 9 47.1 -> 36.8 us; 5081 drawn calls with such a tie, median time 0.90, largest 1.05; packed weights lose by it)
            const bool fuller = !w.packed && cost == best && rb * s > (int64_t)p.row_blocks * p.split;
            if (p.cfg < 0 || cost < best || fuller) {
                p.cfg = i;
                p.split = (int)s;
                p.row_blocks = (int)rb;
                best = cost;
            }
            if (forced > 0 || s == 1)
                break;
        }
        if (forced > 0)
            break;  // the tuning hook pins the first candidate, so that tests reach every split factor
    }
    const auto counters = [&] { return ((size_t)row_tiles * sizeof(int) + 255) / 256 * 256; };  // one per row tile
    const auto partials = [&](int64_t s, int64_t n) { return (size_t)s * (size_t)row_tiles * (size_t)n * 64 * sizeof(float4_t); };
    if (p.split > 1) {
        p.counter_bytes = p.required_counters = counters();
        p.partial_bytes = p.required_partials = partials(p.split, nt);
    } else if (forced <= 0 && shape.split > 1) {
        p.required_counters = counters();
        p.required_partials = partials(shape.split, shape.nt);
    }
    return p;
}

// ---- tiled kernel (prefill-sized N) -----------------------------------------

// Block shapes offered by the tiled kernel: {RT, NT, WM, WN, WK}; block = (16*RT*WM) rows x (16*NT*WN) tokens.  WK: the most k
// groups it is launched with, see two_k_groups().
struct TileShape {
    int rt, nt, wm, wn, wk;
    int rows() const { return 16 * rt * wm; }
    int tokens() const { return 16 * nt * wn; }
};
constexpr TileShape kTile256x128{2, 8, 8, 1, 1};
constexpr TileShape kTile128x128{2, 4, 4, 2, 1};
constexpr TileShape kTile256x64{2, 4, 8, 1, 1};
constexpr TileShape kTile128x64{2, 4, 4, 1, 2};

// A kernel that uses more than 64 KB of dynamic LDS has to be told so once per device.  `done` holds one
// bit per device ordinal (mod 64); safe to call from several host threads.
bool allow_dynamic_lds(const void *kernel, size_t bytes, std::atomic<uint64_t> &done)
{
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess)
        return false;
    const uint64_t bit = 1ull << (device & 63);
    if (done.load(std::memory_order_acquire) & bit)
        return true;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess)
        return false;
    done.fetch_or(bit, std::memory_order_release);
    return true;
}

std::atomic<int> g_forced_tile{0};  // 0 = automatic, else rows * 1024 + tokens (tuning hook)

// ---- block kernel (prompt-sized N: fp16 weights, group-wise scales, and large products) -----------------------

// Block shapes: {rows, tokens}.  Costs are ns per run of 32 columns with most CUs busy (median of 2000 drawn calls, K >= 4096),
// for fp16 weights and for 6-bit weights with group scales.
struct BlockCfg {
    int rows, tokens;
    double fp16_ns, group_ns;
    constexpr int k_groups() const { return rows == 128 ? 2 : 1; }
};
constexpr int kBlockCfgs = 4, kBlock256x256 = 0, kBlock128x128 = 2;
constexpr BlockCfg kBlockCfg[kBlockCfgs] = {{256, 256, 805, 0}, {256, 128, 590, 480}, {128, 128, 258, 293}, {128, 64, 198, 0}};
// BlockShape<RT, NT, WM, WN, WK, SR, XST, WD, ADB> of each, for run-staged (fp16) and packed weights
template <bool RUN_STAGED, int C>
struct BlockShapeOf;
template <> struct BlockShapeOf<false, 0> { typedef BlockShape<4, 8, 4, 2, 1, 1, 6, 1, false> type; };
template <> struct BlockShapeOf<false, 1> { typedef BlockShape<4, 4, 4, 2, 1, 2, 4, 1, true> type; };
template <> struct BlockShapeOf<false, 2> { typedef BlockShape<4, 4, 2, 2, 2, 1, 5, 2, true> type; };
template <> struct BlockShapeOf<true, 0> { typedef BlockShape<4, 8, 4, 2, 1, 1, 4, 1, true> type; };
template <> struct BlockShapeOf<true, 1> { typedef BlockShape<4, 4, 4, 2, 1, 1, 6, 1, true> type; };
template <> struct BlockShapeOf<true, 2> { typedef BlockShape<4, 4, 2, 2, 2, 1, 4, 1, true> type; };
template <> struct BlockShapeOf<true, 3> { typedef BlockShape<4, 2, 2, 2, 2, 1, 6, 1, true> type; };
constexpr int kBlockWaves = 8;

// the source through which the block kernel reads a weight format
template <class Src>
struct BlockSourceOf;
template <> struct BlockSourceOf<PackedFp6Source> { typedef BlockFp6Source type; };
template <> struct BlockSourceOf<PackedFp6GroupSource> { typedef BlockFp6GroupSource type; };
template <> struct BlockSourceOf<PackedFp5Source> { typedef BlockFp5Source type; };
template <> struct BlockSourceOf<PackedFp4Source> { typedef BlockFp4Source type; };
template <> struct BlockSourceOf<PackedFp3Source> { typedef BlockFp3Source type; };
template <> struct BlockSourceOf<PlainFp16Source> { typedef BlockFp16Source type; };

struct BlockPlan {
    int cfg;  // -1: the tiled kernel instead
    int split;
    int row_blocks, n_blocks, chunk;  // chunk: output pieces per XCD
    int counter_step;
    size_t counter_bytes, partial_bytes;  // 0 without k slices
};

enum class Weights { kFp6, kFp5, kFp4, kFp3, kGrouped, kFp16 };
constexpr bool per_row(Weights kind) { return kind != Weights::kGrouped && kind != Weights::kFp16; }  // packed, a scale per row
template <class Src>
constexpr Weights weights_of()
{
    if constexpr (std::is_same_v<Src, PlainFp16Source>)
        return Weights::kFp16;
    else if constexpr (std::is_same_v<Src, PackedFp6GroupSource>)
        return Weights::kGrouped;
    else
        return Src::kBits == 6 ? Weights::kFp6 : Src::kBits == 5 ? Weights::kFp5 : Src::kBits == 4 ? Weights::kFp4 : Weights::kFp3;
}

// partial_limit: bytes that the partial tiles may take
BlockPlan block_plan_of(int cfg, int64_t M, int64_t N, int64_t K, size_t partial_limit = SIZE_MAX)
{
    BlockPlan p;
    p.cfg = cfg;
    const BlockCfg &b = kBlockCfg[cfg];
    const int64_t KT = K / kTileK;
    p.row_blocks = (int)((M + b.rows - 1) / b.rows);
    p.n_blocks = (int)((N + b.tokens - 1) / b.tokens);
    int64_t s = g_forced_split.load(std::memory_order_relaxed);
    if (s <= 0)
        s = kCus / ((int64_t)p.row_blocks * p.n_blocks);  // one block per CU
    const int64_t max_split = KT >= 8 ? KT / 4 : 1;  // at least four k-tiles per slice
    s = s > max_split ? max_split : s;
    s = s > 16 ? 16 : s;
    const size_t tiles = (size_t)p.row_blocks * p.n_blocks, slice_bytes = tiles * b.rows * b.tokens * sizeof(float);
    if (s > 1 && slice_bytes * (size_t)s > partial_limit)
        s = (int64_t)(partial_limit / slice_bytes);
    p.split = (int)(s < 1 ? 1 : s);
    p.chunk = pieces_per_xcd(p.row_blocks * p.split, p.n_blocks);
    p.counter_bytes = p.partial_bytes = 0;
    p.counter_step = counter_step(tiles * kBlockWaves);  // one arrival counter per wave tile
    if (p.split > 1) {
        p.counter_bytes = counter_bytes_of(tiles * kBlockWaves, p.counter_step);
        p.partial_bytes = (size_t)p.split * slice_bytes;
    }
    return p;
}

struct TiledPlan {
    TileShape tile;
    int split, k_groups;
    int row_blocks, n_blocks;
    int counter_step;
    size_t counter_bytes, partial_bytes;  // 0 without k slices
};

// few row blocks and a short prompt: small blocks and little split-K (measured on 8192-row layers)
bool few_blocks(int64_t M, int64_t N) { return N <= 128 && (M + 255) / 256 < 64; }

// Whether the 128 x 64 block of the tiled kernel takes two groups of k-tiles (eight waves) instead of one (four).  Worth it where
// the conversions are long beside the matrix work and a slice is long enough for the second pipeline fill and the meeting in LDS.
// Median time with two over one, 1166 calls of 256 to 57344 rows and 65 to 128 tokens, by k-tiles per slice:
//                  < 8    8-12   12-20  20-40  > 40
//   3 bits         0.95   0.93   0.91   0.89   0.85    (largest 1.15, 0.96, 0.96, 1.03, 0.88)
//   4 bits         0.97   0.96   0.95   0.91   0.91    (1.16, 1.09, 0.99, 0.97, 0.94)
//   5 bits         1.00   0.99   0.98   0.96   0.93    (1.22, 1.04, 1.17, 1.00, 0.95)
//   6 bits         1.03   1.03   1.02   1.00   1.00
//   group scales   1.08   1.04   1.01   0.98   0.97    (1.25, 1.14, 1.09, 0.99, 0.99)
bool two_k_groups(Weights kind, int64_t K, int split)
{
    const int64_t k_tiles = K / kTileK / split;
    return kind != Weights::kFp6 && k_tiles >= (kind == Weights::kFp3 || kind == Weights::kFp4 ? 12 : 20);
}

TiledPlan tiled_plan_of(const TileShape &tile, int64_t M, int64_t N, int64_t K, Weights kind)
{
    TiledPlan p;
    const int64_t row_tiles = M / kTileRows;
    const int64_t KT = K / kTileK;
    p.tile = tile;
    p.row_blocks = (int)((M + p.tile.rows() - 1) / p.tile.rows());
    p.n_blocks = (int)((N + p.tile.tokens() - 1) / p.tile.tokens());
    int64_t s = g_forced_split.load(std::memory_order_relaxed);
    if (s <= 0)
        s = 256 / ((int64_t)p.row_blocks * p.n_blocks);  // one block per CU
    const int64_t max_split = KT >= 8 ? KT / 4 : 1;  // at least four k-tiles per slice
    if (s > max_split)
        s = max_split;
    if (s > 16)
        s = 16;
    if (s < 1)
        s = 1;
    p.split = (int)s;
    p.k_groups = p.tile.wk == 2 && two_k_groups(kind, K, p.split) ? 2 : 1;
    const int bnt = p.tile.nt * p.tile.wn;
    const size_t counters = (size_t)p.row_blocks * p.n_blocks * p.tile.wm * p.tile.wn * p.k_groups;  // one per wave
    p.counter_bytes = p.partial_bytes = 0;
    p.counter_step = counter_step(counters);
    if (p.split > 1) {
        p.counter_bytes = counter_bytes_of(counters, p.counter_step);
        p.partial_bytes = (size_t)p.split * (size_t)row_tiles * (size_t)p.n_blocks * bnt * 64 * sizeof(float4_t);
    }
    return p;
}

// Weights with group scales: the 128 x 64 block (their 128 x 128 one is chosen in plan_prompt).
TiledPlan plan_tiled(int64_t M, int64_t N, int64_t K, Weights kind)
{
    const int forced = g_forced_tile.load(std::memory_order_relaxed);
    const int rows = forced / 1024, tokens = forced % 1024;
    TileShape tile = few_blocks(M, N) ? kTile128x64 : kTile256x128;  // the latter moves the fewest bytes per MFMA
    if (forced > 0)
        tile = rows == 256 ? (tokens == 128 ? kTile256x128 : kTile256x64) : (tokens == 128 ? kTile128x128 : kTile128x64);
    return tiled_plan_of(kind == Weights::kGrouped ? kTile128x64 : tile, M, N, K, kind);
}

// What a call of more than kStreamMaxN tokens launches: the block kernel where `block.cfg` is set, else the tiled one.
struct PromptPlan {
    TiledPlan tiled;
    BlockPlan block;
    bool instead_of_tiled;  // the block where `tiled` says what the call asks its caller for
    bool is_block() const { return block.cfg >= 0; }
    int split() const { return is_block() ? block.split : tiled.split; }
    size_t counter_bytes() const { return is_block() ? block.counter_bytes : tiled.counter_bytes; }
    size_t partial_bytes() const { return is_block() ? block.partial_bytes : tiled.partial_bytes; }
    // What the size query names and a call is refused without: never less than what the launch uses.
    size_t required_counters() const { return instead_of_tiled && tiled.counter_bytes > counter_bytes() ? tiled.counter_bytes : counter_bytes(); }
    size_t required_partials() const { return instead_of_tiled ? tiled.partial_bytes : partial_bytes(); }
};

// Estimated time of a block plan, ns: rounds of 256 blocks at the measured cost per run, a fixed part per round, and for
// split-K what the last arrival reads (its tile of every slice, at the ~50 GB/s one CU gets) and what all slices write.
double block_cost(const BlockPlan &p, int64_t K, double run_ns)
{
    const BlockCfg &b = kBlockCfg[p.cfg];
    const double blocks = (double)p.row_blocks * p.n_blocks * p.split;
    const double rounds = (double)(((int64_t)blocks + kCus - 1) / kCus);
    const double runs = 8.0 * (double)((K / kTileK + p.split - 1) / p.split);
    const double ns = rounds * (runs * run_ns + 8000.0);
    return p.split == 1 ? ns : ns + (double)p.split * b.rows * b.tokens * 4.0 / 50.0 + (double)p.partial_bytes * 1.5e-4;
}
double block_cost(const BlockPlan &p, int64_t K, Weights kind)
{
    const BlockCfg &b = kBlockCfg[p.cfg];
    // 128-row blocks of fp16 weights fetch twice the bytes per product, and long rows of both operands share fewer L2 sets
    // (258 ns up to K = 12288, 300 to 340 beyond 20000)
    const double long_rows = b.rows == 128 && K > 12288 ? 1.0 + 0.25 * (double)((K < 28672 ? K : 28672) - 12288) / 12288.0 : 1.0;
    return block_cost(p, K, kind == Weights::kFp16 ? b.fp16_ns * long_rows : b.group_ns);
}

// Estimated time, us, of the plans that weights with a scale per row choose between: rounds of the chip, each with a fixed part and a
// cost per run of 32 columns that grows with the share of CUs that have a block; what k slices cost; and no faster than the weights
// come from memory.  Fitted to 20514 drawn calls of 128 to 57344 rows and 65 to 4096 tokens, weights from memory (mean error 4.5 to 5 %).
struct PerRowCost {
    double fixed, slices, per_slice, memory_rate, fill, run[4];  // run: 6, 5, 4, 3 bits
    double operator()(double rounds, int64_t blocks, int split, int64_t M, int64_t K, Weights kind, double run_share = 1.0) const
    {
        const int f = kind == Weights::kFp6 ? 0 : kind == Weights::kFp5 ? 1 : kind == Weights::kFp4 ? 2 : 3;
        const double runs = 8.0 * (double)((K / kTileK + split - 1) / split), busy = (double)blocks / kCus / rounds;
        const double alone = rounds * (fixed + runs * run[f] * run_share * (1.0 + fill * (busy < 1.0 ? busy : 1.0))) + (split > 1 ? slices + per_slice * split : 0.0);
        const double memory = (double)M * (double)K * (6 - f) / 8.0 * 1e-6 / memory_rate;
        return alone > memory ? alone : memory;
    }
};
constexpr PerRowCost kBlock128Cost{6.62, 2.11, 0.543, 2.68, 0.606, {0.1398, 0.1516, 0.1244, 0.1295}};
constexpr PerRowCost kTiled256Cost{7.20, 0.995, 1.20, 3.21, 0.534, {0.2476, 0.2487, 0.2268, 0.2257}};
constexpr PerRowCost kTiled64Cost{4.27, 0.88, 0.425, 2.53, 0.336, {0.0951, 0.1073, 0.0845, 0.0883}};

// Whether the block kernel's 128 x 128 block takes a call from the tiled kernel (256 x 128 blocks, or 128 x 64).  It has half as many k
// slices where 256-row blocks leave CUs idle and whole units per XCD where those are dealt unevenly.  Median time over the tiled
// kernel's, drawn calls as above, by their k slices: 256 x 128, two 0.78-0.99, three to five 0.78-0.86, six and more 0.61, none 1.08
// (a tenth of them below 0.73: rounds); 128 x 64 0.88 to 1.55.  As chosen: 0.805 over all 20514 calls, 0.803 if the faster one were
// known; 12 calls more than 3 % slower.  3443 of the calls that it moves, drawn anew, each with the tiled kernel pinned in turn: median 0.69
// (by format and k slices 0.54 to 0.90), five more than 3 % slower, the most 1.10.
//   Fewer rows: the waves of a 256-row block that have none leave its runs cheaper, and the little that the tiled plan asks its caller for
// holds the 128 x 128 block to fewer k slices still (16 x 22016, N = 309, 3 bits, 2 for 16: 64.3 us for 40.3; 16 x 14080, N = 847, 1 for 13:
// 79.4 for 51.6).  Where it has a third of them or less the estimate counts that: of 3078 drawn calls of 16 to 272 rows 36 stay with
// the tiled kernel, 29 of them more than 3 % faster there; of 4065 others five are 3 to 17 % slower, the median 0.63 of its time.
//   128 x 64 tiles: the block only wins for rows of more than 100 000 columns (1152 x 211968, N = 103, 5 bits 152.5 -> 114.4 us; 24 such calls
// 0.74 to 0.91), where those take 14 slices of long runs.
bool block128_is_faster(const BlockPlan &b, const TiledPlan &t, int64_t M, int64_t K, Weights kind)
{
    const double fullest = (double)((int64_t)((t.row_blocks + kXcds - 1) / kXcds) * t.n_blocks * t.split) / kCusPerXcd;
    const bool wide = t.tile.tokens() == 128;
    // two 128 x 64 blocks share a CU
    const double rounds = wide ? (double)(int64_t)(fullest + 1.0 - 1e-9) : fullest <= 1.0 ? 1.0 : fullest > 2.0 ? fullest : 1.0 + 0.9 * (fullest - 1.0);
    const double share = wide && M < 200 && t.split >= 3 * b.split ? 0.2 + 0.8 * std::sqrt((double)M / 200.0) : 1.0;
    const double tiled = (wide ? kTiled256Cost : kTiled64Cost)(rounds, (int64_t)t.row_blocks * t.n_blocks * t.split, t.split, M, K, kind, share);
    const double block = kBlock128Cost((double)((b.chunk + kCusPerXcd - 1) / kCusPerXcd), (int64_t)b.row_blocks * b.n_blocks * b.split, b.split, M, K, kind);
    return 1.03 * block < tiled;
}

// Partial sums with which fp16_linear runs at any rate: those of the block that kFp16AcceptedNs chooses.  These figures are not
// for speed and stay as they are when the ones above are measured anew: a caller that had enough has enough.
constexpr double kFp16AcceptedNs[kBlockCfgs] = {924, 632, 333, 228};
size_t fp16_accepted_partials(int64_t M, int64_t N, int64_t K)
{
    size_t bytes = 0;
    double best = 0.0;
    for (int c = 0; c < kBlockCfgs; ++c) {
        const BlockPlan b = block_plan_of(c, M, N, K);
        const double cost = block_cost(b, K, kFp16AcceptedNs[c]);
        if (c == 0 || cost < best) {
            bytes = b.partial_bytes;
            best = cost;
        }
    }
    return bytes;
}

// Whether the cheapest block plan for group scales has so few k-tiles per block that the tiled kernel's 128 x 128 blocks
// are faster: the block kernel pays more before and after its k loop (its rings fill, two waves meet in LDS, the last
// slice reads its own partial tiles back).  The tiled kernel deals whole row blocks to the XCDs, so it has to be done in one
// round on the fullest of them (in two it takes 1.3 to 2 times as long), and it gains less where few XCDs hold most blocks.
// Median time of the block kernel over the tiled one's, 5400 calls of 256 to 57344 rows and 129 to 1200 tokens, by k-tiles
// per block:
//   no k slices, up to 8 blocks on an XCD     2 1.06, 3 1.04, 4 1.03, 5 1.01, 6 1.00
//   no k slices, more blocks                  2 1.04, 3 1.01, 4 0.98, 5 0.97
//   2 or 3 slices                             4 1.17, 5 1.12, 6 1.08, 7 1.06
//   4 to 7 slices                             4 1.15, 5 1.07, 6 1.05, 7 1.01
//   8 to 16 slices                            4 1.10, 5 1.02, 6 0.96
//   slices, more than 16 blocks on an XCD and 1.6 times the average   4 1.04, 5 1.00, 6 0.97
//   256 x 128 blocks in slices                4 1.03, 5 0.96
// (2048 x 4096, N = 265: 21.2 us against 18.0; 784 x 512, N = 636: 8.2 against 7.7; 6448 x 2048, N = 245: 20.5 against 16.6.)
bool short_blocks(const BlockPlan &b, const TiledPlan &tiled, int64_t K)
{
    const int64_t blocks = (int64_t)tiled.row_blocks * tiled.n_blocks * tiled.split;
    const int64_t fullest = (int64_t)((tiled.row_blocks + kXcds - 1) / kXcds) * tiled.n_blocks * tiled.split;
    if (fullest > kCusPerXcd)
        return false;
    const int64_t k_tiles = (K / kTileK + b.split - 1) / b.split;
    if (b.split == 1)
        return kBlockCfg[b.cfg].rows == 128 && k_tiles <= (fullest <= 8 ? 5 : 3);
    const bool uneven = fullest > 16 && 5 * fullest >= 8 * ((blocks + kXcds - 1) / kXcds);
    if (uneven || kBlockCfg[b.cfg].rows == 256)
        return k_tiles <= 4;
    return k_tiles <= (b.split < 4 ? 7 : b.split < 8 ? 6 : 5);
}

// Which kernel and block (us, this kernel against the tiled one in the same process):
//   per-row packed weights: the 256 x 256 block, at up to 1.17x the rate of the tiled kernel's 256 x 128 one, where its
//     rounds of 256 blocks and its padded tokens take at most 1.1x what that block's do - which also says that it
//     needs no split-K (57344 x 8192, N = 4096 2764 against 3186; 28672 x 8192, N = 3000 1110 against 1167; 9216 x
//     9216, N = 1024, 144 tiles in one round against 288 in two, 172 against 206 with 6 bits, 162 against 188 with 4,
//     202 against 219 with 5, 168 against 193 with 3).  Drawn calls of 256 to 57344 rows and 65 to 4096 tokens, time over
//     that without it, median and largest: 6 bits 0.87, 0.98; 5 bits 0.93, 1.02; 4 bits 0.88, 0.98; 3 bits 0.90, 1.03 (800
//     in all).  Beyond that rule it loses: 8192 x 8192, N = 1024 127 against 110, 28672 x 8192, N = 700 344 against 294,
//     57344 x 4096, N = 300 175 against 155.  Elsewhere the 128 x 128 block, where block128_is_faster();
//   group scales: always, except few rows and few tokens (8192 x 8192, N = 100: 31 against 30; 4096 x 4096 17 against
//     13; but 28672 x 8192, N = 201 107 against 160, 16384 x 8192, N = 2048 497 against 740) and short blocks, see
//     short_blocks();
//   fp16 weights: always (9216 x 9216, N = 256 64 against 155; 16384 x 8192, N = 2048 473 against 1176; 8192 x 8192,
//     N = 100 38 against 43; 1536 x 4864, N = 241 16.4 against 32.8; 608 x 1024, N = 106 6.8 against 12.8; 3684 drawn
//     calls of the range above: median 0.46, largest 0.93).
// Among its blocks the cheapest by block_cost().
PromptPlan plan_prompt(int64_t M, int64_t N, int64_t K, Weights kind, size_t partial_limit = SIZE_MAX)
{
    PromptPlan p;
    p.block.cfg = -1;
    p.instead_of_tiled = false;
    p.tiled = plan_tiled(M, N, K, kind);
    const int forced = g_forced_tile.load(std::memory_order_relaxed);
    if (forced > 0) {
        const int rows = forced / 1024, tokens = forced % 1024;
        int cfg = -1;
        if (tokens == 256)
            cfg = kind == Weights::kGrouped ? 1 : kBlock256x256;
        else if (!per_row(kind) && tokens == 128)
            cfg = rows == 256 ? 1 : 2;
        else if (kind == Weights::kFp16)
            cfg = 3;
        if (cfg >= 0)
            p.block = block_plan_of(cfg, M, N, K);
        return p;
    }
    const int64_t row_blocks = (M + 255) / 256;
    if (per_row(kind)) {
        const int64_t tiles = row_blocks * ((N + 255) / 256), halves = row_blocks * ((N + 127) / 128);
        const int64_t rounds = (tiles + kCus - 1) / kCus, half_rounds = (halves + kCus - 1) / kCus;
        if (20 * rounds <= 11 * half_rounds && 20 * tiles <= 11 * halves) {
            p.block = block_plan_of(kBlock256x256, M, N, K);
        } else if (g_forced_split.load(std::memory_order_relaxed) <= 0) {  // the hook pins the tiled kernel
            // no more partial sums than the tiled plan, whose size the caller was told
            const BlockPlan b = block_plan_of(kBlock128x128, M, N, K, p.tiled.partial_bytes);
            if (block128_is_faster(b, p.tiled, M, K, kind)) {
                p.block = b;
                p.instead_of_tiled = true;
            }
        }
        return p;
    }
    if (kind == Weights::kGrouped && few_blocks(M, N))
        return p;
    double best = 0.0;
    // with group scales the 256 x 256 block does not fit the registers, the 128 x 64 one loses to the tiled kernel
    const bool fp16 = kind == Weights::kFp16;
    for (int c = fp16 ? 0 : 1; c < (fp16 ? kBlockCfgs : kBlockCfgs - 1); ++c) {
        const BlockPlan b = block_plan_of(c, M, N, K, partial_limit);
        const double cost = block_cost(b, K, kind);
        if (p.block.cfg < 0 || cost < best) {
            p.block = b;
            best = cost;
        }
    }
    if (kind == Weights::kGrouped) {
        const TiledPlan tiled = tiled_plan_of(kTile128x128, M, N, K, kind);
        if (tiled.partial_bytes <= partial_limit && short_blocks(p.block, tiled, K)) {
            p.tiled = tiled;
            p.block.cfg = -1;
        }
    }
    return p;
}

template <class Src, int C>
fp6_status launch_block_cfg(const BlockPlan &p, const void *weights, const void *scales, const void *X, void *Y, int64_t M,
                            int64_t N, int64_t K, float4_t *partials, int *counters, const Epilogue &epi, hipStream_t stream)
{
    typedef typename BlockSourceOf<Src>::type Source;
    typedef typename BlockShapeOf<Source::kRunStaged, C>::type Shape;
    static_assert(Shape::BM == kBlockCfg[C].rows && Shape::BN == kBlockCfg[C].tokens && Shape::WAVES == kBlockWaves
                      && Shape::WK == kBlockCfg[C].k_groups(),
                  "the table and the shape disagree");
    auto kernel = linear_block_kernel<Source, Shape>;
    constexpr size_t lds = Shape::template lds_bytes<Source>();
    static_assert(lds <= 160 * 1024, "activation ring and weight tiles exceed the LDS of a CU");
    static std::atomic<uint64_t> lds_done{0};  // per instantiation
    if (!allow_dynamic_lds(reinterpret_cast<const void *>(kernel), lds, lds_done))
        return FP6_ERR_HIP;
    const dim3 grid((unsigned)(kXcds * p.chunk)), block(Shape::kThreads);
    hipLaunchKernelGGL(kernel, grid, block, lds, stream, weights, static_cast<const half_t *>(scales),
                       static_cast<const half_t *>(X), static_cast<half_t *>(Y), (int)M, (int)N, (int)K, p.split,
                       p.n_blocks, p.row_blocks, p.chunk, partials, counters, p.counter_step, epi);
    return hipGetLastError() == hipSuccess ? FP6_OK : FP6_ERR_HIP;
}

template <class Src, int RT, int NT, int WM, int WN, int WK>
fp6_status launch_tiled_cfg(const TiledPlan &p, const void *weights, const void *scales, const void *X, void *Y,
                            int64_t M, int64_t N, int64_t K, float4_t *partials, int *counters, const Epilogue &epi,
                            hipStream_t stream)
{
    auto kernel = linear_tiled_kernel<Src, RT, NT, WM, WN, WK>;
    constexpr size_t lds = (size_t)4 * WK * WN * NT * 256 * 16;  // a ring of four half tiles of activations per k group
    static std::atomic<uint64_t> lds_done{0};  // per instantiation
    if (!allow_dynamic_lds(reinterpret_cast<const void *>(kernel), lds, lds_done))
        return FP6_ERR_HIP;
    // row blocks are dealt to the 8 XCDs round-robin: the grid is padded to a multiple of 8 row blocks
    const int padded_row_blocks = (p.row_blocks + 7) / 8 * 8;
    const dim3 grid((unsigned)(padded_row_blocks * p.n_blocks * p.split)), block(WM * WN * WK * 64);
    hipLaunchKernelGGL(kernel, grid, block, lds, stream, weights, static_cast<const half_t *>(scales),
                       static_cast<const half_t *>(X), static_cast<half_t *>(Y), (int)M, (int)N, (int)K, p.split,
                       p.n_blocks, partials, counters, p.counter_step, epi);
    return hipGetLastError() == hipSuccess ? FP6_OK : FP6_ERR_HIP;
}

// Both kernels address the activations with 32-bit byte offsets, so one launch takes at most this many
// tokens (a multiple of 128, so that a full chunk ends with whole tiled blocks and at most half a 256-token one);
// longer inputs are processed in chunks on the same stream.
int64_t prompt_chunk_tokens(int64_t K)
{
    const int64_t fit = ((1ll << 31) - 1) / (2 * K);
    return fit >= 128 ? fit / 128 * 128 : fit;  // shape_ok() admits K < 2^24 only: at least 64 tokens fit
}

// Token counts of the launches that a prompt-sized call is cut into: the full chunk and the shorter last one (0: none).
struct PromptChunks {
    int64_t n[2];
    const int64_t *begin() const { return n; }
    const int64_t *end() const { return n + 2; }
};
PromptChunks prompt_chunks(int64_t N, int64_t K)
{
    const int64_t chunk = prompt_chunk_tokens(K);
    return {{N < chunk ? N : chunk, N > chunk ? N % chunk : (int64_t)0}};
}

// Bytes at the start of a caller's workspace that hold arrival counters: the same for every shape, and with a forced
// split factor for every weight format of the shape.
size_t counter_region_bytes(int64_t M, int64_t N, int64_t K)
{
    size_t bytes = kCounterBytes;
    if (g_forced_split.load(std::memory_order_relaxed) <= 0)
        return bytes;
    auto at_least = [&](size_t b) { bytes = b > bytes ? b : bytes; };
    if (N <= kStreamMaxN) {
        at_least(plan_stream(M, N, K, stream_weights_of<PackedFp6Source>()).counter_bytes);
        at_least(plan_stream(M, N, K, stream_weights_of<PackedFp3Source>()).counter_bytes);
        at_least(plan_stream(M, N, K, stream_weights_of<PlainFp16Source>()).counter_bytes);
        return bytes;
    }
    for (Weights kind : {Weights::kFp6, Weights::kFp5, Weights::kFp4, Weights::kFp3, Weights::kGrouped, Weights::kFp16})
        for (int64_t n : prompt_chunks(N, K))
            if (n > 0)
                at_least(plan_prompt(M, n, K, kind).required_counters());
    return bytes;
}

// Workspace of a call: the counters and the most partial tiles that one of its launches has (the last, shorter chunk of
// a prompt may use more k slices than the full ones).
size_t split_workspace_bytes(size_t partial_bytes, int64_t M, int64_t N, int64_t K)
{
    return partial_bytes > 0 ? counter_region_bytes(M, N, K) + partial_bytes : 0;
}

// The largest of the given weights (formats that share a size query).
size_t stream_workspace_bytes(int64_t M, int64_t N, int64_t K, std::initializer_list<StreamWeights> weights)
{
    size_t bytes = 0;
    for (const StreamWeights &w : weights) {
        const size_t b = plan_stream(M, N, K, w).required_partials;
        bytes = b > bytes ? b : bytes;
    }
    return split_workspace_bytes(bytes, M, N, K);
}

size_t prompt_workspace_bytes(int64_t M, int64_t N, int64_t K, Weights kind)
{
    size_t partial_bytes = 0;
    for (int64_t n : prompt_chunks(N, K))
        if (n > 0) {
            const size_t b = plan_prompt(M, n, K, kind).required_partials();
            partial_bytes = b > partial_bytes ? b : partial_bytes;
        }
    return split_workspace_bytes(partial_bytes, M, N, K);
}

// The plan of a launch on the workspace that the caller brought.  The queried size holds the k slices of the best plan.
// A smaller one, or none, is refused - unless it holds what 128 x 128 blocks need (128 x 64 on few row blocks): they
// need no k slices where more than half of the CUs have a block, and callers of fp16_linear and fp6g_linear may rely on
// that; or, fp16_linear, what fp16_accepted_partials() says.  The call then runs with as many slices as fit (8192 x 22016,
// N = 512, fp16: 67 MB and 256 x 256 blocks in 4 slices as queried, 128 x 128 blocks without a workspace).
fp6_status plan_prompt_within(int64_t M, int64_t N, int64_t K, Weights kind, const WorkspaceRef &workspace, PromptPlan &p, SplitBuffers &buf)
{
    p = plan_prompt(M, N, K, kind);
    const fp6_status fits = workspace.view(p.required_counters(), p.required_partials(), buf);
    if (fits != FP6_ERR_WORKSPACE || !p.is_block() || p.instead_of_tiled || g_forced_split.load(std::memory_order_relaxed) > 0)
        return fits;
    const TiledPlan least = tiled_plan_of(few_blocks(M, N) ? kTile128x64 : kTile128x128, M, N, K, kind);
    const size_t bytes = workspace.base ? workspace.bytes : 0, region = workspace.counter_region;
    size_t enough = least.partial_bytes;
    if (kind == Weights::kFp16 && fp16_accepted_partials(M, N, K) < enough)
        enough = fp16_accepted_partials(M, N, K);
    if (enough > 0 && bytes < region + enough)
        return fits;
    p = plan_prompt(M, N, K, kind, bytes > region ? bytes - region : 0);
    return workspace.view(p.counter_bytes(), p.partial_bytes(), buf);
}

template <class Src>
fp6_status launch_prompt_chunk(const void *weights, const void *scales, const void *X, void *Y, int64_t M, int64_t N,
                              int64_t K, const WorkspaceRef &workspace, const Epilogue &epi, hipStream_t stream)
{
    PromptPlan p;
    SplitBuffers buf;
    const fp6_status fits = plan_prompt_within(M, N, K, weights_of<Src>(), workspace, p, buf);
    if (fits != FP6_OK)
        return fits;
    int *counters = buf.counters;
    float4_t *partials = reinterpret_cast<float4_t *>(buf.partials);
    if (p.is_block()) {
        const BlockPlan &b = p.block;
#define FP6_BLOCK_CASE(C_)                                                                                         \
    if (b.cfg == C_)                                                                                               \
        return launch_block_cfg<Src, C_>(b, weights, scales, X, Y, M, N, K, partials, counters, epi, stream);
        if constexpr (weights_of<Src>() != Weights::kGrouped) {
            FP6_BLOCK_CASE(0)
        }
        FP6_BLOCK_CASE(2)
        if constexpr (!per_row(weights_of<Src>())) {
            FP6_BLOCK_CASE(1)
        }
        if constexpr (weights_of<Src>() == Weights::kFp16) {
            FP6_BLOCK_CASE(3)
        }
#undef FP6_BLOCK_CASE
        return FP6_ERR_SHAPE;  // not reached: plan_prompt only picks the blocks above
    }
    const TileShape &t = p.tiled.tile;
#define FP6_TILED_CASE(RT_, NT_, WM_, WN_, WK_)                                                                        \
    if (t.rt == RT_ && t.nt == NT_ && t.wm == WM_ && t.wn == WN_ && p.tiled.k_groups == WK_)                                      \
        return launch_tiled_cfg<Src, RT_, NT_, WM_, WN_, WK_>(p.tiled, weights, scales, X, Y, M, N, K, partials, counters, epi, \
                                                         stream);
    if constexpr (weights_of<Src>() != Weights::kFp16) {
        if constexpr (weights_of<Src>() != Weights::kFp6) {
            FP6_TILED_CASE(2, 4, 4, 1, 2)
        }
        FP6_TILED_CASE(2, 4, 4, 1, 1)
        FP6_TILED_CASE(2, 4, 4, 2, 1)
    }
    if constexpr (per_row(weights_of<Src>())) {
        FP6_TILED_CASE(2, 4, 8, 1, 1)
        FP6_TILED_CASE(2, 8, 8, 1, 1)
    }
#undef FP6_TILED_CASE
    return FP6_ERR_SHAPE;  // not reached: plan_prompt only picks the shapes above
}

template <class Src>
fp6_status launch_prompt(const void *weights, const void *scales, const void *X, void *Y, int64_t M, int64_t N,
                        int64_t K, const WorkspaceRef &workspace, const Epilogue &epi, hipStream_t stream)
{
    const int64_t chunk = prompt_chunk_tokens(K);
    if (chunk <= 0)
        return FP6_ERR_SHAPE;  // one token's activations exceed a 32-bit byte offset
    // every chunk's plan must fit before anything is launched
    for (int64_t n : prompt_chunks(N, K)) {
        if (n <= 0)
            continue;
        PromptPlan p;
        SplitBuffers unused;
        const fp6_status fits = plan_prompt_within(M, n, K, weights_of<Src>(), workspace, p, unused);
        if (fits != FP6_OK)
            return fits;
    }
    const int64_t Mout = epi.gated ? M / 2 : M;
    for (int64_t n0 = 0; n0 < N; n0 += chunk) {
        // a short last chunk still goes through this kernel (it handles any token count)
        const int64_t n = N - n0 < chunk ? N - n0 : chunk;
        Epilogue e = epi;
        if (e.residual)
            e.residual += n0 * Mout;
        const fp6_status st = launch_prompt_chunk<Src>(weights, scales, static_cast<const half_t *>(X) + n0 * K,
                                                      static_cast<half_t *>(Y) + n0 * Mout, M, n, K, workspace, e,
                                                      stream);
        if (st != FP6_OK)
            return st;
    }
    return FP6_OK;
}

template <class Src, int C>
fp6_status launch_stream_cfg(const StreamPlan &p, const void *weights, const void *scales, const void *X, void *Y,
                             int64_t M, int64_t N, int64_t K, float4_t *partials, int *counters, const Epilogue &epi,
                             hipStream_t stream)
{
    typedef typename StreamShapeOf<Src::kPackedConfigs, C>::type Shape;
    constexpr StreamCfg c = StreamShapeOf<Src::kPackedConfigs, C>::c;
    static_assert(Shape::template lds_bytes<Src>() == stream_lds_bytes(c, Src::kTileCols, Src::kLdsTileBytes), "the plan's LDS");
    auto kernel = linear_stream_kernel<Src, Shape>;
    constexpr size_t lds = Shape::template lds_bytes<Src>();
    static_assert(lds <= 160 * 1024, "activation stages and staged weight tiles exceed the LDS of a CU");
    static std::atomic<uint64_t> lds_done{0};  // per instantiation
    if (!allow_dynamic_lds(reinterpret_cast<const void *>(kernel), lds, lds_done))
        return FP6_ERR_HIP;
    const dim3 grid((unsigned)p.row_blocks, (unsigned)p.split), block(Shape::kThreads);  // x runs fastest: row blocks of one k slice
    hipLaunchKernelGGL(kernel, grid, block, lds, stream, weights, static_cast<const half_t *>(scales), static_cast<const half_t *>(X),
                       static_cast<half_t *>(Y), (int)M, (int)N, (int)K, p.split,
                       (int)((K + Src::kTileCols - 1) / Src::kTileCols / p.split), partials, counters, epi);
    return hipGetLastError() == hipSuccess ? FP6_OK : FP6_ERR_HIP;
}

template <class Src, int C = 0>
fp6_status launch_stream_plan(const StreamPlan &p, const void *weights, const void *scales, const void *X, void *Y, int64_t M,
                              int64_t N, int64_t K, float4_t *partials, int *counters, const Epilogue &epi, hipStream_t stream)
{
    if constexpr (C < (Src::kPackedConfigs ? kStreamCfgs : kStreamCfgsFp16)) {
        if constexpr (stream_cfg_built(StreamShapeOf<Src::kPackedConfigs, C>::c, stream_weights_of<Src>()))
            if (p.cfg == C)
                return launch_stream_cfg<Src, C>(p, weights, scales, X, Y, M, N, K, partials, counters, epi, stream);
        return launch_stream_plan<Src, C + 1>(p, weights, scales, X, Y, M, N, K, partials, counters, epi, stream);
    }
    return FP6_ERR_SHAPE;  // not reached: plan_stream only picks the configurations above
}

template <class Src>  // the source of a format, as the entry points name it
fp6_status launch_stream(const void *weights, const void *scales, const void *X, void *Y, int64_t M, int64_t N,
                         int64_t K, const WorkspaceRef &workspace, const Epilogue &epi, hipStream_t stream)
{
    const StreamPlan p = plan_stream(M, N, K, stream_weights_of<Src>());
    SplitBuffers buf;
    const fp6_status fits = stream_buffers(p, workspace, buf);
    if (fits != FP6_OK)
        return fits;
    return launch_stream_plan<typename Src::StreamSource>(p, weights, scales, X, Y, M, N, K,
                                                          reinterpret_cast<float4_t *>(buf.partials), buf.counters, epi, stream);
}

std::atomic<int> g_pack_polls{kPartWaitPolls};  // (tuning hook)

int64_t pack_parts(int64_t K) { return (K / kTileK + kPartWaves - 1) / kPartWaves; }

// Whether a matrix is quantized in one pass (time over that of two launches, 6 / 4 / 3 bits):
//   1024 columns and less, no exchange: 0.57-0.62 / 0.61-0.64 / 0.65-0.70 from 1024 to 57344 rows;
//   more, 6, 5 and 4 bits: 8192 x 2048 0.94 / 0.94, 2048 x 8192 0.93 / 0.94, 4096 x 4096 0.92 / 0.90, 8192 x 22016 0.77 / 0.79,
//     57344 x 8192 0.63 / 0.64; but 3072 x 4096 0.95 / 1.00, 4096 x 2048 1.09 / 1.08, 1024 x 2048 1.16 / 1.16, and where the last
//     part is mostly idle 16384 x 1280 1.11 / 1.10 (57344 x 1280 0.89 / 0.93);
//   many parts wait for one another longer: 8192 x 33024 (33) 0.81 / 0.80, 4096 x 65536 (64) 1.14 / 1.13;
//   3 bits, which the chip has no conversion for (a block computes while nothing of it is in flight): 8192 x 22016 1.05, 57344 x
//     8192 0.87.
template <class Fmt>
bool one_pass_pack(int64_t M, int64_t K)
{
    const int64_t KT = K / kTileK, parts = pack_parts(K);
    if (parts == 1)
        return true;
    if (std::is_same_v<Fmt, E2M0Format>)
        return parts <= 16 && M * K >= 1 << 28;
    const bool full = 4 * KT >= 3 * kPartWaves * parts;
    return parts <= kMaxParts && M * K >= (full ? 1 << 24 : 1 << 26);
}

// LDS that a block of the second of two launches is given, and does not use, so that few enough of them share a CU.  A wave's weights lie in
// sixteen rows, and with all the waves that the registers hold (20 to 32 per CU) a large matrix is read out of order: time over that of the
// kernel which held 16, by weights, without -> with 12 waves (3 bits 16):
//   6 bits 1024 x 65536 0.97 -> 0.94, 4096 x 65536 1.01 -> 0.98, 16384 x 57344 1.01 -> 0.98 (744 us); 5 bits 0.97 -> 0.96, 1.005 -> 0.995,
//   1.02 -> 1.00; 4 bits 0.97 -> 0.95, 1.01 -> 0.98, 1.01 -> 0.99; 3 bits 0.99 -> 0.965, 1.02 -> 1.00, 1.01 -> 0.99, 8192 x 22016 0.99 -> 0.98.
// Smaller ones lose by it: 32768 x 1280 0.87 -> 0.90, 0.87 -> 0.92, 0.86 -> 0.90, 0.92 -> 0.945.
template <class Fmt>
unsigned tiles_lds(int64_t M, int64_t K)
{
    return M * K < 1 << 26 ? 0 : std::is_same_v<Fmt, E2M0Format> ? kMaxLds / 4 : (kMaxLds / 3) & ~1023;
}

template <class Fmt>
fp6_status quantize_pack_impl(const void *W_f16, int64_t M, int64_t K, void *packed, void *scales_f16, void *stream)
{
    if (!W_f16 || !packed || !scales_f16)
        return FP6_ERR_NULL;
    if (!packed_shape_ok(M, K))
        return FP6_ERR_SHAPE;
    if (!aligned16(W_f16) || !aligned16(packed) || !aligned16(scales_f16))
        return FP6_ERR_ALIGN;
    const hipStream_t st = static_cast<hipStream_t>(stream);
    const half_t *W = static_cast<const half_t *>(W_f16);
    uint8_t *out = static_cast<uint8_t *>(packed);
    half_t *scales = static_cast<half_t *>(scales_f16);
    const int64_t RT = M / kTileRows, KT = K / kTileK, parts = pack_parts(K);
    if (one_pass_pack<Fmt>(M, K)) {
        if (parts > 1) {
            hipLaunchKernelGGL(clear_exchange_kernel, dim3((unsigned)((RT * (kExchangeBytes / 16) + 255) / 256)), dim3(256), 0, st, out, (int)RT,
                               Fmt::kTileBytes);
            if (hipGetLastError() != hipSuccess)
                return FP6_ERR_HIP;
        }
        hipLaunchKernelGGL(quantize_rows_kernel<Fmt>, dim3((unsigned)(RT * parts)), dim3(kPartWaves * 64), 0, st, W, (int)M, (int)K, out, scales,
                           (int)parts, g_pack_polls.load(std::memory_order_relaxed));
        return hipGetLastError() == hipSuccess ? FP6_OK : FP6_ERR_HIP;
    }
    hipLaunchKernelGGL(row_scale_kernel<Fmt>, dim3((unsigned)((M + kScaleWavesPerBlock - 1) / kScaleWavesPerBlock)),
                       dim3(kScaleWavesPerBlock * 64), 0, st, W, (int)M, (int)K, scales);
    if (hipGetLastError() != hipSuccess)
        return FP6_ERR_HIP;
    hipLaunchKernelGGL(quantize_tiles_kernel<Fmt>, dim3((unsigned)((RT * KT + 3) / 4)), dim3(256), tiles_lds<Fmt>(M, K), st, W, (int)M, (int)K, out, scales);
    return hipGetLastError() == hipSuccess ? FP6_OK : FP6_ERR_HIP;
}

template <class Src>
fp6_status unpack_impl(const void *packed, const void *scales_f16, int64_t M, int64_t K, void *W_f16_out, void *stream)
{
    if (!packed || !scales_f16 || !W_f16_out)
        return FP6_ERR_NULL;
    if (!packed_shape_ok(M, K))
        return FP6_ERR_SHAPE;
    if (!aligned16(packed) || !aligned16(scales_f16) || !aligned16(W_f16_out))
        return FP6_ERR_ALIGN;
    const int64_t tiles = (M / kTileRows) * (K / kTileK);
    hipLaunchKernelGGL(unpack_kernel<Src>, dim3((unsigned)((tiles + 3) / 4)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), static_cast<const uint8_t *>(packed),
                       static_cast<const half_t *>(scales_f16), (int)M, (int)K, static_cast<half_t *>(W_f16_out));
    return hipGetLastError() == hipSuccess ? FP6_OK : FP6_ERR_HIP;
}

// ---- the library's own split-K buffer (fp6_linear_static) ------------------------------------------
// A file-scope device array: every GPU the library runs on holds its own copy, at its own address, until
// the process ends.  In host code the array's name is only a handle for hipGetSymbolAddress; the device
// address that the kernels and the fill take is looked up once per device and kept.
static __device__ __align__(256) unsigned char scratch[FP6_STATIC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
std::atomic<void *> g_scratch_ptr[kMaxDevices];

fp6_status static_scratch_address(void **out)
{
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kMaxDevices)
        return FP6_ERR_HIP;
    void *ptr = g_scratch_ptr[device].load(std::memory_order_acquire);
    if (!ptr) {
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr)
            return FP6_ERR_HIP;
        g_scratch_ptr[device].store(ptr, std::memory_order_release);  // racing threads store the same address
    }
    *out = ptr;
    return FP6_OK;
}

// Counter bytes that a call of the packed 6-bit layer needs in the static buffer, or FP6_ERR_WORKSPACE when
// the call does not fit it.  Host arithmetic only.
fp6_status static_plan(int64_t M, int64_t N, int64_t K, size_t &counter_bytes)
{
    const WorkspaceRef probe{reinterpret_cast<void *>(uintptr_t(256)), FP6_STATIC_SCRATCH_BYTES, kStaticCounterBytes, true};  // never dereferenced
    SplitBuffers unused;
    counter_bytes = 0;
    if (N <= kStreamMaxN) {
        const StreamPlan p = plan_stream(M, N, K, stream_weights_of<PackedFp6Source>());
        counter_bytes = p.counter_bytes;
        return probe.view(p.counter_bytes, p.partial_bytes, unused);
    }
    for (int64_t n : prompt_chunks(N, K)) {
        if (n <= 0)
            continue;
        const PromptPlan p = plan_prompt(M, n, K, Weights::kFp6);
        if (p.required_counters() > counter_bytes)
            counter_bytes = p.required_counters();
        const fp6_status fits = probe.view(p.required_counters(), p.required_partials(), unused);
        if (fits != FP6_OK)
            return fits;
    }
    return FP6_OK;
}

template <class Src>
fp6_status packed_linear_impl(const void *packed, const void *scales_f16, const void *X_f16, void *Y_f16, int64_t M,
                              int64_t N, int64_t K, void *workspace, size_t workspace_bytes, void *stream,
                              const Epilogue &epi = Epilogue{nullptr, nullptr, 0}, bool static_buffer = false)
{
    if (!packed || !scales_f16 || !X_f16 || !Y_f16)
        return FP6_ERR_NULL;
    if (!packed_shape_ok(M, K) || N <= 0 || N >= (1ll << 31))
        return FP6_ERR_SHAPE;
    if (!aligned16(packed) || !aligned16(scales_f16) || !aligned16(X_f16) || !aligned16(Y_f16) || !aligned16(epi.bias)
        || !aligned16(epi.residual))
        return FP6_ERR_ALIGN;
    const WorkspaceRef ws{workspace, workspace_bytes, static_buffer ? kStaticCounterBytes : counter_region_bytes(M, N, K), static_buffer};
    if (N > kStreamMaxN)
        return launch_prompt<Src>(packed, scales_f16, X_f16, Y_f16, M, N, K, ws, epi, static_cast<hipStream_t>(stream));
    return launch_stream<Src>(packed, scales_f16, X_f16, Y_f16, M, N, K, ws, epi, static_cast<hipStream_t>(stream));
}

// What fp6_tuning_plan reports, and what the queries beside it do.
struct PlanDetails {
    int k_groups;                    // groups of k-tiles of a workgroup
    size_t used_partials, required_partials;  // that the launch writes; that its caller has to bring
};
fp6_status plan_of_call(int weight_bits, int64_t M, int64_t N, int64_t K, int64_t token, size_t workspace_bytes, fp6_launch_plan &plan,
                        PlanDetails &details)
{
    const bool fp16 = weight_bits == 16, grouped = weight_bits == -6;
    if (!(fp16 ? shape_ok(M, K) : packed_shape_ok(M, K)) || token < 0 || token >= N || N >= (1ll << 31)
        || !(fp16 || grouped || (weight_bits >= 3 && weight_bits <= 6)))
        return FP6_ERR_SHAPE;
    const size_t region = counter_region_bytes(M, N, K);
    const WorkspaceRef ws{reinterpret_cast<void *>(uintptr_t(256)), workspace_bytes, region};  // never dereferenced
    SplitBuffers unused;
    if (N <= kStreamMaxN) {
        const StreamWeights w = fp16               ? stream_weights_of<PlainFp16Source>()
                                : weight_bits == 3 ? stream_weights_of<PackedFp3Source>()
                                : weight_bits == 4 ? stream_weights_of<PackedFp4Source>()
                                : weight_bits == 5 ? stream_weights_of<PackedFp5Source>()
                                : grouped          ? stream_weights_of<PackedFp6GroupSource>() : stream_weights_of<PackedFp6Source>();
        const StreamPlan p = plan_stream(M, N, K, w);
        const fp6_status fits = stream_buffers(p, ws, unused);
        if (fits != FP6_OK)
            return fits;
        const StreamCfg &c = (fp16 ? kStreamCfgFp16 : kStreamCfg)[p.cfg];
        plan = {FP6_KERNEL_STREAM, kTileRows * c.wm, 16 * c.nt, p.split, 0, N, p.counter_bytes, region, p.partial_bytes};
        details = {c.wk, p.partial_bytes, p.required_partials};
        return FP6_OK;
    }
    const Weights kind = fp16               ? Weights::kFp16
                         : grouped          ? Weights::kGrouped
                         : weight_bits == 3 ? Weights::kFp3
                         : weight_bits == 4 ? Weights::kFp4 : weight_bits == 5 ? Weights::kFp5 : Weights::kFp6;
    const int64_t chunk = prompt_chunk_tokens(K), first = token / chunk * chunk, tokens = N - first < chunk ? N - first : chunk;
    PromptPlan p;
    const fp6_status fits = plan_prompt_within(M, tokens, K, kind, ws, p, unused);
    if (fits != FP6_OK)
        return fits;
    plan = {p.is_block() ? FP6_KERNEL_BLOCK : FP6_KERNEL_TILED, p.is_block() ? kBlockCfg[p.block.cfg].rows : p.tiled.tile.rows(),
            p.is_block() ? kBlockCfg[p.block.cfg].tokens : p.tiled.tile.tokens(), p.split(), first, tokens, p.counter_bytes(),
            region, p.split() > 1 ? p.required_partials() : 0};
    details = {p.is_block() ? kBlockCfg[p.block.cfg].k_groups() : p.tiled.k_groups, p.partial_bytes(), p.required_partials()};
    return FP6_OK;
}

}  // namespace

extern "C" {

const char *fp6_status_str(int status)
{
    switch (status) {
    case FP6_OK: return "FP6_OK";
    case FP6_ERR_NULL: return "FP6_ERR_NULL: a required pointer is NULL";
    case FP6_ERR_SHAPE: return "FP6_ERR_SHAPE: need M % 16 == 0, K % 256 == 0, M, N, K > 0";
    case FP6_ERR_WORKSPACE: return "FP6_ERR_WORKSPACE: workspace missing or too small";
    case FP6_ERR_ALIGN: return "FP6_ERR_ALIGN: pointers must be 16-byte aligned";
    case FP6_ERR_HIP: return "FP6_ERR_HIP: kernel launch failed";
    default: return "unknown fp6 status";
    }
}

int fp6_layout_version(void) { return kLayoutVersion; }

size_t fp6_packed_bytes(int64_t M, int64_t K) { return packed_shape_ok(M, K) ? (size_t)(M * K / 4 * 3) : 0; }

size_t fp6_linear_workspace_bytes(int64_t M, int64_t N, int64_t K)
{
    if (!packed_shape_ok(M, K) || N <= 0)
        return 0;
    if (N <= kStreamMaxN)
        // fp5, fp4 and fp6g ask here too
        return stream_workspace_bytes(M, N, K, {stream_weights_of<PackedFp6Source>(), stream_weights_of<PackedFp6GroupSource>(),
                                                stream_weights_of<PackedFp5Source>(), stream_weights_of<PackedFp4Source>()});
    // fp6g_linear asks here too (fp5 and fp4 have the partial sums of fp6)
    const size_t bytes = prompt_workspace_bytes(M, N, K, Weights::kFp6), grouped = prompt_workspace_bytes(M, N, K, Weights::kGrouped);
    return bytes > grouped ? bytes : grouped;
}

size_t fp16_linear_workspace_bytes(int64_t M, int64_t N, int64_t K)
{
    if (!shape_ok(M, K) || N <= 0)
        return 0;
    return N <= kStreamMaxN ? stream_workspace_bytes(M, N, K, {stream_weights_of<PlainFp16Source>()})
                            : prompt_workspace_bytes(M, N, K, Weights::kFp16);
}

size_t fp6_workspace_zero_bytes(int64_t M, int64_t N, int64_t K)
{
    return shape_ok(M, K) && N > 0 ? counter_region_bytes(M, N, K) : 0;
}

void fp6_tuning_set_split_k(int split_k) { g_forced_split.store(split_k < 0 ? 0 : split_k); }

void fp6_tuning_set_tile(int block_rows, int block_tokens)
{
    const bool known = ((block_rows == 128 || block_rows == 256) && (block_tokens == 64 || block_tokens == 128))
                       || (block_rows == 256 && block_tokens == 256);
    g_forced_tile.store(known ? block_rows * 1024 + block_tokens : 0);
}

fp6_status fp6_tuning_plan(int weight_bits, int64_t M, int64_t N, int64_t K, int64_t token, size_t workspace_bytes,
                           fp6_launch_plan *plan)
{
    PlanDetails details;
    return plan ? plan_of_call(weight_bits, M, N, K, token, workspace_bytes, *plan, details) : FP6_ERR_NULL;
}

int fp6_tuning_plan_k_groups(int weight_bits, int64_t M, int64_t N, int64_t K, int64_t token, size_t workspace_bytes)
{
    fp6_launch_plan plan;
    PlanDetails details;
    return plan_of_call(weight_bits, M, N, K, token, workspace_bytes, plan, details) == FP6_OK ? details.k_groups : 0;
}

fp6_status fp6_tuning_plan_partials(int weight_bits, int64_t M, int64_t N, int64_t K, int64_t token, size_t workspace_bytes, size_t *used,
                                    size_t *required)
{
    if (!used || !required)
        return FP6_ERR_NULL;
    fp6_launch_plan plan;
    PlanDetails details;
    const fp6_status status = plan_of_call(weight_bits, M, N, K, token, workspace_bytes, plan, details);
    if (status == FP6_OK) {
        *used = details.used_partials;
        *required = details.required_partials;
    }
    return status;
}

void fp6_tuning_set_pack_polls(int polls) { g_pack_polls.store(polls < 0 ? kPartWaitPolls : polls); }

int fp6_tuning_pack_parts(int weight_bits, int64_t M, int64_t K)
{
    if (!packed_shape_ok(M, K) || weight_bits < 3 || weight_bits > 6)
        return -1;
    const bool one_pass = weight_bits == 6   ? one_pass_pack<E3M2Format>(M, K)
                          : weight_bits == 5 ? one_pass_pack<E2M2Format>(M, K)
                          : weight_bits == 4 ? one_pass_pack<E2M1Format>(M, K) : one_pass_pack<E2M0Format>(M, K);
    return one_pass ? (int)pack_parts(K) : 0;
}

fp6_status fp6_workspace_init(void *workspace, size_t workspace_bytes, void *stream)
{
    if (workspace_bytes == 0)
        return FP6_OK;
    if (!workspace)
        return FP6_ERR_NULL;
    if (!aligned16(workspace) || workspace_bytes % 16)
        return FP6_ERR_ALIGN;
    const size_t n16 = workspace_bytes / 16;
    hipLaunchKernelGGL(zero_fill_kernel, dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), static_cast<u32x4 *>(workspace), n16);
    return hipGetLastError() == hipSuccess ? FP6_OK : FP6_ERR_HIP;
}

fp6_status fp6_quantize_pack(const void *W_f16, int64_t M, int64_t K, void *packed, void *scales_f16, void *stream)
{
    return quantize_pack_impl<E3M2Format>(W_f16, M, K, packed, scales_f16, stream);
}

fp6_status fp6_unpack(const void *packed, const void *scales_f16, int64_t M, int64_t K, void *W_f16_out, void *stream)
{
    return unpack_impl<PackedFp6Source>(packed, scales_f16, M, K, W_f16_out, stream);
}

fp6_status fp6_linear(const void *packed, const void *scales_f16, const void *X_f16, void *Y_f16, int64_t M, int64_t N,
                      int64_t K, void *workspace, size_t workspace_bytes, void *stream)
{
    return packed_linear_impl<PackedFp6Source>(packed, scales_f16, X_f16, Y_f16, M, N, K, workspace, workspace_bytes,
                                               stream);
}

fp6_status fp6_linear_static(const void *packed, const void *scales_f16, const void *X_f16, void *Y_f16, int64_t M,
                             int64_t N, int64_t K, void *stream)
{
    if (!packed || !scales_f16 || !X_f16 || !Y_f16)
        return FP6_ERR_NULL;
    if (!packed_shape_ok(M, K) || N <= 0 || N >= (1ll << 31))
        return FP6_ERR_SHAPE;
    if (!aligned16(packed) || !aligned16(scales_f16) || !aligned16(X_f16) || !aligned16(Y_f16))
        return FP6_ERR_ALIGN;
    size_t counter_bytes = 0;
    const fp6_status fits = static_plan(M, N, K, counter_bytes);  // before the device is touched
    if (fits != FP6_OK)
        return fits;
    void *buffer = nullptr;
    if (counter_bytes > 0) {
        const fp6_status found = static_scratch_address(&buffer);
        if (found != FP6_OK)
            return found;
        // the array keeps what the last call left: the arrival counters must start at zero (a fill kernel,
        // not a memset node, so that the call can be captured into a graph)
        const size_t n16 = counter_bytes / 16;
        hipLaunchKernelGGL(zero_fill_kernel, dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0,
                           static_cast<hipStream_t>(stream), static_cast<u32x4 *>(buffer), n16);
        if (hipGetLastError() != hipSuccess)
            return FP6_ERR_HIP;
    }
    return packed_linear_impl<PackedFp6Source>(packed, scales_f16, X_f16, Y_f16, M, N, K, buffer,
                                               buffer ? (size_t)FP6_STATIC_SCRATCH_BYTES : 0, stream,
                                               Epilogue{nullptr, nullptr, 0}, true);
}

fp6_status fp6_linear_fused(const void *packed, const void *scales_f16, const void *X_f16, void *Y_f16, int64_t M,
                            int64_t N, int64_t K, const void *bias_f16, const void *residual_f16, int gated,
                            void *workspace, size_t workspace_bytes, void *stream)
{
    const Epilogue epi{static_cast<const half_t *>(bias_f16), static_cast<const half_t *>(residual_f16), gated ? 1 : 0};
    return packed_linear_impl<PackedFp6Source>(packed, scales_f16, X_f16, Y_f16, M, N, K, workspace, workspace_bytes,
                                               stream, epi);
}

fp6_status fp6g_quantize_pack(const void *W_f16, int64_t M, int64_t K, int64_t group, void *packed, void *scales_f16,
                              void *stream)
{
    if (!W_f16 || !packed || !scales_f16)
        return FP6_ERR_NULL;
    if (!packed_shape_ok(M, K) || group != kGroupColumns)
        return FP6_ERR_SHAPE;
    if (!aligned16(W_f16) || !aligned16(packed) || !aligned16(scales_f16))
        return FP6_ERR_ALIGN;
    const int64_t tiles = (M / kTileRows) * (K / kTileK);
    hipLaunchKernelGGL(quantize_pack_group_kernel, dim3((unsigned)((tiles + 3) / 4)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), static_cast<const half_t *>(W_f16), (int)M, (int)K,
                       static_cast<uint8_t *>(packed), static_cast<half_t *>(scales_f16));
    return hipGetLastError() == hipSuccess ? FP6_OK : FP6_ERR_HIP;
}

fp6_status fp6g_unpack(const void *packed, const void *scales_f16, int64_t M, int64_t K, int64_t group, void *W_f16_out,
                       void *stream)
{
    if (group != kGroupColumns)
        return FP6_ERR_SHAPE;
    return unpack_impl<PackedFp6GroupSource>(packed, scales_f16, M, K, W_f16_out, stream);
}

fp6_status fp6g_linear(const void *packed, const void *scales_f16, const void *X_f16, void *Y_f16, int64_t M, int64_t N,
                       int64_t K, int64_t group, void *workspace, size_t workspace_bytes, void *stream)
{
    if (group != kGroupColumns)
        return FP6_ERR_SHAPE;
    return packed_linear_impl<PackedFp6GroupSource>(packed, scales_f16, X_f16, Y_f16, M, N, K, workspace,
                                                    workspace_bytes, stream);
}

size_t fp5_packed_bytes(int64_t M, int64_t K) { return packed_shape_ok(M, K) ? (size_t)(M * K / 8 * 5) : 0; }

size_t fp5_linear_workspace_bytes(int64_t M, int64_t N, int64_t K) { return fp6_linear_workspace_bytes(M, N, K); }

fp6_status fp5_quantize_pack(const void *W_f16, int64_t M, int64_t K, void *packed, void *scales_f16, void *stream)
{
    return quantize_pack_impl<E2M2Format>(W_f16, M, K, packed, scales_f16, stream);
}

fp6_status fp5_unpack(const void *packed, const void *scales_f16, int64_t M, int64_t K, void *W_f16_out, void *stream)
{
    return unpack_impl<PackedFp5Source>(packed, scales_f16, M, K, W_f16_out, stream);
}

fp6_status fp5_linear(const void *packed, const void *scales_f16, const void *X_f16, void *Y_f16, int64_t M, int64_t N,
                      int64_t K, void *workspace, size_t workspace_bytes, void *stream)
{
    return packed_linear_impl<PackedFp5Source>(packed, scales_f16, X_f16, Y_f16, M, N, K, workspace, workspace_bytes,
                                               stream);
}

size_t fp4_packed_bytes(int64_t M, int64_t K) { return packed_shape_ok(M, K) ? (size_t)(M * K / 2) : 0; }

size_t fp4_linear_workspace_bytes(int64_t M, int64_t N, int64_t K) { return fp6_linear_workspace_bytes(M, N, K); }

fp6_status fp4_quantize_pack(const void *W_f16, int64_t M, int64_t K, void *packed, void *scales_f16, void *stream)
{
    return quantize_pack_impl<E2M1Format>(W_f16, M, K, packed, scales_f16, stream);
}

fp6_status fp4_unpack(const void *packed, const void *scales_f16, int64_t M, int64_t K, void *W_f16_out, void *stream)
{
    return unpack_impl<PackedFp4Source>(packed, scales_f16, M, K, W_f16_out, stream);
}

fp6_status fp4_linear(const void *packed, const void *scales_f16, const void *X_f16, void *Y_f16, int64_t M, int64_t N,
                      int64_t K, void *workspace, size_t workspace_bytes, void *stream)
{
    return packed_linear_impl<PackedFp4Source>(packed, scales_f16, X_f16, Y_f16, M, N, K, workspace, workspace_bytes,
                                               stream);
}

// tiles of 16 x 512 codes: a K that is an odd multiple of 256 pads its last tile
size_t fp3_packed_bytes(int64_t M, int64_t K)
{
    return packed_shape_ok(M, K) ? (size_t)((K + 511) / 512 * (M / kTileRows) * kTileBytes3) : 0;
}

size_t fp3_linear_workspace_bytes(int64_t M, int64_t N, int64_t K)
{
    if (!packed_shape_ok(M, K) || N <= 0)
        return 0;
    return N <= kStreamMaxN ? stream_workspace_bytes(M, N, K, {stream_weights_of<PackedFp3Source>()})
                            : prompt_workspace_bytes(M, N, K, Weights::kFp3);
}

fp6_status fp3_quantize_pack(const void *W_f16, int64_t M, int64_t K, void *packed, void *scales_f16, void *stream)
{
    return quantize_pack_impl<E2M0Format>(W_f16, M, K, packed, scales_f16, stream);
}

fp6_status fp3_unpack(const void *packed, const void *scales_f16, int64_t M, int64_t K, void *W_f16_out, void *stream)
{
    return unpack_impl<PackedFp3Source>(packed, scales_f16, M, K, W_f16_out, stream);
}

fp6_status fp3_linear(const void *packed, const void *scales_f16, const void *X_f16, void *Y_f16, int64_t M, int64_t N,
                      int64_t K, void *workspace, size_t workspace_bytes, void *stream)
{
    return packed_linear_impl<PackedFp3Source>(packed, scales_f16, X_f16, Y_f16, M, N, K, workspace, workspace_bytes,
                                               stream);
}

#define FP6_FUSED_ENTRY(NAME, SRC)                                                                                     \
    fp6_status NAME(const void *packed, const void *scales_f16, const void *X_f16, void *Y_f16, int64_t M, int64_t N, \
                    int64_t K, const void *bias_f16, const void *residual_f16, int gated, void *workspace,             \
                    size_t workspace_bytes, void *stream)                                                              \
    {                                                                                                                  \
        const Epilogue epi{static_cast<const half_t *>(bias_f16), static_cast<const half_t *>(residual_f16),         \
                           gated ? 1 : 0};                                                                             \
        return packed_linear_impl<SRC>(packed, scales_f16, X_f16, Y_f16, M, N, K, workspace, workspace_bytes, stream,  \
                                       epi);                                                                           \
    }
FP6_FUSED_ENTRY(fp5_linear_fused, PackedFp5Source)
FP6_FUSED_ENTRY(fp4_linear_fused, PackedFp4Source)
FP6_FUSED_ENTRY(fp3_linear_fused, PackedFp3Source)
#undef FP6_FUSED_ENTRY

fp6_status fp6g_linear_fused(const void *packed, const void *scales_f16, const void *X_f16, void *Y_f16, int64_t M,
                             int64_t N, int64_t K, int64_t group, const void *bias_f16, const void *residual_f16,
                             int gated, void *workspace, size_t workspace_bytes, void *stream)
{
    if (group != kGroupColumns)
        return FP6_ERR_SHAPE;
    const Epilogue epi{static_cast<const half_t *>(bias_f16), static_cast<const half_t *>(residual_f16), gated ? 1 : 0};
    return packed_linear_impl<PackedFp6GroupSource>(packed, scales_f16, X_f16, Y_f16, M, N, K, workspace,
                                                    workspace_bytes, stream, epi);
}

fp6_status fp6_probe_read(const void *buffer, size_t bytes, void *sink, void *stream)
{
    if (!buffer || !sink)
        return FP6_ERR_NULL;
    if (!aligned16(buffer))
        return FP6_ERR_ALIGN;
    // 1024 waves (four per CU), each at least one double step of 2 x 8 KB
    const unsigned blocks = kCus;
    if (bytes < (size_t)blocks * 4 * 16384)
        return FP6_ERR_SHAPE;
    hipLaunchKernelGGL(probe_read_kernel, dim3(blocks), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<const uint8_t *>(buffer), bytes, static_cast<uint32_t *>(sink));
    return hipGetLastError() == hipSuccess ? FP6_OK : FP6_ERR_HIP;
}

size_t fp6_probe_read_bytes(size_t bytes) { return bytes / (kCus * 4) / 16384 * 16384 * (kCus * 4); }

size_t fp6_probe_mfma_sink_bytes(void) { return (size_t)kCus * 4 * 256 * sizeof(float); }

fp6_status fp6_probe_mfma(int64_t iters, void *sink, void *stream)
{
    if (!sink)
        return FP6_ERR_NULL;
    if (iters <= 0 || iters >= (1ll << 31))
        return FP6_ERR_SHAPE;
    // four blocks of four waves per CU: four waves per SIMD
    hipLaunchKernelGGL(probe_mfma_kernel, dim3(kCus * 4), dim3(256), 0, static_cast<hipStream_t>(stream), (int)iters,
                       static_cast<float *>(sink));
    return hipGetLastError() == hipSuccess ? FP6_OK : FP6_ERR_HIP;
}

fp6_status fp16_linear(const void *W_f16, const void *X_f16, void *Y_f16, int64_t M, int64_t N, int64_t K,
                       void *workspace, size_t workspace_bytes, void *stream)
{
    if (!W_f16 || !X_f16 || !Y_f16)
        return FP6_ERR_NULL;
    if (!shape_ok(M, K) || N <= 0 || N >= (1ll << 31))
        return FP6_ERR_SHAPE;
    if (!aligned16(W_f16) || !aligned16(X_f16) || !aligned16(Y_f16))
        return FP6_ERR_ALIGN;
    const WorkspaceRef ws{workspace, workspace_bytes, counter_region_bytes(M, N, K)};
    if (N > kStreamMaxN)
        return launch_prompt<PlainFp16Source>(W_f16, nullptr, X_f16, Y_f16, M, N, K, ws, Epilogue{nullptr, nullptr, 0},
                                             static_cast<hipStream_t>(stream));
    return launch_stream<PlainFp16Source>(W_f16, nullptr, X_f16, Y_f16, M, N, K, ws, Epilogue{nullptr, nullptr, 0},
                                          static_cast<hipStream_t>(stream));
}

}  // extern "C"
