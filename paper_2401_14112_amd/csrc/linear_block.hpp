// Block-tiled linear-layer kernel for prompt-sized token counts: fp16 weights, weights with group scales, and of those with a
// scale per row the products that fill the chip with 256 x 256 blocks or that 128 x 128 blocks suit better than the tiled
// kernel's (linear_tiled.hpp: the others).
//
// A block of WM x WN x WK waves computes a BM x BN piece of Y (BM = 16*RT*WM rows, BN = 16*NT*WN tokens); wave
// (wm, wn) owns RT x NT tiles of 16 rows x 16 tokens in fp32 accumulators of v_mfma_f32_16x16x32_f16.  With WK = 2
// two waves share such a piece: one takes the first four runs of 32 columns of every k-tile, the other the last four,
// and their sums meet in LDS at the end (twice the waves per output tile without smaller wave tiles).
//
// What bounds it, measured: with every CU busy the chip is limited by power, not by issue slots.  A loop of nothing but
// matrix instructions on random fp16 activations and e3m2 weights in registers reaches 2060-2130 TFLOP/s with the
// 16 x 16 x 32 form (1700 with 32 x 32 x 16: hence the former); one 128-bit LDS read per four of them costs 7 %, one
// per two 25 %; under the 256 x 256 block the engine runs at 1.87 GHz with the matrix pipes 0.70 busy (57344 x 8192,
// N = 4096, 6 bits).  So a wave tile is tall (RT = 4: an activation fragment read from LDS serves four matrix
// instructions) and the block is as large as the accumulators allow (fewer copies from L2 per product).  The 6-bit
// conversion occupies the SIMD for 65 clk and is paid once per row tile and token half: 1/NT of the matrix time.
// Measured, before this kernel and with it, in one process each: 57344 x 8192, N = 4096, 6 bits 3186 -> 2764 us = 1392
// TFLOP/s; 9216 x 9216, N = 256, fp16 155 -> 64 us (weights in the last-level cache); 28672 x 8192, N = 201, group scales
// 160 -> 107 us.  Where a stage is one run per k group, both operands of fp16 weights, and the activations of every format, are
// copied in pieces of 64 bytes per row, so each 128-byte line is requested twice (fp16, 8192 x 22016, N = 512, 256 x 256: 23.4 M
// requests from the L1 for 1.44 GB of copies, the waves waiting 0.54 of their cycles and the matrix pipes 0.39 busy).  Where it
// is a pair of neighbouring runs they are copied in whole lines: fp16, 128 x 128 blocks, 4096 x 8192, N = 1024 80.3 -> 60.3 us, 8192 x
// 8192, N = 128 45.6 -> 40.5; 128 x 64, 1536 x 4864, N = 241 16.6 -> 13.4; group scales, 256 x 128 with four stages instead of
// five, 8192 x 22016, N = 512 179.1 -> 175.1.  It takes rings of four stages: with three, which is what the LDS holds of 256 x 128
// fp16 blocks, each wait is for the copies just requested (82.9 -> 83.9 on 9216 x 9216, N = 256; 128 x 128 with three 83).
// Tried and not kept: four more waves that only copy (two for activations, two for weights, each with a counter of its
// own): -7 to +5 %; four waves of 128 x 64 (one per SIMD): equal; ring depths of 4 to 8 stages: within 3 %; the last
// step as loops over tiles staged in LDS (a fifth of the code): 1-2 us slower per launch.
#pragma once
#include "fp6_device.hpp"

namespace fp6 {

// ---- weight sources of the block kernel ---------------------------------------------------------
// Packed tiles are copied to LDS as they are; a lane's share of a tile (a "piece") comes back plane by plane.  A source
// says which planes of a piece a pair of runs (2 * pair, 2 * pair + 1) is made from and turns the pieces of two row
// tiles into the fragments of a pair.
struct BlockFp6Source {
    typedef PackedFp6Source::Tile Piece;
    static constexpr bool kRunStaged = false, kHasScale = true, kFused = true, kGroupScales = false, kHalfTiles = false;
    static constexpr int kTileBytes = 3072, kPlanes = 3;
    static constexpr int plane_bytes(int) { return 1024; }  // of a 16-row tile
    static constexpr int planes_of(int pair) { return pair == 0 ? 1 : pair == 1 ? 3 : pair == 2 ? 6 : 4; }  // bit p: plane p
    template <int P>
    __device__ static __forceinline__ void read_plane(Piece &d, const uint8_t *tile, int lane, int)
    {
        const u32x4 v = *reinterpret_cast<const u32x4 *>(tile + lane * 16);
        if (P == 0)
            d.p0 = v;
        else if (P == 1)
            d.p1 = v;
        else
            d.p2 = v;
    }
    // a pair of runs is three words of a piece: one conversion serves the pair for two pieces
    template <int G>
    __device__ static __forceinline__ void fragments(const Piece &a, const Piece &b, half8_t (&fa)[2], half8_t (&fb)[2])
    {
        auto word = [](const Piece &t, int i) { return i < 4 ? t.p0[i] : i < 8 ? t.p1[i - 4] : t.p2[i - 8]; };
        const u32x6 d = {word(a, 3 * G), word(a, 3 * G + 1), word(a, 3 * G + 2), word(b, 3 * G), word(b, 3 * G + 1), word(b, 3 * G + 2)};
        const half32_t h = dequant_stream(d);
        fa[0] = (half8_t){h[0], h[1], h[2], h[3], h[4], h[5], h[6], h[7]};
        fa[1] = (half8_t){h[8], h[9], h[10], h[11], h[12], h[13], h[14], h[15]};
        fb[0] = (half8_t){h[16], h[17], h[18], h[19], h[20], h[21], h[22], h[23]};
        fb[1] = (half8_t){h[24], h[25], h[26], h[27], h[28], h[29], h[30], h[31]};
    }
};

struct BlockFp6GroupSource : BlockFp6Source {
    static constexpr bool kHasScale = false, kGroupScales = true;
};

// the formats whose fragments come from one piece at a time
template <class Src>
struct BlockPieceSource {
    typedef typename Src::Tile Piece;
    static constexpr bool kRunStaged = false, kHasScale = true, kFused = true, kGroupScales = false;
    template <int G>
    __device__ static __forceinline__ void fragments(const Piece &a, const Piece &b, half8_t (&fa)[2], half8_t (&fb)[2])
    {
        Src::template fragments<G>(a, fa[0], fa[1]);
        Src::template fragments<G>(b, fb[0], fb[1]);
    }
};

struct BlockFp5Source : BlockPieceSource<PackedFp5Source> {
    static constexpr bool kHalfTiles = false;
    static constexpr int kTileBytes = 2560, kPlanes = 3;
    static constexpr int plane_bytes(int p) { return p < 2 ? 1024 : 512; }
    static constexpr int planes_of(int pair) { return pair == 0 ? 1 : pair == 1 ? 3 : 6; }
    template <int P>
    __device__ static __forceinline__ void read_plane(Piece &d, const uint8_t *tile, int lane, int)
    {
        if (P == 0)
            d.p0 = *reinterpret_cast<const u32x4 *>(tile + lane * 16);
        else if (P == 1)
            d.p1 = *reinterpret_cast<const u32x4 *>(tile + lane * 16);
        else
            d.p2 = *reinterpret_cast<const u32x2 *>(tile + lane * 8);
    }
};

struct BlockFp4Source : BlockPieceSource<PackedFp4Source> {
    static constexpr bool kHalfTiles = false;
    static constexpr int kTileBytes = 2048, kPlanes = 2;
    static constexpr int plane_bytes(int) { return 1024; }
    static constexpr int planes_of(int pair) { return pair < 2 ? 1 : 2; }
    template <int P>
    __device__ static __forceinline__ void read_plane(Piece &d, const uint8_t *tile, int lane, int)
    {
        (P == 0 ? d.p0 : d.p1) = *reinterpret_cast<const u32x4 *>(tile + lane * 16);
    }
};

// Half a 512-column tile per k-tile: plane 0 (or 2) and the lane's 8 bytes of the middle plane, which is copied whole.
struct BlockFp3Source : BlockPieceSource<PackedFp3Source> {
    static constexpr bool kHalfTiles = true;
    static constexpr int kTileBytes = kTileBytes3, kPlanes = 2;
    static constexpr int plane_bytes(int) { return 1024; }
    static constexpr int planes_of(int pair) { return pair < 2 ? 1 : 3; }
    template <int P>
    __device__ static __forceinline__ void read_plane(Piece &d, const uint8_t *tile, int lane, int half)
    {
        if (P == 0)
            d.p0 = *reinterpret_cast<const u32x4 *>(tile + lane * 16);
        else
            d.p1 = *reinterpret_cast<const u32x2 *>(tile + lane * 16 + half * 8);
    }
};

// Row-major fp16 weights: staged run by run in the layout of the activations (fragments are read as they are).
struct BlockFp16Source {
    struct Piece {};
    static constexpr bool kRunStaged = true, kHasScale = false, kGroupScales = false, kHalfTiles = false;
    static constexpr bool kFused = false;  // no call has steps after the sum
    static constexpr int kTileBytes = 0, kPlanes = 0;
    static constexpr int plane_bytes(int) { return 0; }
    static constexpr int planes_of(int) { return 0; }
};

// ---- shape ------------------------------------------------------------------------------------------
// SR: runs (of 32 columns) each wave computes per stage, one barrier per stage; XST: stages in the LDS ring of
// activations; WD: k-tiles of packed weights in LDS; ADB: the A fragments of the next pair of runs get registers of
// their own.
template <int RT_, int NT_, int WM_, int WN_, int WK_, int SR_, int XST_, int WD_, bool ADB_>
struct BlockShape {
    static constexpr int RT = RT_, NT = NT_, WM = WM_, WN = WN_, WK = WK_, SR = SR_, XST = XST_, WD = WD_;
    static constexpr bool ADB = ADB_;
    static constexpr int WAVES = WM * WN * WK, BM = 16 * RT * WM, BN = 16 * NT * WN;
    static constexpr int RUNS = 8 / WK;  // of a k-tile, per wave
    static constexpr int kThreads = WAVES * 64;
    template <class Src>
    static constexpr int slot_bytes()
    {
        return BN * 64 + (Src::kRunStaged ? BM * 64 : 0);
    }
    template <class Src>
    static constexpr int ring_bytes()
    {
        return SR * WK * XST * slot_bytes<Src>();
    }
    template <class Src>
    static constexpr int wtile_bytes()
    {
        int b = 0;
        for (int p = 0; p < Src::kPlanes; ++p)
            b += BM / 16 * Src::plane_bytes(p);
        return b + (Src::kGroupScales ? BM * 4 : 0);  // the group scales of a k-tile behind its planes
    }
    template <class Src>
    static constexpr int plane_offset(int p)
    {
        int b = 0;
        for (int i = 0; i < p; ++i)
            b += BM / 16 * Src::plane_bytes(i);
        return b;
    }
    template <class Src>
    static constexpr int lds_bytes()
    {
        return ring_bytes<Src>() + WD * wtile_bytes<Src>();
    }
    // copies one wave contributes to plane p of a k-tile
    template <class Src>
    static constexpr int plane_copies(int p)
    {
        const int n = BM / 16 * Src::plane_bytes(p) / 1024;
        return n >= WAVES ? n / WAVES : 1;
    }
    // first pair of its own (0 .. RUNS/2 - 1) for which a wave of k group wk needs plane p; -1: never
    template <class Src>
    static constexpr int need(int p, int wk)
    {
        for (int l = 0; l < RUNS / 2; ++l)
            if (Src::planes_of(wk * (RUNS / 2) + l) >> p & 1)
                return l;
        return -1;
    }
    // first and last such pair over the k groups
    template <class Src>
    static constexpr int need_min(int p)
    {
        int m = RUNS;
        for (int k = 0; k < WK; ++k)
            m = need<Src>(p, k) >= 0 && need<Src>(p, k) < m ? need<Src>(p, k) : m;
        return m;
    }
    template <class Src>
    static constexpr int need_max(int p)
    {
        int m = 0;
        for (int k = 0; k < WK; ++k)
            m = need<Src>(p, k) > m ? need<Src>(p, k) : m;
        return m;
    }
    // run during which the planes that a wave's pair l needs first are read from LDS (of the k-tile before for l = 0)
    static constexpr int read_run(int l) { return (2 * l + RUNS - (ADB ? 2 : 1)) % RUNS; }
    // stage, counted from the k-tile's first, in which those reads are issued (-1: the last stage of the k-tile before)
    static constexpr int read_stage(int l) { return l == 0 ? -1 : read_run(l) / SR; }
    // stage of a k-tile in which the slot of plane p is requested again: the one after its last read is issued.  The
    // barrier that opens such a stage comes after a wait for the wave's LDS reads, see block_barrier().
    template <class Src>
    static constexpr int request_stage(int p)
    {
        return read_stage(need_max<Src>(p)) + 1;
    }
    // weight and scale copies one wave requests in stage s of a k-tile
    template <class Src>
    static constexpr int stage_w_copies(int s)
    {
        int n = Src::kGroupScales && s == 0 ? 1 : 0;
        for (int p = 0; p < Src::kPlanes; ++p)
            n += request_stage<Src>(p) == s ? plane_copies<Src>(p) : 0;
        return n;
    }
    static constexpr int kStagesPerTile = RUNS / SR;
    // A stage is two neighbouring runs: what is staged run by run is copied and stored as 64 columns, in whole 128-byte lines.
    // (With two k groups that makes them take the even and the odd runs, which only run-staged weights can do.)
    template <class Src>
    static constexpr bool paired()
    {
        return SR * WK == 2 && (WK == 1 || Src::kRunStaged);
    }
    template <class Src>
    static constexpr int x_copies()
    {
        return SR * WK * (BN + (Src::kRunStaged ? BM : 0)) / 16 / WAVES;
    }
    // requests of a wave after those of stage s + 1, counted at the top of stage s
    template <class Src>
    static constexpr int copies_after(int s)
    {
        int n = 0;
        for (int d = 1; d <= XST - 3; ++d)
            n += x_copies<Src>() + stage_w_copies<Src>((s - d + 8 * kStagesPerTile) % kStagesPerTile);
        return n;
    }
    // every plane has landed when it is read: requested no later than the activations of the stage after that
    template <class Src>
    static constexpr bool planes_land()
    {
        for (int p = 0; p < Src::kPlanes; ++p) {
            const int l = need_min<Src>(p);
            const int reads = (RUNS * (l == 0 ? WD - 1 : WD) + read_run(l)) / SR;
            if (request_stage<Src>(p) > reads + 2 - XST)
                return false;
            if (request_stage<Src>(p) >= kStagesPerTile)
                return false;
        }
        return true;
    }
    // no plane is requested again in or before the stage in which a wave of some k group issues its reads of it (group
    // scales are read with the planes of pair 0 and requested in stage 0)
    template <class Src>
    static constexpr bool planes_released()
    {
        for (int p = 0; p < Src::kPlanes; ++p)
            for (int k = 0; k < WK; ++k)
                if (need<Src>(p, k) >= 0 && read_stage(need<Src>(p, k)) >= request_stage<Src>(p))
                    return false;
        return !Src::kGroupScales || read_stage(0) < 0;
    }
};

// Which piece a block works on: unit (row block and k slice) and token block; unit = units: none.  Consecutive block ids
// land on consecutive XCDs.  Each XCD takes `chunk` consecutive pieces.  The pieces are ordered by eighths of the units
// (slice-major, so that an eighth shares the activations of few slices), each walked in groups of eight units x all token
// blocks, units fastest.
//   An XCD takes an eighth of the units with all their token blocks where that gives the fullest one no more rounds of its 32
// CUs than dealing the pieces evenly does, and at most 1/8 more pieces: no weights are then read by two XCDs.  (Weights
// that stay in the L2s from call to call, fp16: 6400 x 1280, N = 102 8.6 us against 12.9 with even pieces; weights from
// memory, 1200 calls: median equal; several rounds, fp16: equal to 2 %, up to 13 %.)
//   Elsewhere the pieces are dealt evenly: 20 units x 11 token blocks give each XCD 27 or 28 blocks, where whole units gave
// six of them 33 and the launch a second round (5104 x 1024, N = 2571, 3 bits 54.5 -> 36.1 us; 6992 x 11008, N = 301,
// group scales 110.8 -> 71.4).
struct BlockPiece {
    int unit, n_block;
};
constexpr int kXcds = 8, kCusPerXcd = 32;
__host__ __device__ constexpr int pieces_per_xcd(int units, int n_blocks)
{
    const int64_t whole = (int64_t)((units + kXcds - 1) / kXcds) * n_blocks;
    const int64_t even = ((int64_t)units * n_blocks + kXcds - 1) / kXcds;
    const bool same_rounds = (whole + kCusPerXcd - 1) / kCusPerXcd == (even + kCusPerXcd - 1) / kCusPerXcd;
    return (int)(same_rounds && 8 * whole <= 9 * even ? whole : even);
}
__host__ __device__ constexpr BlockPiece piece_of_block(int id, int units, int n_blocks, int chunk)
{
    constexpr int kGroup = 8;
    const int eighth = (units + kXcds - 1) / kXcds;
    int rest = id % kXcds * chunk + id / kXcds;
    const int first = rest / (eighth * n_blocks) * eighth;
    if (first >= units)
        return {units, 0};  // the grid is padded to a multiple of eight
    rest -= first * n_blocks;
    const int here = units - first < eighth ? units - first : eighth;
    const int group = rest / (kGroup * n_blocks) * kGroup;
    if (group >= here)
        return {units, 0};
    rest -= group * n_blocks;
    const int in_group = here - group < kGroup ? here - group : kGroup;
    return rest < in_group * n_blocks ? BlockPiece{first + group + rest % in_group, rest / in_group} : BlockPiece{units, 0};
}

// Copies into the LDS slot of a weight plane or of group scales.  The comment in the statement marks them in the
// generated assembly, where the build looks for LDS reads in flight at the barrier before them.
template <int IMM>
__device__ __forceinline__ void issue_refill_b128(rsrc_t rsrc, int lane_off, uint32_t lds_base)
{
    static_assert(IMM >= 0 && IMM < 4096, "the immediate offset of a buffer load is a 12-bit field");
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen offset:%3 lds ; slot refill"
                 : : "s"(lds_base), "v"(lane_off), "s"(rsrc), "n"(IMM) : "memory");
}

__device__ __forceinline__ void issue_refill_b32(rsrc_t rsrc, int lane_off, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen offset:0 lds ; slot refill"
                 : : "s"(lds_base), "v"(lane_off), "s"(rsrc) : "memory");
}

// A bare barrier: unlike __syncthreads it does not wait for LDS reads.  Those in flight across it are activation (and
// fp16 weight) fragments of the stage that it opens, whose slots nobody requests again before the next barrier.  Where
// the stage requests a weight slot again, the wave first waits for its LDS reads (wait_lds_reads): the words that other
// waves' copies are about to overwrite have then arrived.  (57344 x 8192, N = 4096, 6 bits: 2717 us with that wait, 2719
// with one for the reads of planes alone; requests one stage later, after the conversions, take the same time and spill
// with 5 bits.)
// Everything before the barrier in the program, the matrix instructions that consumed earlier reads included, stays
// before it.
__device__ __forceinline__ void block_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" : : : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" : : : "memory");
    __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }

template <class Src, class Shape>
__global__ __launch_bounds__(Shape::kThreads) void linear_block_kernel(
    const void *__restrict__ weights, const half_t *__restrict__ scales, const half_t *__restrict__ X, half_t *Y, int M,
    int N, int K, int S, int n_blocks, int row_blocks, int chunk, float4_t *__restrict__ partials,
    int *__restrict__ counters, int counter_step, Epilogue epi)
{
    constexpr int RT = Shape::RT, NT = Shape::NT, WM = Shape::WM, WN = Shape::WN, WK = Shape::WK;
    constexpr int SR = Shape::SR, XST = Shape::XST, WD = Shape::WD, WAVES = Shape::WAVES;
    constexpr int BM = Shape::BM, BN = Shape::BN, RUNS = Shape::RUNS;
    constexpr bool ADB = Shape::ADB || Src::kRunStaged;
    constexpr int SLOT = Shape::template slot_bytes<Src>(), RING = Shape::template ring_bytes<Src>();
    constexpr int WTILE = Shape::template wtile_bytes<Src>();
    constexpr int XCOPIES = Shape::template x_copies<Src>();
    constexpr int NST = Shape::kStagesPerTile;
    constexpr bool PAIR = Shape::template paired<Src>();
    static_assert(SR * WK * BN / 16 % WAVES == 0 && (!Src::kRunStaged || SR * WK * BM / 16 % WAVES == 0),
                  "copies of a stage must split evenly over the waves");
    static_assert(Shape::template planes_land<Src>(), "a weight plane could be read before it has landed");
    static_assert(Shape::template planes_released<Src>(), "a weight plane could be overwritten before its reads have returned");
    static_assert(XST >= 3 && XST - 3 <= NST && RUNS % SR == 0, "bad stage");
    static_assert(!Src::kGroupScales || XST <= (RUNS * WD - (ADB ? 2 : 1)) / SR + 2, "group scales could be read before they have landed");
    static_assert(RT % 2 == 0, "pieces are converted two at a time");

    extern __shared__ u32x4 xs_dyn[];
    uint8_t *const lds = reinterpret_cast<uint8_t *>(xs_dyn);
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(xs_dyn);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM % WN, wk = wave / (WM * WN);
    const int KT = K / kTileK;
    const int n_row_tiles = M / kTileRows;

    const BlockPiece at = piece_of_block(blockIdx.x, row_blocks * S, n_blocks, chunk);
    if (at.unit >= row_blocks * S)
        return;  // padding (whole block, before any barrier)
    const int unit = at.unit, n_block = at.n_block;
    const int split = unit / row_blocks, row_block = unit - split * row_blocks;
    const int row0 = row_block * BM, col0 = n_block * BN;
    // k-tiles split, split + S, ... of the row block
    const int n_valid = KT / S + (split < KT % S ? 1 : 0);

    // ---- requests.  Copy c of a stage of activations serves ring slot e = c / (BN/16) of the stage and token tile
    // c % (BN/16); slot e holds run e / WK of k group e % WK, which starts at run RUNS * (e % WK) of the k-tile.
    const rsrc_t x_rsrc = make_rsrc(X, (uint32_t)N * (uint32_t)K * 2u);
    constexpr int XC = SR * WK * BN / 16 / WAVES;  // of activations, per wave
    uint32_t x_off[XC];
    int x_dst[XC];
    {
        const int n = lane >> 2, rho = lane >> 3;
#pragma unroll
        for (int i = 0; i < XC; ++i) {
            const int c = wave + WAVES * i, e = c / (BN / 16), tile = c % (BN / 16);
            const int q = (lane & 3) ^ x_swizzle(n), run = e / WK + e % WK * RUNS;
            const int col = col0 + (PAIR ? c * 8 + rho : tile * 16 + n);
            const int k = split * kTileK + (PAIR ? ((lane & 7) ^ w_swizzle(rho)) * 8 : run * 32 + q * 8);
            x_off[i] = col < N ? (uint32_t)(col * K + k) * 2u : (uint32_t)kOutOfRange;
            x_dst[i] = PAIR ? c * 1024 : e * SLOT + tile * 1024;
        }
    }
    int a_off = 0;  // lane offset in a row tile of run-staged weights
    if constexpr (Src::kRunStaged) {
        const int n = PAIR ? lane >> 3 : lane >> 2;
        a_off = (n * K + split * kTileK + (PAIR ? (lane & 7) ^ w_swizzle(n) : (lane & 3) ^ x_swizzle(n)) * 8) * 2;
    }
    const int x_step = S * kTileK * 2;  // bytes of activations (or of row-major weights) from one k-tile to the next
    // copy i of the stage that starts at run `run` of k-tile t, into the ring slots at `slot`
    auto x_issue = [&](int t, int run, int i, int slot) {
        issue_load_to_lds_b128<0>(x_rsrc, (int)(x_off[i] + (uint32_t)(t * x_step + run * (PAIR ? WK * 64 : 64))),
                                  (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + slot + x_dst[i])));
    };
    auto a_issue = [&](int t, int run, int i, int slot) {
        const int c = wave + WAVES * i, e = c / (BM / 16), tile = PAIR ? c / 2 : c % (BM / 16);
        const int rt = row0 / 16 + tile < n_row_tiles ? row0 / 16 + tile : n_row_tiles - 1;
        const rsrc_t r = make_rsrc(static_cast<const half_t *>(weights) + ((int64_t)rt * kTileRows + (PAIR ? c % 2 * 8 : 0)) * K,
                                   (uint32_t)((PAIR ? 8 : kTileRows) * K * 2));
        const int k_bytes = (PAIR ? run * WK : run + e / WK + e % WK * RUNS) * 64;
        issue_load_to_lds_b128<0>(r, a_off + t * x_step + k_bytes,
                                  (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + slot + (PAIR ? BN * 128 + c * 1024 : e * SLOT + BN * 64 + tile * 1024))));
    };
    auto x_issue_one = [&](int t, int run, int i, int slot) {  // copy i of both: activations first, then run-staged weights
        if (i < XC)
            x_issue(t, run, i < XC ? i : 0, slot);
        else
            a_issue(t, run, i - XC, slot);
    };

    // packed weights: the slice's k-tiles, every row tile of the matrix
    constexpr int PC = BM / 16 / WAVES > 0 ? BM / 16 / WAVES : 1;  // copies per wave of a 1 KB plane
    rsrc_t w_rsrc;
    constexpr int HC = BM / 32 / WAVES > 0 ? BM / 32 / WAVES : 1;  // ... of a 512-byte plane
    int w_off[PC], w_half_off[HC], w_stride = 0;
    if constexpr (!Src::kRunStaged) {
        const int tiles0 = Src::kHalfTiles ? split / 2 : split;
        const int KTT = Src::kHalfTiles ? (KT + 1) / 2 : KT;
        w_stride = n_row_tiles * Src::kTileBytes;
        w_rsrc = make_rsrc(static_cast<const uint8_t *>(weights) + (int64_t)tiles0 * w_stride, (uint32_t)((KTT - tiles0) * w_stride));
#pragma unroll
        for (int i = 0; i < PC; ++i) {
            const int tile = (wave + WAVES * i) % (BM / 16);
            const int rt = row0 / 16 + tile < n_row_tiles ? row0 / 16 + tile : n_row_tiles - 1;
            w_off[i] = rt * Src::kTileBytes + lane * 16;
        }
        if (Src::plane_bytes(Src::kPlanes - 1) == 512) {  // two tiles per copy
#pragma unroll
            for (int i = 0; i < HC; ++i) {
                const int tile = 2 * ((wave + WAVES * i) % (BM / 32));
                const int rt = row0 / 16 + tile < n_row_tiles ? row0 / 16 + tile : n_row_tiles - 1;
                w_half_off[i] = (rt + (lane >> 5)) * Src::kTileBytes + (lane & 31) * 16;
            }
        }
    }
    // byte offset of k-tile t of the slice from the first; out of range past the slice
    auto w_at = [&](int t) {
        int o;
        if (Src::kHalfTiles) {
            const int kt = split + t * S;
            o = ((kt >> 1) - (split >> 1)) * w_stride;
        } else {
            o = t * S * w_stride;
        }
        return t < n_valid ? o : kOutOfRange;
    };
    auto w_issue_one = [&](auto pc, int t, int i, int wslot) {
        constexpr int p = decltype(pc)::value;
        if constexpr (!Src::kRunStaged) {
            // the immediate offset of a copy counts on both sides
            constexpr int dst = RING + Shape::template plane_offset<Src>(p) - p * 1024;
            if constexpr (Src::plane_bytes(p) == 1024) {
                const int tile = (wave + WAVES * i) % (BM / 16);
                const int half = Src::kHalfTiles && p == 0 ? ((split + t * S) & 1) * 2048 : 0;
                issue_refill_b128<p * 1024>(w_rsrc, w_off[i < PC ? i : 0] + w_at(t) + half,
                                            (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + dst + wslot + tile * 1024)));
            } else {
                const int c = (wave + WAVES * i) % (BM / 32);
                issue_refill_b128<p * 1024>(w_rsrc, w_half_off[i < HC ? i : 0] + w_at(t),
                                            (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + dst + wslot + c * 1024)));
            }
        }
    };
    // group scales: one word (two groups) per row and k-tile, copied 64 rows at a time
    const int wrow0 = row0 + wm * RT * 16;  // first row of the wave
    constexpr int SCALES = RING + WTILE - BM * 4;
    rsrc_t s_rsrc;
    int s_off = 0;
    if constexpr (Src::kGroupScales) {
        const int groups = K / kGroupColumns, c = wave % (BM / 64);
        const int base = row0 + 64 * c < M ? row0 + 64 * c : M - 1, rows = M - base < 64 ? M - base : 64;
        s_rsrc = make_rsrc(scales + (int64_t)base * groups, (uint32_t)(rows * groups * 2));
        s_off = ((lane < rows ? lane : rows - 1) * groups + 2 * split) * 2;
    }
    auto s_issue = [&](int t, int wslot) {
        if constexpr (Src::kGroupScales)
            issue_refill_b32(s_rsrc, s_off + (t < n_valid ? t * S * 4 : 0),
                             (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + SCALES + wslot + wave % (BM / 64) * 256)));
    };

    // ---- LDS reads
    // a run's 16 rows x 32 columns (unpaired: 1 KB), or its half of 16 rows x 64 columns (paired: chunk 4 * odd + q of each row)
    const int piece_row = lane & 15;
    const int piece = PAIR ? ((piece_row >> 3) * 64 + 8 * (piece_row & 7) + ((lane >> 4) ^ w_swizzle(piece_row))) * 16 : x_piece_of_lane(lane) * 16;
    constexpr int TILE = PAIR ? 2048 : 1024;
    const int b_base = (PAIR ? 0 : wk * SLOT) + wn * NT * TILE, a_base = (PAIR ? BN * 128 : wk * SLOT + BN * 64) + wm * RT * TILE;
    const int b_even = b_base + piece, b_odd = b_base + (piece ^ 64), a_even = a_base + piece, a_odd = a_base + (piece ^ 64);
    auto ldb = [&](int slot, int nt, bool odd) { return bit_cast<half8_t>(*reinterpret_cast<const u32x4 *>(lds + (slot + (odd ? b_odd : b_even)) + nt * TILE)); };
    auto lda = [&](int slot, int g, bool odd) { return bit_cast<half8_t>(*reinterpret_cast<const u32x4 *>(lds + (slot + (odd ? a_odd : a_even)) + g * TILE)); };
    typename Src::Piece pieces[RT];
    half2_t group_scale[RT];
    // planes that first serve the wave's pair l of k-tile t, row tile g
    auto read_planes = [&](auto wk_c, auto pair_c, auto unit_c, int wslot, int t) {
        constexpr int wkc = decltype(wk_c)::value, l = decltype(pair_c)::value, g = decltype(unit_c)::value;
        if constexpr (!Src::kRunStaged) {
            static_for<Src::kPlanes>([&](auto pc) {
                constexpr int p = decltype(pc)::value;
                if constexpr (Shape::template need<Src>(p, wkc) == l) {
                    constexpr int pb = Src::plane_bytes(p);
                    Src::template read_plane<p>(pieces[g], lds + RING + Shape::template plane_offset<Src>(p) + wslot + (wm * RT + g) * pb,
                                                lane, Src::kHalfTiles ? (split + t * S) & 1 : 0);
                }
            });
            if constexpr (Src::kGroupScales && l == 0)
                group_scale[g] = bit_cast<half2_t>(*reinterpret_cast<const uint32_t *>(lds + SCALES + wslot + ((wm * RT + g) * 16 + (lane & 15)) * 4));
        }
    };
    half8_t a[ADB ? 2 : 1][2][RT];  // [buffer][run of the pair][row tile]
    // pieces 2 * unit and 2 * unit + 1 of the wave -> their fragments of its pair l
    auto convert = [&](auto wk_c, auto pair_c, auto buf_c, auto unit_c) {
        constexpr int pair = decltype(wk_c)::value * (RUNS / 2) + decltype(pair_c)::value;
        constexpr int buf = decltype(buf_c)::value, g = 2 * decltype(unit_c)::value;
        if constexpr (!Src::kRunStaged) {
            half8_t f0[2], f1[2];
            Src::template fragments<pair>(pieces[g], pieces[g + 1], f0, f1);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                if constexpr (Src::kGroupScales) {
                    f0[e] *= group_scale[g][pair / 2];
                    f1[e] *= group_scale[g + 1][pair / 2];
                }
                a[buf][e][g] = f0[e];
                a[buf][e][g + 1] = f1[e];
            }
        }
    };

    float4_t acc[RT][NT];
#pragma unroll
    for (int g = 0; g < RT; ++g)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            acc[g][nt] = (float4_t){0.f, 0.f, 0.f, 0.f};

    // ---- requests of a stage: k-tile t's refill of the planes whose last read was in the stage before
    auto w_stage_unit = [&](auto stage_c, auto unit_c, int t, int wslot) {
        constexpr int stage = decltype(stage_c)::value, k = decltype(unit_c)::value;
        constexpr int sc0 = Src::kGroupScales && stage == 0 ? 1 : 0;
        if constexpr (k < sc0) {
            s_issue(t, wslot);
        } else {
            static_for<Src::kPlanes>([&](auto pc) {
                constexpr int p = decltype(pc)::value;
                constexpr int first = [] {
                    int n = sc0;
                    for (int u = 0; u < p; ++u)
                        n += Shape::template request_stage<Src>(u) == stage ? Shape::template plane_copies<Src>(u) : 0;
                    return n;
                }();
                if constexpr (Shape::template request_stage<Src>(p) == stage && k >= first
                              && k < first + Shape::template plane_copies<Src>(p))
                    w_issue_one(pc, t, k - first, wslot);
            });
        }
    };
    auto w_tile = [&](int t, int wslot) {  // a whole k-tile, in the order of the stages
        static_for<NST>([&](auto sc) {
            static_for<Shape::template stage_w_copies<Src>(decltype(sc)::value)>([&](auto kc) { w_stage_unit(sc, kc, t, wslot); });
        });
    };
    constexpr int STAGE_BYTES = SR * WK * SLOT;

    // ---- prologue: WD k-tiles of weights, XST - 1 stages of activations
    static_for<WD>([&](auto dc) { w_tile(decltype(dc)::value, decltype(dc)::value * WTILE); });
    static_for<XST - 1>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
#pragma unroll
        for (int i = 0; i < XCOPIES; ++i)
            x_issue_one(s / NST, s % NST * SR, i, s * STAGE_BYTES);
    });
    wait_loads<(XST - 2) * XCOPIES>();
    block_barrier();

    constexpr int LOOK = NT < 4 ? 2 : RT * NT == 32 ? 2 : 4;  // B fragments requested ahead of their use
    static_assert(NT % LOOK == 0, "ring of B fragments");
    auto k_loop = [&](auto wk_c) {
        half8_t bq[LOOK];
        // whether a run of the wave is the odd one of its pair
        constexpr auto odd = [](int run) { return PAIR && (WK == 2 ? decltype(wk_c)::value == 1 : run % 2 == 1); };
        static_for<LOOK>([&](auto ic) { bq[decltype(ic)::value] = ldb(0, decltype(ic)::value, odd(0)); });
        static_for<RT>([&](auto uc) {
            read_planes(wk_c, std::integral_constant<int, 0>{}, uc, 0, 0);
            if constexpr (Src::kRunStaged)
                a[0][0][decltype(uc)::value] = lda(0, decltype(uc)::value, odd(0));
        });
        if constexpr (!Src::kRunStaged && ADB)
            static_for<RT / 2>([&](auto uc) { convert(wk_c, std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, uc); });

        int slot = 0, prev_stage = (XST - 1) * SR * WK * SLOT;  // ring offsets of the current run and of the previous stage
        int wslot = 0;                                          // of the k-tile's weights
        for (int t = 0; t < n_valid; ++t) {
            const int wnext = wslot + WTILE == WD * WTILE ? 0 : wslot + WTILE;
            static_for<RUNS>([&](auto rc) {
                constexpr int run = decltype(rc)::value, e = run & 1, pair = run / 2, stage = run / SR, NP = RUNS / 2;
                typedef std::integral_constant<int, (pair + 1) % NP> NextPair;
                if constexpr (run % SR == 0) {
                    // the activations of the next stage have landed (this stage's became visible one stage ago)
                    if (t == 0)
                        wait_loads<(XST - 3) * XCOPIES>();
                    else
                        wait_loads<Shape::template copies_after<Src>(stage)>();
                    if constexpr (Shape::template stage_w_copies<Src>(stage) > 0)
                        wait_lds_reads();
                    block_barrier();
                }
                constexpr int STEP = !PAIR ? WK * SLOT : WK == 2 || run % 2 == 1 ? 2 * SLOT : 0;
                const int next_slot = slot + STEP == RING ? 0 : slot + STEP;
                if constexpr (!Src::kRunStaged && !ADB && e == 0)
                    static_for<RT / 2>([&](auto uc) { convert(wk_c, std::integral_constant<int, pair>{}, std::integral_constant<int, 0>{}, uc); });
                static_for<NT>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    const half8_t b = bq[i % LOOK];
                    // the A fragments ahead of their use: reads of packed words, conversions, or (run-staged) the reads themselves
                    if constexpr (Src::kRunStaged) {
                        static_for<RT>([&](auto uc) {
                            constexpr int u = decltype(uc)::value;
                            if constexpr (u * NT / RT == i)
                                a[(run + 1) & 1][0][u] = lda(next_slot, u, odd(run + 1));
                        });
                    } else {
                        if constexpr (e == (ADB ? 0 : 1))
                            static_for<RT>([&](auto uc) {
                                if constexpr (decltype(uc)::value * NT / RT == i)
                                    read_planes(wk_c, NextPair{}, uc, pair == NP - 1 ? wnext : wslot, pair == NP - 1 ? t + 1 : t);
                            });
                        if constexpr (ADB && e == 1)
                            static_for<RT / 2>([&](auto uc) {
                                if constexpr (decltype(uc)::value * NT / (RT / 2) == i)
                                    convert(wk_c, NextPair{}, std::integral_constant<int, (pair + 1) & 1>{}, uc);
                            });
                    }
                    bq[i % LOOK] = i + LOOK < NT ? ldb(slot, i + LOOK, odd(run)) : ldb(next_slot, i + LOOK - NT, odd(run + 1));
#pragma unroll
                    for (int g = 0; g < RT; ++g) {
                        const half8_t &af = Src::kRunStaged ? a[ADB ? run & 1 : 0][0][g] : a[ADB ? pair & 1 : 0][e][g];
                        acc[g][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af, b, acc[g][i], 0, 0, 0);
                    }
                    // requests of this stage, spread over its steps: weights first, then the activations XST - 1 stages ahead
                    constexpr int SSTEPS = SR * NT, st = run % SR * NT + i;
                    constexpr int WC = Shape::template stage_w_copies<Src>(stage), UNITS = WC + XCOPIES;
                    static_for<UNITS>([&](auto kc) {
                        constexpr int k = decltype(kc)::value;
                        constexpr int at = (k + 1) * SSTEPS / (UNITS + 1) - 1;
                        if constexpr ((at < 0 ? 0 : at) == st) {
                            if constexpr (k < WC) {
                                w_stage_unit(std::integral_constant<int, stage>{}, kc, t + WD, wslot);
                            } else {
                                constexpr int ahead_run = (stage + XST - 1) * SR;
                                x_issue_one(t + ahead_run / RUNS, ahead_run % RUNS, k - WC, prev_stage);
                            }
                        }
                    });
                    __builtin_amdgcn_sched_barrier(0);  // the steps stay in this order
                });
                if constexpr (run % SR == SR - 1)
                    prev_stage = next_slot - SR * WK * SLOT < 0 ? next_slot - SR * WK * SLOT + RING : next_slot - SR * WK * SLOT;
                slot = next_slot;
            });
            wslot = wnext;
        }
    };
    if (WK == 1 || wk == 0)
        k_loop(std::integral_constant<int, 0>{});
    else
        k_loop(std::integral_constant<int, WK - 1>{});
    wait_loads<0>();  // the look-ahead copies land before the block gives up its LDS

    // ---- the two waves of a piece meet: each ends up with half of its 16 x 16 tiles
    constexpr int OWN_ROWS = RT / WK, OWN = OWN_ROWS * NT;  // tile o = r * NT + nt of the wave's own
    static_assert(RT % WK == 0, "tiles of a wave pair");
    float4_t own[OWN_ROWS][NT];
    if constexpr (WK == 2) {
        __syncthreads();
        float4_t *ex = reinterpret_cast<float4_t *>(lds);
        static_assert(WAVES * OWN * 1024 <= Shape::template lds_bytes<Src>(), "exchange buffer");
#pragma unroll
        for (int o = 0; o < OWN; ++o)
            ex[(wave * OWN + o) * 64 + lane] = wk == 0 ? acc[OWN_ROWS + o / NT][o % NT] : acc[o / NT][o % NT];
        __syncthreads();
        const int partner = wave ^ (WM * WN);
#pragma unroll
        for (int o = 0; o < OWN; ++o)
            own[o / NT][o % NT] = (wk == 0 ? acc[o / NT][o % NT] : acc[OWN_ROWS + o / NT][o % NT]) + ex[(partner * OWN + o) * 64 + lane];
    } else {
#pragma unroll
        for (int o = 0; o < OWN; ++o)
            own[o / NT][o % NT] = acc[o / NT][o % NT];
    }

    // ---- last step.  Lane L holds rows 4*(L/16) + i of token column L%16 of a 16 x 16 tile.
    const int own_row0 = wrow0 + wk * OWN_ROWS * 16, own_col0 = col0 + wn * NT * 16;
    RowTerms terms[OWN_ROWS];
    row_terms_of_tiles<Src::kHasScale, Src::kFused>(terms, epi, scales, own_row0, M, lane);
    if (S > 1) {
        // split-K, one arrival counter per wave tile: see linear_stream.hpp for the protocol
        const int64_t tile_id = (int64_t)row_block * n_blocks + n_block;
        const int64_t tiles = (int64_t)row_blocks * n_blocks;
        constexpr int WAVE_BYTES = OWN * 1024;
        auto slice_of = [&](int s) {
            return partial_buffer(reinterpret_cast<uint8_t *>(partials) + ((s * tiles + tile_id) * WAVES + wave) * WAVE_BYTES, WAVE_BYTES);
        };
        {
            const partial_rsrc_t dst = slice_of(split);
#pragma unroll
            for (int o = 0; o < OWN; ++o)
                if (own_col0 + o % NT * 16 < N && own_row0 + o / NT * 16 < M)  // the same for every lane
                    agent_store(dst, o * 1024 + lane * 16, own[o / NT][o % NT]);
        }
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's partial stores are done
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        int arrived = 0;
        int *counter = counters + (tile_id * WAVES + wave) * counter_step;
        if (lane == 0)
            arrived = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        arrived = __builtin_amdgcn_readfirstlane(arrived);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        if (arrived != S - 1)
            return;
        if (lane == 0)
            *counter = 0;  // re-arm for the next call on this workspace
        // groups of output tiles as large as the registers hold, finished as they are: brought together with the accumulators of
        // calls without slices they would spill
        constexpr int GT = OWN <= 16 ? NT : 2, GR = OWN <= 16 && OWN_ROWS >= 2 ? 2 : 1, OG = GR * GT;
#pragma unroll
        for (int o0 = 0; o0 < OWN; o0 += OG) {
            const int r0 = o0 / NT, t0 = o0 % NT;
            float4_t sum[OG], group[GR][GT];
            RowTerms group_terms[GR];
            add_slices<3>(sum, S, split, [&](int o) { return own[r0 + o / GT][t0 + o % GT]; }, [&](float4_t (&part)[OG], int s) {
                const partial_rsrc_t src = slice_of(s);
#pragma unroll
                for (int o = 0; o < OG; ++o)
                    part[o] = agent_load(src, (o0 + o) * 1024 + lane * 16);
            });
#pragma unroll
            for (int o = 0; o < OG; ++o) {
                group[o / GT][o % GT] = sum[o];
                group_terms[o / GT] = terms[r0 + o / GT];
            }
            finish_tiles<Src::kHasScale, Src::kFused>(epi, group_terms, group, own_row0 + r0 * 16, own_col0 + t0 * 16, M, N, Y, lane);
        }
        return;
    }
    finish_tiles<Src::kHasScale, Src::kFused>(epi, terms, own, own_row0, own_col0, M, N, Y, lane);
}

}  // namespace fp6
