// Weight-streaming linear-layer kernel for small token counts (N <= 64), where the
// layer is bound by reading the weights once from HBM (Section 3 and Section 7.1 of
// the paper: linear layers at batch < 128 are limited by weight traffic).
//
// Work split: a block is WM row tiles of 16 rows times WK groups of k-tiles, one wave each; a wave owns its group's share of
// one split-K slice of one row tile (the
// weight source says how wide a tile is: 256 columns, 512 for the sources whose lane
// loads only come out as whole 128-bit pieces that way); weights go HBM -> VGPR with a
// few 128-bit loads per lane per tile (three for 6 bits), requested two tiles ahead,
// and are used by exactly one wave, so they never touch LDS (one source, row-major fp16
// weights, stages its tiles in a region of LDS private to the wave instead).  The
// activations (16*NT tokens) are the only shared operand: the block copies
// them global -> LDS without passing through registers, whole lines at a time, swizzled so
// that B fragments read without bank conflicts, a stage of WK k-tiles (one per group) at a time,
// double-buffered, with one barrier per stage.  The groups of a row tile add their sums in LDS at the end: on a layer with few
// row tiles that fills the chip without the trips to memory that k slices cost (2.5 us of a launch).
// fp32 accumulation in v_mfma_f32_16x16x32_f16; the row scale is applied once in the
// epilogue.
//
// Split-K: every wave writes its fp32 partial tile, bumps the arrival counter of its
// row tile, and the wave that arrives last adds the S partials in split order (so the
// result does not depend on arrival order), scales, rounds and stores Y.  The counter
// is reset by that wave, so a zeroed workspace stays reusable.
#pragma once
#include "fp6_device.hpp"

namespace fp6 {

// Shape of one instantiation: NT token tiles per wave; a block is WM row tiles x WK groups of k-tiles, one wave each;
// DEPTH weight tiles in flight per wave; XR tokens of a token tile staged in LDS (16, or with one token tile 8 or 2 for
// calls that have no more: fewer copies).
template <int NT_, int WM_, int WK_, int DEPTH_, int XR_ = 16>
struct StreamShape {
    static constexpr int NT = NT_, WM = WM_, WK = WK_, DEPTH = DEPTH_, XR = XR_;
    static constexpr int WAVES = WM_ * WK_, kThreads = WAVES * 64;
    static_assert(XR == 16 || (NT == 1 && (XR == 8 || XR == 2)), "token rows");
    // 1 KB copies per k-tile of tile_cols columns
    static constexpr int copies_per_tile(int tile_cols) { return NT * (tile_cols / 32) * XR / 16; }
    // bytes of two stages of activations, a stage being WK k-tiles
    static constexpr int x_bytes(int tile_cols) { return 2 * WK * copies_per_tile(tile_cols) * 1024; }
    // dynamic LDS of a launch: the activation stages, then (sources that stage their weights in LDS) DEPTH
    // tiles per wave
    template <class Src>
    static constexpr int lds_bytes()
    {
        return x_bytes(Src::kTileCols) + WAVES * DEPTH * Src::kLdsTileBytes;
    }
};

template <class Src, class Shape>
__global__ __launch_bounds__(Shape::kThreads) void linear_stream_kernel(
    const void *__restrict__ weights, const half_t *__restrict__ scales, const half_t *__restrict__ X,
    half_t *Y, int M, int N, int K, int S, int kt_per_slice, float4_t *__restrict__ partials,
    int *__restrict__ counters, Epilogue epi)
{
    constexpr int NT = Shape::NT, WM = Shape::WM, WK = Shape::WK, WAVES = Shape::WAVES, DEPTH = Shape::DEPTH, XR = Shape::XR;
    constexpr int TILE_COLS = Src::kTileCols;  // columns of one weight tile: one step of the loop (a "k-tile" below)
    constexpr int RUNS = TILE_COLS / 32;        // MFMA steps per tile
    constexpr int TILE_COPIES = Shape::copies_per_tile(TILE_COLS), COPIES = WK * TILE_COPIES;  // per k-tile, per stage
    // copies i of a wave are numbers wave + WAVES * i of the stage; where they do not split evenly some waves have one less
    constexpr int XPER = (COPIES + WAVES - 1) / WAVES;
    constexpr int STAGE_PIECES = COPIES * 64;  // 16-byte pieces of one stage
    constexpr int U = DEPTH % 2 ? 2 * DEPTH : DEPTH;  // unroll: both the stage buffer and the ring slot are static
    constexpr int WLOADS = Src::kLoads;  // weight loads of one wave per k-tile

    extern __shared__ u32x4 xs_dyn[];  // [2][STAGE_PIECES], then [WAVES][DEPTH] weight tiles for sources that stage them

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KT = (K + TILE_COLS - 1) / TILE_COLS;  // a K that is not a multiple of the tile: the last tile is padded
    const int n_row_tiles = M / kTileRows;
    // consecutive blocks take consecutive row blocks of the same k slice (measured a few per cent better at
    // N = 32, 64 than alternating the slices, no difference below)
    // The grid is (row blocks, k slices) and the host passes KT / S: nothing is divided here (a division by
    // a run-time value is a chain of ~30 dependent instructions, and the first request waits for it).
    const int row_block = blockIdx.x;
    const int split = blockIdx.y;
    const int wm = wave % WM, wk = wave / WM;
    const int row_tile = row_block * WM + wm;
    // Split-K: slice s takes k-tiles s, s + S, s + 2S, ... of a row tile: the waves of all slices then stand at the same
    // depth of the k-tile-major weight stream and the launch sweeps memory as one front, whatever S is.  Tile i of wave
    // group wk is number wk + i * WK of the slice.
    const int rem = KT - S * kt_per_slice;
    const int n_valid = kt_per_slice + (split < rem ? 1 : 0);  // k-tiles of this slice (>= 1)
    const int T = kt_per_slice + (rem > 0 ? 1 : 0);            // of the longest slice
    const int n_stages = (T + WK - 1) / WK;
    const int n_own = (n_valid - wk + WK - 1) / WK;  // k-tiles of this wave

    // Waves without a row tile (ragged last row block) or without k-tiles stream a valid tile and drop the result:
    // the request pattern is the same for all of them.
    typename Src::Stream w_stream;
    w_stream.init(weights, scales, row_tile < n_row_tiles ? row_tile : n_row_tiles - 1, n_own > 0 ? split + wk * S : split, S * WK,
                  n_own > 0 ? n_own : 1, n_row_tiles, K, lane);
    const rsrc_t x_rsrc = make_rsrc(X, (uint32_t)N * (uint32_t)K * 2u);

    // ---- activation staging.  A k-tile is stored as blocks of 1 KB, one copy each: token tile nt, segment of 64 columns, half
    // h of the token tile (rows 8h .. 8h+7).  Lane 8*rho + pi of a copy fetches row 8h + rho, 8-column
    // chunk pi ^ w_swizzle(row) of the segment, so the eight lanes of a row fetch one whole 128-byte line (8192 x 22016,
    // N = 64 36.0 -> 34.7 us against copies of 16 rows x 64 bytes with nothing but the copies and the weight loads running;
    // the L1 asks the L2 for each line once either way, 2.53 M requests).  XR = 8: no second half; XR = 2: a block is two rows of 256 columns, chunk pi ^ 4 * row.
    // Tokens >= N lie past the end of the buffer; k-tiles past the end of the slice and segments past K (the padding of a
    // last tile) get an offset outside it: nothing is fetched and zeros land in LDS.
    constexpr int ROWS = XR < 8 ? XR : 8, ROW_LANES = 64 / ROWS, SEG = 8 * ROW_LANES, HALVES = XR / ROWS;
    const uint32_t xs_lds = (uint32_t)reinterpret_cast<uintptr_t>(xs_dyn);  // LDS byte address
    auto segment_of = [&](int j) { return j / HALVES % (TILE_COLS / SEG) * SEG; };  // first column in the tile
    uint32_t x_off[XPER];
#pragma unroll
    for (int i = 0; i < XPER; ++i) {
        const int j = wave + WAVES * i, g = j / TILE_COPIES, nt = NT == 1 ? 0 : j / RUNS % NT;
        const int rho = lane / ROW_LANES, swizzle = XR < 8 ? 4 * rho : w_swizzle(rho);
        const int row = nt * 16 + j % HALVES * 8 + rho;
        const int col = (split + g * S) * TILE_COLS + segment_of(j) + 8 * (lane % ROW_LANES ^ swizzle);
        x_off[i] = ((uint32_t)row * (uint32_t)K + (uint32_t)col) * 2u;
    }
    const uint32_t x_step = (uint32_t)(WK * S * TILE_COLS * 2);
    auto x_issue = [&](int stage, int buf) {
#pragma unroll
        for (int i = 0; i < XPER; ++i) {
            const int j = wave + WAVES * i, t = stage * WK + j / TILE_COPIES;
            if (COPIES % WAVES != 0 && j >= COPIES)
                continue;
            const bool inside = t < n_valid && (K % TILE_COLS == 0 || (split + t * S) * TILE_COLS + segment_of(j) < K);
            const uint32_t lds_base = (uint32_t)__builtin_amdgcn_readfirstlane(
                (int)(xs_lds + (uint32_t)(buf * STAGE_PIECES + j * 64) * 16u));
            issue_load_to_lds_b128<0>(x_rsrc, inside ? (int)(x_off[i] + (uint32_t)stage * x_step) : kOutOfRange, lds_base);
        }
    };

    // B fragment of run f, token tile nt: lane (q, n) reads chunk 4*f + q of token n (with XR < 16 tokens that do not exist
    // read another one's: their columns of the result are dropped)
    const int n_in_tile = lane & 15, q = lane >> 4;
    const int b_row = n_in_tile % ROWS, b_half = XR == 16 ? n_in_tile / 8 * 64 : 0;
    const int b_swizzle = XR < 8 ? 4 * b_row : w_swizzle(b_row);
    const int b_even = b_half + b_row * ROW_LANES + (q ^ b_swizzle), b_odd = b_half + b_row * ROW_LANES + ((4 + q) ^ b_swizzle);
    auto ldb = [&](const u32x4 *xb, int st) {  // step st of a k-tile = run st / NT, token tile st % NT
        const int f = st / NT, nt = st % NT;
        constexpr int PAIRS = ROW_LANES / 8;  // pairs of runs in a segment
        return bit_cast<half8_t>(xb[nt * (RUNS * 64) + f / 2 / PAIRS * (HALVES * 64) + f / 2 % PAIRS * 8 + (f & 1 ? b_odd : b_even)]);
    };
    float4_t acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
        acc[nt] = (float4_t){0.f, 0.f, 0.f, 0.f};

    // One k-tile, RUNS x NT steps of one matrix instruction.  The B fragments travel through a ring of LOOK registers: left to
    // the compiler, every pair of reads is waited for right before its use (8192 x 22016, N = 64: a wave computes for 1.2 of
    // the 1.7 us of a k-tile that way, 0.65 with the ring).  The A fragments of a pair of runs are made one pair ahead.
    // xb: first piece of this k-tile's activations in LDS.  What is left is the memory path: without the matrix work, the LDS
    // reads or both the launch takes the same time, without the activation copies 4 to 7 us less at N = 64.  (10240 x 8192,
    // N = 64 23.3 -> 21.5 us, 12288 x 12288, N = 45, 5 bits 34.8 -> 30.8 with three token tiles instead of four; rings of 4, 6
    // and 12 within 2 %.)
    constexpr int STEPS = RUNS * NT, LOOK = 8;
    auto compute = [&](const typename Src::Tile &t, const u32x4 *xb) {
        half8_t bq[LOOK], a[2][2];
        Src::template fragments<0>(t, a[0][0], a[0][1]);
        static_for<LOOK>([&](auto ic) { bq[decltype(ic)::value] = ldb(xb, decltype(ic)::value); });
        __builtin_amdgcn_sched_barrier(0);
        static_for<STEPS>([&](auto sc) {
            constexpr int st = decltype(sc)::value, f = st / NT, p = f / 2;
            if constexpr (st % (2 * NT) == 0 && p + 1 < RUNS / 2)
                Src::template fragments<p + 1>(t, a[(p + 1) & 1][0], a[(p + 1) & 1][1]);
            acc[st % NT] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[p & 1][f & 1], bq[st % LOOK], acc[st % NT], 0, 0, 0);
            if constexpr (st + LOOK < STEPS)
                bq[st % LOOK] = ldb(xb, st + LOOK);
            __builtin_amdgcn_sched_barrier(0);  // the steps stay in this order
        });
    };

    // ---- software pipeline.  Slot t % DEPTH of the register ring holds weight tile t of the wave; it is
    // requested DEPTH tiles ahead, right after the slot's previous tile has been consumed.  The activation copies of stage t+1
    // are requested at the start of stage t, after its barrier (by then every wave has finished
    // reading the buffer they overwrite).  Loads complete in order, so "at most n outstanding" with n = the
    // loads requested after the ones needed means those have arrived.  The copies of stage t, and the weights of tile t before
    // them, are followed by the weights of one tile only: past the wait that tile alone is in flight, joined by the copies of
    // the next stage while tile t is computed.  A deeper ring alone changes nothing of that, its further tiles have arrived.  (More in flight, three or four buffers of activations with three
    // or four weight tiles: 8192 x 22016, N = 64 36.1 -> 37-43 us, N = 32 equal.)
    // Tiles past the end of the slice read as zeros
    // through the buffer bounds check (no memory traffic), so the request pattern never varies.
    static_assert(DEPTH >= 2, "the wait below leaves the weights of one tile in flight");
    typename Src::Tile w[DEPTH];
    w_stream.bind_slots(w, xs_dyn + 2 * STAGE_PIECES + wave * (DEPTH * Src::kLdsTileBytes / 16), lane);
    x_issue(0, 0);
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        w_stream.issue(w[d], d);
    for (int t0 = 0; t0 < n_stages; t0 += U) {
        static_for<U>([&](auto uc) {
            constexpr int u = decltype(uc)::value, slot = u % DEPTH;
            const int t = t0 + u;
            wait_loads<WLOADS>();
            Src::pin_tile(w[slot]);
            __syncthreads();  // the copies of this stage by all waves have landed; the other buffer is no longer read
            x_issue(t + 1, (u + 1) & 1);
            if (t < n_own)
                compute(w[slot], xs_dyn + (u & 1) * STAGE_PIECES + wk * (TILE_COPIES * 64));
            w_stream.issue(w[slot], t + DEPTH);
        });
    }
    // drain: the look-ahead requests (weights out of range, activation copies into the unused buffer)
    // must land before the registers are reused and before the block gives up its LDS
    wait_loads<0>();
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        Src::pin_tile(w[d]);

    // ---- the groups of k-tiles meet in LDS, added in order
    if constexpr (WK > 1) {
        static_assert((WK - 1) * WM * NT * 1024 <= Shape::x_bytes(TILE_COLS), "exchange buffer");
        float4_t *ex = reinterpret_cast<float4_t *>(xs_dyn);
        __syncthreads();
        if (wk > 0) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                ex[((wave - WM) * NT + nt) * 64 + lane] = acc[nt];
        }
        __syncthreads();
        if (wk > 0)
            return;
#pragma unroll
        for (int k = 0; k < WK - 1; ++k)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                acc[nt] += ex[((k * WM + wm) * NT + nt) * 64 + lane];
    }

    // ---- epilogue.  Lane L holds, per token tile, rows 4*(L/16)+i (i=0..3) of token column L%16.
    if (row_tile >= n_row_tiles)
        return;  // no barrier follows
    const int m0 = row_tile * kTileRows + 4 * (lane >> 4);
    // Scales and bias are requested before the partial sums leave (only the last wave needs them, but then they cost it
    // no trip to memory), the residual beside the partial sums of the other slices.
    RowTerms terms = row_terms<Src::kHasScale>(epi, scales, m0);
    half4_t residual[NT];
    auto request_residual = [&] {
        if (epi.residual) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                if (nt * 16 + n_in_tile < N)
                    residual[nt] = residual_rows(epi, nt * 16 + n_in_tile, m0, M);
        }
    };
    auto finish = [&](const float4_t (&sum)[NT]) {
        pin(terms);
        if (epi.residual) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                pin(residual[nt]);
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int col = nt * 16 + n_in_tile;
            if (col < N)
                finish_rows<Src::kHasScale>(epi, terms, residual[nt], sum[nt], col, m0, M, Y);
        }
    };
    if (S == 1) {
        request_residual();
        finish(acc);
        return;
    }

    // Split-K, one arrival counter per row tile: every wave is on its own from here (no barrier, so a wave
    // that finishes its stream early does not wait for the slowest wave of its block).  The partial tiles
    // are written and read with device-scope atomic (relaxed) accesses: such accesses are performed at the
    // point where all CUs of the device agree (they are not left in, nor served from, a non-coherent
    // cache), so no cache write-back or invalidate is needed.  Order: this wave's stores complete (vmcnt)
    // -> arrival count -> the last wave's loads; the signal fences keep the compiler from moving memory
    // operations across those two points.  The last wave adds the S partial tiles in split order, taking its
    // own from registers (the same bits it stored), so the sum does not depend on who is last.
    auto slice = [&](int s) { return partial_buffer(partials + ((int64_t)s * n_row_tiles + row_tile) * NT * 64, NT * 1024); };
    {
        const partial_rsrc_t dst = slice(split);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            if (nt * 16 + n_in_tile < N)
                agent_store(dst, nt * 1024 + lane * 16, acc[nt]);
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's partial stores are done
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    int arrived = 0;
    if (lane == 0)
        arrived = __hip_atomic_fetch_add(&counters[row_tile], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    arrived = __builtin_amdgcn_readfirstlane(arrived);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    if (arrived != S - 1)
        return;
    request_residual();
    // (every lane loads: lanes of token columns >= N read words that nobody stored, their sums are never written)
    float4_t sum[NT];
    auto own = [&](int nt) { return acc[nt]; };
    auto load = [&](float4_t (&part)[NT], int s) {
        const partial_rsrc_t src = slice(s);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            part[nt] = agent_load(src, nt * 1024 + lane * 16);
    };
    // Three slices together (four of one or two token tiles): with eight, the tests of slices that are not there cost more than trips to
    // memory saved (S = 4, 8192 x 8192, N = 8 11.65 -> 11.53 us, 8192 x 22016, N = 1 22.83 -> 22.65).  One token tile in threes took up to
    // 5.5 % longer from six slices on than in fours with the own tile among them (1376 x 20736, N = 3, fp16, S = 11 15.3 -> 15.8).
    if constexpr (NT == 1)
        add_slices_untested<4>(sum, S, split, own, load);
    else
        add_slices<NT == 2 ? 4 : 3>(sum, S, split, own, load);
    finish(sum);
    if (lane == 0)
        counters[row_tile] = 0;  // re-arm for the next call on this workspace
}

}  // namespace fp6
