// Tiled linear-layer kernel for packed weights at prefill-sized token counts (N > 64) that the block kernel's pieces
// (linear_block.hpp) do not suit better, where the layer is bound by
// the matrix cores (Section 7.1 of the paper: all kernels become compute-bound beyond batch 128).
//
// A block is WM x WN x WK waves; wave (wm, wn) owns RT 16-row tiles and NT 16-token tiles, i.e. a
// (16*RT) x (16*NT) piece of Y held in fp32 accumulators; the block covers (16*RT*WM) rows and
// (16*NT*WN) tokens.  Per 256-column k-tile a wave fetches its RT packed weight tiles straight into
// registers, de-quantizes four runs of 32 columns with one conversion and feeds every run to NT MFMAs (the
// conversion is amortised over 4*NT matrix instructions); every activation fragment read from LDS feeds RT
// MFMAs.  The activations (all tokens of the block) are shared by the block: they are copied
// global -> LDS without passing through registers, already in B-fragment order (the 64 lanes of one
// copy instruction fetch the 64 pieces that the 64 lanes of one MFMA will read), half a k-tile (128
// columns) at a time into a ring of four buffers, requested three half tiles ahead and made visible one
// half tile ahead; weights are double-buffered in registers, one k-tile ahead.  With WK = 2 two waves share such a piece, one
// takes the even and one the odd k-tiles of the slice, and their sums meet in LDS: two waves per SIMD instead of one for the
// blocks of 128 x 64, whose conversions and LDS reads then run under each other's matrix instructions (6656 x 17920, N = 100,
// 3 bits 38.6 -> 34.9 us, 12288 x 12288, N = 96, 5 bits 58.3 -> 54.5, 10240 x 8192, N = 96, 4 bits 33.0 -> 30.1; 6 bits, whose
// conversion is short, gain nothing).  Copying the activations in whole 128-byte lines changed none of them, nor the other blocks.
//
// Split-K and the epilogue are those of the streaming kernel (linear_stream.hpp).
#pragma once
#include "fp6_device.hpp"

namespace fp6 {

template <class Src, int RT, int NT, int WM, int WN, int WK>
__global__ __launch_bounds__(WM * WN * WK * 64) void linear_tiled_kernel(
    const void *__restrict__ weights, const half_t *__restrict__ scales, const half_t *__restrict__ X,
    half_t *Y, int M, int N, int K, int S, int n_blocks, float4_t *__restrict__ partials,
    int *__restrict__ counters, int counter_step, Epilogue epi)
{
    constexpr int WAVES = WM * WN * WK;
    static_assert(WK == 1 || (WK == 2 && RT == 2), "two k groups share two row tiles");
    constexpr int BNT = WN * NT;             // 16-token tiles of the block
    // Activations are staged half a k-tile (128 columns = runs 0..3 or 4..7) at a time in a ring of XS
    // buffers; weights are double-buffered in registers (whole k-tiles).
    constexpr int XS = 4;
    constexpr int XHPIECES = WK * BNT * 256; // 16-byte pieces of one half tile of activations (of every k group)
    constexpr int XHBYTES = XHPIECES * 16;
    constexpr int HCOPIES = WK * BNT * 4;    // copy instructions per half tile (one per token tile and run)
    static_assert(HCOPIES % WAVES == 0, "activation copies must split evenly over the waves");
    constexpr int XPERH = HCOPIES / WAVES;
    constexpr int WLOADS = RT * Src::kLoads; // weight loads of one wave per k-tile

    extern __shared__ u32x4 xs_dyn[];  // [XS][XHPIECES]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM % WN, wk = wave / (WM * WN);
    const int KT = K / kTileK;
    const int n_row_tiles = M / kTileRows;
    // block -> (row block, token block, k slice).  Consecutive block ids land on consecutive XCDs (8 of
    // them, each with its own L2).  The blocks of one XCD take row blocks congruent to the XCD index and,
    // running side by side, all token blocks / k slices of those row blocks: a weight tile is then fetched
    // from memory by one XCD only and the other token blocks hit it in that XCD's L2, while the (much
    // smaller) activations are the operand that every XCD reads in full.
    constexpr int kXcds = 8;
    const int combos = n_blocks * S;
    const int xcd = blockIdx.x % kXcds;
    const int rest = blockIdx.x / kXcds;
    const int combo = rest % combos;
    const int row_block = (rest / combos) * kXcds + xcd;  // may run past the last row block: handled as a ragged edge
    const int n_block = combo % n_blocks;
    const int split = combo / n_blocks;
    if (row_block * WM * RT >= n_row_tiles)
        return;  // padding block of the XCD round-robin (whole block, before any barrier)
    const int row_tile0 = (row_block * WM + wm) * RT;
    const int block_col0 = n_block * BNT * 16;
    const int col0 = block_col0 + wn * NT * 16;  // first token of this wave
    const int kt0 = (int)(((unsigned)KT * (unsigned)split) / (unsigned)S);
    const int kt1 = (int)(((unsigned)KT * (unsigned)(split + 1)) / (unsigned)S);
    const int n_valid = kt1 - kt0;
    // k group wk takes k-tiles wk, wk + WK, ... of the slice ("k-tile t" below is the wave's t-th); a group that has one less, or
    // none, multiplies zero activations
    const int n_steps = (n_valid + WK - 1) / WK, n_own = (n_valid - wk + WK - 1) / WK;

    typename Src::Stream w_stream[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int rt = row_tile0 + r;
        w_stream[r].init(weights, scales, rt < n_row_tiles ? rt : n_row_tiles - 1, n_own > 0 ? kt0 + wk : kt0, WK, n_own > 0 ? n_own : 1, n_row_tiles, K, lane);
    }
    const rsrc_t x_rsrc = make_rsrc(X, (uint32_t)N * (uint32_t)K * 2u);

    // Activation copies: copy j = wave + WAVES*i of half tile h serves token tile nt = j/4 and run
    // f = j%4 + 4*(h%2) of k-tile h/2; lane p of the copy fetches
    // X[block_col0 + 16*nt + n][k0 + k_offset(f, q) ..+8] for the (n, q) that piece p of the 1 KB holds (see
    // x_source_of_piece), and its 16 bytes land at piece 64*j + p of the ring buffer.  Half tiles past the
    // end of the slice and token columns >= N get an offset outside the buffer: zeros land in LDS.
    int xq, xn;
    x_source_of_piece(lane, xn, xq);
    const int b_piece = x_piece_of_lane(lane);
    // LDS byte address of the activation buffers (the low 32 bits of a shared-memory pointer)
    const uint32_t xs_lds = (uint32_t)reinterpret_cast<uintptr_t>(xs_dyn);
    // copy i (of the XPERH this wave contributes) of half tile h into ring buffer buf
    auto x_issue_one = [&](int h, int buf, int i) {
        const int j = wave + WAVES * i;
        const int t = WK * (h >> 1) + (WK == 1 ? 0 : j / (BNT * 4));
        const int nt = (WK == 1 ? j : j % (BNT * 4)) >> 2, f = (j & 3) + 4 * (h & 1);
        const int col = block_col0 + nt * 16 + xn;
        const int off = (t < n_valid && col < N)
                            ? (col * K + (kt0 + t) * kTileK + Src::k_offset(f, xq)) * 2
                            : kOutOfRange;
        const uint32_t lds_base = (uint32_t)__builtin_amdgcn_readfirstlane((int)(xs_lds + buf * XHBYTES + j * 1024));
        issue_load_to_lds_b128<0>(x_rsrc, off, lds_base);
    };
    auto x_issue = [&](int h, int buf) {
#pragma unroll
        for (int i = 0; i < XPERH; ++i)
            x_issue_one(h, buf, i);
    };

    float4_t acc[RT][NT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            acc[r][nt] = (float4_t){0.f, 0.f, 0.f, 0.f};

    // One half tile = 4 runs x NT token tiles = 4*NT steps of RT MFMAs, in two groups of two runs.  B
    // fragments travel through a small ring of registers: the LDS read of step s+LOOK is issued when step s
    // is consumed, and the ring runs on across half tiles (the next half tile is already visible, see
    // below), so the matrix pipe does not drain at a boundary.  The A fragments of the next group are
    // produced (conversion + register moves, VALU work) while the MFMAs of the current group execute.  The
    // sched_group_barrier sequence fixes the instruction order inside a group to "1 LDS read, RT MFMAs, a few
    // VALU" per step: a wave cannot issue anything else while one of its MFMAs is being issued, so the VALU
    // work is laid out in small pieces that the other waves of the SIMD can cover with their own MFMAs.
    constexpr int LOOK = 4;
    constexpr int STEPS = 4 * NT;
    constexpr int VALU_PER_STEP = 2;  // VALU instructions the scheduler may place after the MFMAs of a step
    half8_t a[2][2][RT];  // [group parity][even/odd run][row tile]
    half8_t bq[LOOK];
    auto ldb = [&](const u32x4 *xbuf, int st) {
        return bit_cast<half8_t>(xbuf[(((wk * WN + wn) * NT + (st % NT)) * 4 + st / NT) * 64 + b_piece]);
    };
    // HP: which half of the k-tile t; xbuf: its activations; xnext: those of the following half tile;
    // request(step): called after each of the 4*NT steps of the half tile, issues the memory requests that the
    // schedule places there (the requests of a half step are spread over its matrix work: issued in one burst
    // after the barrier, the ten requests of each of the eight waves queue up in the CU's address unit and the
    // waves stand at the issue of their loads for a quarter of the half step with the matrix pipe idle)
    auto compute_half = [&](auto hp_c, const typename Src::Tile (&t)[RT], const u32x4 *xbuf, const u32x4 *xnext,
                            auto &&request) {
        constexpr int HP = decltype(hp_c)::value;
        static_for<2>([&](auto gh_c) {
            constexpr int GH = decltype(gh_c)::value;
            __builtin_amdgcn_sched_barrier(0);
            if (HP == 0 || GH == 0) {
#pragma unroll
                for (int r = 0; r < RT; ++r)
                    Src::template fragments<(2 * HP + GH + 1 <= 3 ? 2 * HP + GH + 1 : 3)>(t[r], a[GH ^ 1][0][r], a[GH ^ 1][1][r]);
            }
            static_for<2 * NT>([&](auto i_c) {
                constexpr int i = decltype(i_c)::value;
                constexpr int st = 2 * GH * NT + i;
                const half8_t b = bq[st % LOOK];
                bq[st % LOOK] = st + LOOK < STEPS ? ldb(xbuf, st + LOOK) : ldb(xnext, st + LOOK - STEPS);
#pragma unroll
                for (int r = 0; r < RT; ++r)
                    acc[r][st % NT] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[GH][i / NT][r], b, acc[r][st % NT], 0, 0, 0);
                request(std::integral_constant<int, st>{});
            });
#pragma unroll
            for (int i = 0; i < 2 * NT; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, RT, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, VALU_PER_STEP, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // ---- software pipeline.  Half step h (k-tile t = h/2) computes half tile h.  At its top the wave waits
    // for the activations of half tile h+1 (its own copies of them, requested at half step h-2) and, when h
    // is even, for the weights of k-tile t (requested at half step h-2, before those copies); one barrier
    // then makes half tile h+1 visible to the whole block - half tile h became visible one step earlier,
    // which is what lets the B-fragment ring run across the boundary - and guarantees that half tile h-1 is
    // no longer being read, so its buffer takes the copies of half tile h+3, requested next, after the
    // weights of k-tile t+1 when h is even.  Loads complete in order, so "at most n outstanding" with n = the
    // loads requested after the ones needed (the copies of half step h-1, plus its weight loads when h is
    // odd) means they have arrived.
    typename Src::Tile w[2][RT];
    auto w_issue = [&](typename Src::Tile (&dst)[RT], int t) {
#pragma unroll
        for (int r = 0; r < RT; ++r)
            w_stream[r].issue(dst[r], t);
    };
    auto pin_tiles = [&](typename Src::Tile (&dst)[RT]) {
#pragma unroll
        for (int r = 0; r < RT; ++r)
            Src::pin_tile(dst[r]);
    };
    w_issue(w[0], 0);
#pragma unroll
    for (int i = 0; i < XS - 1; ++i)
        x_issue(i, i);
    // half tile 0 has to be visible before the ring is primed
    wait_loads<XPERH>();
    __syncthreads();
#pragma unroll
    for (int i = 0; i < LOOK; ++i)
        bq[i] = ldb(xs_dyn, i);
    const int n_half = 2 * n_steps;
    for (int h0 = 0; h0 < n_half; h0 += XS) {
        static_for<XS>([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            constexpr int hp = u & 1, xb = u % XS, ws = (u / 2) % 2;
            constexpr int n_after = hp == 1 ? XPERH + WLOADS : XPERH;
            const int h = h0 + u;
            if (h < n_half) {  // the same for every wave of the block
                wait_loads<n_after>();
                if (hp == 0)
                    pin_tiles(w[ws]);
                __syncthreads();
                if (hp == 0) {
#pragma unroll
                    for (int r = 0; r < RT; ++r)
                        Src::template fragments<0>(w[ws][r], a[0][0][r], a[0][1][r]);
                }
                // the requests of this half step, unit by unit (the weights of one row tile of k-tile t+1 when h
                // is even, then one activation copy of half tile h+3 each), unit k after step (k+1)*STEPS/(units+1)
                constexpr int W_UNITS = hp == 0 ? RT : 0, UNITS = W_UNITS + XPERH;
                compute_half(std::integral_constant<int, hp>{}, w[ws], xs_dyn + xb * XHPIECES,
                             xs_dyn + ((xb + 1) % XS) * XHPIECES, [&](auto st_c) {
                                 constexpr int st = decltype(st_c)::value;
                                 static_for<UNITS>([&](auto k_c) {
                                     constexpr int k = decltype(k_c)::value;
                                     if constexpr ((k + 1) * STEPS / (UNITS + 1) - 1 == st) {
                                         if constexpr (k < W_UNITS)
                                             w_stream[k].issue(w[ws ^ 1][k], (h >> 1) + 1);
                                         else
                                             x_issue_one(h + XS - 1, (xb + XS - 1) % XS, k - W_UNITS);
                                     }
                                 });
                             });
            }
        });
    }
    // the look-ahead requests (out of range: zeros) must land before the registers are reused and before
    // the block gives up its LDS
    wait_loads<0>();
    pin_tiles(w[0]);
    pin_tiles(w[1]);

    // ---- two k groups meet in LDS: group wk keeps row tile wk of the two
    constexpr int OWN = RT / WK;  // row tiles from here on
    float4_t own[OWN][NT];
    const int row_own = row_tile0 + (WK == 1 ? 0 : wk);
    if constexpr (WK == 2) {
        static_assert(WAVES * NT * 1024 <= XS * XHBYTES, "exchange buffer");
        float4_t *ex = reinterpret_cast<float4_t *>(xs_dyn);
        __syncthreads();
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            ex[(wave * NT + nt) * 64 + lane] = wk == 0 ? acc[1][nt] : acc[0][nt];
        __syncthreads();
        const int partner = wk == 0 ? wave + WM * WN : wave - WM * WN;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            own[0][nt] = (wk == 0 ? acc[0][nt] : acc[1][nt]) + ex[(partner * NT + nt) * 64 + lane];
    } else {
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                own[r][nt] = acc[r][nt];
    }

    // ---- epilogue.  Lane L holds, per (row tile, token tile), rows 4*(L/16)+i of token column L%16.
    const int n_in_tile = lane & 15;
    const int n_tiles_total = n_blocks * BNT;
    RowTerms terms[OWN];
    row_terms_of_tiles<Src::kHasScale, true>(terms, epi, scales, row_own * kTileRows, M, lane);

    if (S > 1) {
        // split-K: see linear_stream.hpp for the protocol (device-scope accesses, ordered sum), here with one arrival counter per
        // wave, so that no wave waits for its block before the hand-over
        // (8192 x 22016, N = 512 151.0 -> 148.4 us, N = 256 87.2 -> 85.9, 28672 x 8192, N = 128 66.1 -> 64.8)
        auto slice = [&](int s, int r) {  // the wave's NT tiles of row tile r
            return partial_buffer(partials + (((int64_t)s * n_row_tiles + (row_own + r)) * n_tiles_total + (n_block * WN + wn) * NT) * 64, NT * 1024);
        };
#pragma unroll
        for (int r = 0; r < OWN; ++r)
            if (row_own + r < n_row_tiles) {
                const partial_rsrc_t dst = slice(split, r);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    if (col0 + nt * 16 + n_in_tile < N)
                        agent_store(dst, nt * 1024 + lane * 16, own[r][nt]);
            }
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's partial stores are done
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        int *counter = counters + (((int64_t)row_block * n_blocks + n_block) * WAVES + wave) * counter_step;
        int arrived = 0;
        if (lane == 0)
            arrived = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        arrived = __builtin_amdgcn_readfirstlane(arrived);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        if (arrived != S - 1)
            return;
        if (lane == 0)
            *counter = 0;  // re-arm for the next call on this workspace
#pragma unroll
        for (int r = 0; r < OWN; ++r) {
            if (row_own + r >= n_row_tiles)
                continue;
            float4_t sum[NT];
            add_slices<NT >= 8 ? 2 : 4>(sum, S, split, [&](int nt) { return own[r][nt]; }, [&](float4_t (&part)[NT], int s) {
                const partial_rsrc_t src = slice(s, r);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    part[nt] = agent_load(src, nt * 1024 + lane * 16);
            });
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                own[r][nt] = sum[nt];
        }
    }
    finish_tiles<Src::kHasScale, true>(epi, terms, own, row_own * kTileRows, col0, M, N, Y, lane);
}

}  // namespace fp6
