// fp6_quantize_pack and fp6_unpack kernels for gfx950.
//
// quantize_pack: one pass over W finds the row maxima and the fp16 scales, rounds every weight to its code and writes
// whole tiles of the packed stream with 16-byte stores per lane and plane (the ahead-of-time re-layout
// of the paper's Section 5.2, in this library's order); for small matrices two launches, the maxima first.
//
// unpack: one wave per tile; the same register-level decode as the GEMM, followed by
// the row scale and a single rounding to fp16.
#pragma once
#include "fp6_device.hpp"

namespace fp6 {

typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));

// The row scale as the encoder needs it: the scale itself and its reciprocal (0 for a zero scale).
struct RowScale {
    float scale, inv;
};
__device__ __forceinline__ RowScale make_row_scale(float scale)
{
    RowScale r;
    r.scale = scale;
    r.inv = scale == 0.0f ? 0.0f : 1.0f / scale;
    return r;
}
// ... for the weights of runs F0 .. F0 + F - 1.  Infinities and NaN are not weights; a row that has them still gets one well-defined
// answer, the largest magnitude with the sign of each weight, which is not left to the conversions.
template <int F0, int F>
__device__ __forceinline__ RowScale row_scale_of(float scale, u32x4 (&v)[8])
{
    if (!(scale <= 65504.0f)) {
#pragma unroll
        for (int f = F0; f < F0 + F; ++f)
            v[f] = (v[f] & 0x80008000u) | 0x7bff7bffu;
        scale = 1.0f;
    }
    return make_row_scale(scale);
}

// w / scale with one Newton correction on top of the reciprocal product.  When the exact quotient is a
// grid midpoint m (the only case where the last bit matters), q = m(1+e), the fused remainder q*scale - w
// is exact and the corrected value m(1+O(e^2)) rounds to m itself; everywhere else the exact quotient is
// at least 2^-16 (relative) away from every midpoint, far more than the error of q.  So rounding the result to a
// grid (nearest, ties to even) rounds the exact quotient.  The sign of a zero is that of w, also for a zero scale.
__device__ __forceinline__ float ratio_of(half_t w, RowScale rs)
{
    const float a = (float)w, q = a * rs.inv;
    return __builtin_fmaf(-__builtin_fmaf(q, rs.scale, -a), rs.inv, q);
}

// ---- the weight formats as the encoder sees them ---------------------------------------------------
// encode<C>(): the lane's weights of runs 4C .. 4C+3 (run f, columns run*32 + 8q + j: half j of v[f]) -> its kHalfWords words
// of that half of the tile; store_tile() / store_half(): the lane's words -> its bytes of the tile.  6, 5 and 4 bits: the chip's
// conversions round to nearest, ties to the even code, saturate (5 bits: by hand) and keep the sign of a zero: every fp16 magnitude
// under 512 row maxima of all binades, ratios down to 2^-37 among them, gets the oracle's code (tests/test_gpu_pack_rounding.py; the
// quotient: tests/test_host_logic.py).  18 VALU instructions per weight before, 4 and a conversion now.
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef short short2_t __attribute__((ext_vector_type(2)));

struct E3M2Format {
    static constexpr float kMax = 28.0f;
    static constexpr int kTileBytes = 3072, kHalfWords = 6;
    static constexpr bool kHalfTiles = false;
    // a dense stream: code i = 8*(run%4) + j at bits [6i, 6i+6); the conversion takes even and odd codes apart
    template <int C>
    __device__ static __forceinline__ void encode(const u32x4 (&v)[8], RowScale rs, uint32_t (&d)[2 * kHalfWords])
    {
        float16_t even, odd;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const half2_t w = bit_cast<half2_t>(v[4 * C + i / 4][i % 4]);
            even[i] = ratio_of(w[0], rs);
            odd[i] = ratio_of(w[1], rs);
        }
        const u32x6 words = __builtin_amdgcn_cvt_scalef32_2xpk16_bf6_f32(even, odd, 1.0f);
#pragma unroll
        for (int i = 0; i < kHalfWords; ++i)
            d[C * kHalfWords + i] = words[i];
    }
    __device__ static __forceinline__ void store_tile(const uint32_t (&d)[2 * kHalfWords], uint8_t *tile, int lane)
    {
        u32x4 *t = reinterpret_cast<u32x4 *>(tile) + lane;
        t[0] = (u32x4){d[0], d[1], d[2], d[3]};
        t[64] = (u32x4){d[4], d[5], d[6], d[7]};
        t[128] = (u32x4){d[8], d[9], d[10], d[11]};
    }
};

// e2m2: grid 0 .25 .5 .75 | 1 .. 1.75 | 2 .. 3.5 | 4 .. 7 (Eq. 1 with bias 1, subnormal E = 0 binade).  Times 2^-14 that is the
// lower end of the e5m2 numbers, whose bytes "s 000 e1 e0 m1 m0" are what the layout stores in place.
struct E2M2Format {
    static constexpr float kMax = 7.0f;
    static constexpr int kTileBytes = 2560, kHalfWords = 5;
    static constexpr bool kHalfTiles = false;
    __device__ static __forceinline__ uint32_t four_bytes(uint32_t w01, uint32_t w23, RowScale rs)
    {
        float r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            r[i] = __builtin_amdgcn_fmed3f(ratio_of(bit_cast<half2_t>(i < 2 ? w01 : w23)[i % 2], rs), -kMax, kMax);
        short2_t b = {0, 0};
        b = __builtin_amdgcn_cvt_scalef32_pk_bf8_f32(b, r[0], r[1], 16384.0f, false);
        b = __builtin_amdgcn_cvt_scalef32_pk_bf8_f32(b, r[2], r[3], 16384.0f, true);
        return bit_cast<uint32_t>(b);
    }
    template <int C>
    __device__ static __forceinline__ void encode(const u32x4 (&v)[8], RowScale rs, uint32_t (&d)[2 * kHalfWords])
    {
        uint32_t b[8];  // codes 4i .. 4i+3 of the half, one byte each
#pragma unroll
        for (int i = 0; i < 8; ++i)
            b[i] = four_bytes(v[4 * C + i / 2][i % 2 * 2], v[4 * C + i / 2][i % 2 * 2 + 1], rs);
        // codes 0 .. 19 in place, the others in bits 6, 5, 4 of their bytes (fp6_device.hpp lists where)
        uint32_t *w = d + C * kHalfWords;
        w[0] = b[0] | ((b[5] >> 1) & 0x40404040u) | ((b[5] << 2) & 0x30303030u);
        w[1] = b[1] | ((b[5] << 5) & 0x60606060u) | ((b[6] >> 3) & 0x10101010u);
        w[2] = b[2] | ((b[6] << 3) & 0x70707070u);
        w[3] = b[3] | ((b[6] << 6) & 0x40404040u) | ((b[7] >> 2) & 0x20202020u) | ((b[7] << 1) & 0x10101010u);
        w[4] = b[4] | ((b[7] << 4) & 0x70707070u);
    }
    __device__ static __forceinline__ void store_tile(const uint32_t (&d)[2 * kHalfWords], uint8_t *tile, int lane)
    {
        u32x4 *t = reinterpret_cast<u32x4 *>(tile) + lane;
        t[0] = (u32x4){d[0], d[1], d[2], d[3]};
        t[64] = (u32x4){d[4], d[5], d[6], d[7]};
        reinterpret_cast<u32x2 *>(tile + 2048)[lane] = (u32x2){d[8], d[9]};
    }
};

// e2m1: grid 0 .5 | 1 1.5 | 2 3 | 4 6 (Eq. 1 with bias 1, subnormal E = 0 binade).
struct E2M1Format {
    static constexpr float kMax = 6.0f;
    static constexpr int kTileBytes = 2048, kHalfWords = 4;
    static constexpr bool kHalfTiles = false;
    template <int C>
    __device__ static __forceinline__ void encode(const u32x4 (&v)[8], RowScale rs, uint32_t (&d)[2 * kHalfWords])
    {
#pragma unroll
        for (int run = 0; run < 4; ++run) {
            const u32x4 &p = v[4 * C + run];
            uint32_t w = 0;
            static_for<4>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                const half2_t h = bit_cast<half2_t>(p[j]);
                w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, ratio_of(h[0], rs), ratio_of(h[1], rs), 1.0f, j);
            });
            d[C * kHalfWords + run] = w;
        }
    }
    __device__ static __forceinline__ void store_tile(const uint32_t (&d)[2 * kHalfWords], uint8_t *tile, int lane)
    {
        u32x4 *t = reinterpret_cast<u32x4 *>(tile) + lane;
        t[0] = (u32x4){d[0], d[1], d[2], d[3]};
        t[64] = (u32x4){d[4], d[5], d[6], d[7]};
    }
};

// e2m0: grid 0 | 1 | 2 | 4 (Eq. 1 with bias 1 and no mantissa bits; the E = 0 binade holds only 0).  No conversion of the chip
// rounds to it.
struct E2M0Format {
    static constexpr float kMax = 4.0f;
    static constexpr int kTileBytes = 3072;       // 16 rows x 512 columns: k-tile kt (256 columns) is half kt % 2 of tile kt / 2
    static constexpr int kHalfWords = 3;
    static constexpr bool kHalfTiles = true;
    // code s e1 e0: the midpoints 0.5, 1.5 and 3 go to the even codes 0, 2 and 2
    __device__ static __forceinline__ uint32_t code_of(half_t w, RowScale rs)
    {
        const float ratio = ratio_of(w, rs), a = __builtin_fabsf(ratio);
        uint32_t g = bit_cast<uint32_t>(ratio) >> 31 << 2;
        g += a > 0.5f;
        g += a >= 1.5f;
        g += a > 3.0f;
        return g;
    }
    template <int C>
    __device__ static __forceinline__ void encode(const u32x4 (&v)[8], RowScale rs, uint32_t (&d)[2 * kHalfWords])
    {
        uint32_t w[4] = {0, 0, 0, 0};  // codes of a run, four bits each
#pragma unroll
        for (int run = 0; run < 4; ++run) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                w[run] |= code_of(bit_cast<half2_t>(v[4 * C + run][j / 2])[j % 2], rs) << (4 * j);
            __builtin_amdgcn_sched_barrier(0);  // run by run: fewer registers
        }
        // runs 0 .. 2 in place, field "s e1 e0 .", run 3 spread over the free bits
#pragma unroll
        for (int i = 0; i < 3; ++i)
            d[C * kHalfWords + i] = w[i] << 1 | ((w[3] >> i) & 0x11111111u);
    }
    // the lane's bytes of one half of a tile: 16 in plane 0 (first half) or 2 (second half), 8 in the middle
    // plane; pad_other: the matrix ends with this half (K an odd multiple of 256) and the lane also writes the
    // zero padding of the other half
    __device__ static __forceinline__ void store_half(const uint32_t (&d)[2 * kHalfWords], uint8_t *tile, int half, bool pad_other,
                                                      int lane)
    {
        *(reinterpret_cast<u32x4 *>(tile + half * 2048) + lane) = (u32x4){d[0], d[1], d[2], d[3]};
        *(reinterpret_cast<u32x2 *>(tile + 1024) + 2 * lane + half) = (u32x2){d[4], d[5]};
        if (pad_other) {
            *(reinterpret_cast<u32x4 *>(tile + (half ^ 1) * 2048) + lane) = (u32x4){0, 0, 0, 0};
            *(reinterpret_cast<u32x2 *>(tile + 1024) + 2 * lane + (half ^ 1)) = (u32x2){0, 0};
        }
    }
};

// The lane's words of k-tile kt (256 columns) of row tile `row_tile` into the packed stream (tiles stored
// k-tile major; RT row tiles, KT k-tiles of 256 columns).
template <class Fmt>
__device__ __forceinline__ void store_k_tile(const uint32_t (&d)[2 * Fmt::kHalfWords], uint8_t *packed, int64_t kt, int64_t row_tile, int64_t RT, int KT,
                                             int lane)
{
    if constexpr (Fmt::kHalfTiles)
        Fmt::store_half(d, packed + ((kt >> 1) * RT + row_tile) * Fmt::kTileBytes, (int)(kt & 1), (kt & 1) == 0 && kt == KT - 1, lane);
    else
        Fmt::store_tile(d, packed + (kt * RT + row_tile) * Fmt::kTileBytes, lane);
}

// ---- per-row scales, small matrices: two launches ---------------------------------------------------
// row_scale_kernel: one wave per row finds max |W| and writes scale = fp16(max / Fmt::kMax) (a plain read of
// W at streaming rate).  quantize_tiles_kernel: one wave per 16 x 256 tile reads the tile once, rounds every
// weight with its row's scale and writes the packed tile.  The scales array is the only thing that passes
// between the two; W is read twice.
constexpr int kScaleWavesPerBlock = 4;

template <class Fmt>
__global__ __launch_bounds__(kScaleWavesPerBlock * 64) void row_scale_kernel(const half_t *__restrict__ W, int M, int K,
                                                                              half_t *__restrict__ scales)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = blockIdx.x * kScaleWavesPerBlock + wave;
    if (m >= M)
        return;
    const u32x4 *row = reinterpret_cast<const u32x4 *>(W + (int64_t)m * K);
    const int n16 = K / 8;  // 16-byte pieces of the row (K % 256 == 0, so n16 % 32 == 0)
    ushort2_t mx = {0, 0};
    int i = lane;
    for (; i + 448 < n16; i += 512) {  // eight independent loads in flight
        u32x4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            v[u] = __builtin_nontemporal_load(row + i + 64 * u);
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                mx = __builtin_elementwise_max(mx, bit_cast<ushort2_t>(v[u][j] & 0x7fff7fffu));
    }
    for (; i < n16; i += 64) {
        const u32x4 v = row[i];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            mx = __builtin_elementwise_max(mx, bit_cast<ushort2_t>(v[j] & 0x7fff7fffu));
    }
    uint32_t amax = mx[0] > mx[1] ? mx[0] : mx[1];  // finite fp16 magnitudes order like integers
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t other = __shfl_xor(amax, off, 64);
        amax = other > amax ? other : amax;
    }
    if (lane == 0)
        scales[m] = (half_t)((float)bit_cast<half_t>((uint16_t)amax) / Fmt::kMax);  // fp32 quotient, one rounding
}

template <class Fmt>
__global__ __launch_bounds__(256) void quantize_tiles_kernel(const half_t *__restrict__ W, int M, int K,
                                                             uint8_t *__restrict__ packed,
                                                             const half_t *__restrict__ scales)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int KT = K / kTileK;
    const int64_t tile = (int64_t)blockIdx.x * 4 + wave;
    if (tile >= (int64_t)(M / kTileRows) * KT)
        return;
    // the waves of a block take neighbouring k-tiles of one row tile (2 KB of every row of W between them);
    // in the packed stream tiles are stored k-tile major
    const int64_t RT = M / kTileRows, row_tile = tile / KT, kt = tile % KT;
    const int r = lane & 15, q = lane >> 4;  // lane (r, q) builds its bytes of the tile
    const half_t *row = W + (row_tile * kTileRows + r) * K + kt * kTileK + q * 8;
    u32x4 v[8];
#pragma unroll
    for (int f = 0; f < 8; ++f)
        v[f] = *reinterpret_cast<const u32x4 *>(row + f * 32);
    const RowScale scale = row_scale_of<0, 8>((float)scales[row_tile * kTileRows + r], v);
    uint32_t d[2 * Fmt::kHalfWords];
    Fmt::template encode<0>(v, scale, d);
    Fmt::template encode<1>(v, scale, d);
    store_k_tile<Fmt>(d, packed, kt, row_tile, RT, KT, lane);
}

// ---- per-row scales, one pass over W -----------------------------------------------------------------
// A block of four waves holds 16 rows x 1024 columns in registers (a part of a row tile; one k-tile per wave), and the parts
// of a row tile agree on the row maxima through memory: W is read once.  Each block raises the sixteen maxima with atomics, counts
// itself as arrived, waits until all parts have, and reads them back.  Bound by memory: 361 MB read + 135 MB written for 8192 x
// 22016 in 115 us (4.3 TB/s) against 145 in two launches; 57344 x 8192 377 -> 241, 4096 x 4096 15.5 -> 14.4, 4 bits 8192 x 22016
// 129 -> 103.  Five or six blocks per CU cover the exchange; eight (64 registers, some spilled) gain nothing.  The parts of a row
// tile follow one another in the grid, that is on different XCDs: all on one XCD 163 us.  Non-temporal loads 121.
//   The exchange happens in the first 128 bytes of the row tile's first packed tile: cleared by a launch of their own, written
// over by whichever block is the last to have read the maxima (it fetches k-tile 0 again).  So nothing is waited for but
// arrivals, and that wait is bounded: a block that has polled max_polls times reads its sixteen rows itself, and raises the maxima and
// the arrival word for the parts that have not started yet, which then neither wait nor read.  (In a launch alone on the chip the wait
// ends without that: blocks start in order on each XCD, so the earliest unfinished row tile always finds room for its parts.)  The
// bound is four times what was needed: 8192 x 22016, 0 / 16 / 32 / 64 polls 860 / 117 / 113 / 113 us alone, 1060 / 890 / 500-850 / 298 beside
// 57344 x 8192, N = 4096 on another stream, 980 / 770 / 240-750 / 245 beside 8192 x 22016, N = 512, 910 / 206 / 160 / 131 beside N = 16; more
// polls change nothing (two launches, W read twice: 160 alone, 515, 420 and 203).
constexpr int kPartWaves = 4, kMaxParts = 40, kPartWaitPolls = 256;
constexpr int kExchangeBytes = 128, kArrivedWord = 16, kReadWord = 17;  // words 0 .. 15: the maxima
constexpr uint32_t kMaximaComplete = 1u << 16;  // in the arrival word: more than any number of parts

__global__ __launch_bounds__(256) void clear_exchange_kernel(uint8_t *packed, int row_tiles, int tile_bytes)
{
    constexpr int kPieces = kExchangeBytes / 16;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i / kPieces < row_tiles)
        *reinterpret_cast<u32x4 *>(packed + (int64_t)(i / kPieces) * tile_bytes + i % kPieces * 16) = (u32x4){0u, 0u, 0u, 0u};
}

// the lane's share of a 16 x 256 tile: eight runs of 32 columns
__device__ __forceinline__ void load_weights(u32x4 (&v)[8], const half_t *p)
{
#pragma unroll
    for (int f = 0; f < 8; ++f)
        v[f] = *reinterpret_cast<const u32x4 *>(p + f * 32);
}
// largest magnitude of the lane's values, as bits: finite fp16 magnitudes order like integers
__device__ __forceinline__ uint32_t magnitude_max(const u32x4 (&v)[8])
{
    ushort2_t mx = {0, 0};
#pragma unroll
    for (int f = 0; f < 8; ++f)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            mx = __builtin_elementwise_max(mx, bit_cast<ushort2_t>(v[f][j] & 0x7fff7fffu));
    return mx[0] > mx[1] ? mx[0] : mx[1];
}
// ... of the four lanes that share a row
__device__ __forceinline__ uint32_t row_of_tile_max(uint32_t amax)
{
#pragma unroll
    for (int off = 16; off < 64; off <<= 1) {
        const uint32_t other = __shfl_xor(amax, off, 64);
        amax = other > amax ? other : amax;
    }
    return amax;
}

template <class Fmt>
__global__ __launch_bounds__(kPartWaves * 64) void quantize_rows_kernel(const half_t *__restrict__ W, int M, int K, uint8_t *packed,
                                                                        half_t *__restrict__ scales, int parts, int max_polls)
{
    static_assert(kMaxParts < (int)kMaximaComplete && Fmt::kTileBytes % kExchangeBytes == 0 && kExchangeBytes <= 1024, "the exchange lies in the first plane of a tile");
    __shared__ uint32_t part_max[kPartWaves][16], row_max[16], last_reader;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int KT = K / kTileK, RT = M / kTileRows;
    const int row_tile = blockIdx.x / parts, part = blockIdx.x % parts;
    const int kt = part * kPartWaves + wave;
    const int r = lane & 15, q = lane >> 4;
    const half_t *row = W + ((int64_t)row_tile * kTileRows + r) * K + q * 8;
    u32x4 v[8];
    load_weights(v, row + (kt < KT ? kt : KT - 1) * kTileK);  // waves past the last k-tile repeat it
    const uint32_t tile_max = row_of_tile_max(magnitude_max(v));
    if (lane < 16)
        part_max[wave][lane] = tile_max;
    __syncthreads();
    if (wave == 0) {
        uint32_t m = 0;
#pragma unroll
        for (int w = 0; w < kPartWaves; ++w)
            m = part_max[w][r] > m ? part_max[w][r] : m;
        bool last = true;
        if (parts > 1) {
            // order: this part's maxima are in memory (vmcnt) -> its arrival; all arrivals -> the maxima are read -> this part has
            // read them.  Accesses of agent scope, as in the split-K hand-over (linear_stream.hpp).
            uint32_t *line = reinterpret_cast<uint32_t *>(packed + (int64_t)row_tile * Fmt::kTileBytes);
            if (lane < 16)
                __hip_atomic_fetch_max(line + lane, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            int arrived = 0;
            if (lane == 0)
                arrived = (int)__hip_atomic_fetch_add(line + kArrivedWord, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
            arrived = __builtin_amdgcn_readfirstlane(arrived);
            for (int i = 0; arrived < parts && i < max_polls; ++i) {
                __builtin_amdgcn_s_sleep(1);
                arrived = __builtin_amdgcn_readfirstlane((int)__hip_atomic_load(line + kArrivedWord, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            }
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            if (arrived >= parts) {
                m = __hip_atomic_load(line + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                m = 0;
                for (int t = 0; t < KT; ++t) {
                    u32x4 other[8];
                    load_weights(other, row + t * kTileK);
                    const uint32_t x = magnitude_max(other);
                    m = x > m ? x : m;
                }
                m = row_of_tile_max(m);
                if (lane < 16)
                    __hip_atomic_fetch_max(line + lane, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
                __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): before the word that says so
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
                if (lane == 0)
                    __hip_atomic_fetch_or(line + kArrivedWord, kMaximaComplete, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): the maxima have been read
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            uint32_t readers = 0;
            if (lane == 0)
                readers = __hip_atomic_fetch_add(line + kReadWord, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
            last = __builtin_amdgcn_readfirstlane((int)readers) == parts;
        }
        if (lane < 16)
            row_max[lane] = m;
        if (lane == 0)
            last_reader = last ? 1u : 0u;
    }
    __syncthreads();
    const half_t sc = (half_t)((float)bit_cast<half_t>((uint16_t)row_max[r]) / Fmt::kMax);  // fp32 quotient, one rounding
    if (part == 0 && wave == 0 && lane < 16)
        scales[row_tile * kTileRows + lane] = sc;
    RowScale scale = row_scale_of<0, 8>((float)sc, v);
    uint32_t d[2 * Fmt::kHalfWords];
    if (kt < KT && (kt > 0 || parts == 1)) {
        Fmt::template encode<0>(v, scale, d);
        Fmt::template encode<1>(v, scale, d);
        store_k_tile<Fmt>(d, packed, kt, row_tile, RT, KT, lane);
    }
    if (parts > 1 && wave == 0 && last_reader) {
        load_weights(v, row);
        scale = row_scale_of<0, 8>((float)sc, v);
        Fmt::template encode<0>(v, scale, d);
        Fmt::template encode<1>(v, scale, d);
        store_k_tile<Fmt>(d, packed, 0, row_tile, RT, KT, lane);
    }
}

// Group-wise scales (one per row and per 128 columns): a group lies inside one tile and inside one of a
// lane's two streams, so row maxima need only a reduction over the four lanes (q = 0..3) that share a row:
// one pass over W, one wave per tile.  scales: fp16 [M][K/128].
__global__ __launch_bounds__(256) void quantize_pack_group_kernel(const half_t *__restrict__ W, int M, int K,
                                                                  uint8_t *__restrict__ packed,
                                                                  half_t *__restrict__ scales)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int KT = K / kTileK;
    const int64_t tile = (int64_t)blockIdx.x * 4 + wave;
    if (tile >= (int64_t)(M / kTileRows) * KT)
        return;
    // the waves of a block take neighbouring k-tiles of one row tile (2 KB of every row of W between them);
    // in the packed stream tiles are stored k-tile major
    const int64_t RT = M / kTileRows, row_tile = tile / KT, kt = tile % KT, packed_tile = kt * RT + row_tile;
    const int r = lane & 15, q = lane >> 4;
    const half_t *row = W + (row_tile * kTileRows + r) * K + kt * kTileK + q * 8;
    u32x4 v[8];
#pragma unroll
    for (int f = 0; f < 8; ++f)
        v[f] = *reinterpret_cast<const u32x4 *>(row + f * 32);
    uint32_t d[2 * E3M2Format::kHalfWords];
    uint32_t scale_bits[2];
    static_for<2>([&](auto cc) {
        constexpr int c = decltype(cc)::value;
        ushort2_t mx = {0, 0};
#pragma unroll
        for (int f = 4 * c; f < 4 * c + 4; ++f)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                mx = __builtin_elementwise_max(mx, bit_cast<ushort2_t>(v[f][j] & 0x7fff7fffu));
        uint32_t amax = mx[0] > mx[1] ? mx[0] : mx[1];  // finite fp16 magnitudes order like integers
#pragma unroll
        for (int off = 16; off < 64; off <<= 1) {        // the four lanes of a row
            const uint32_t other = __shfl_xor(amax, off, 64);
            amax = other > amax ? other : amax;
        }
        const half_t sc = (half_t)((float)bit_cast<half_t>((uint16_t)amax) / E3M2Format::kMax);
        scale_bits[c] = bit_cast<uint16_t>(sc);
        const RowScale scale = row_scale_of<4 * c, 4>((float)sc, v);
        E3M2Format::encode<c>(v, scale, d);
    });
    E3M2Format::store_tile(d, packed + packed_tile * E3M2Format::kTileBytes, lane);
    if (q == 0) {
        const int64_t groups = K / kGroupColumns;
        *reinterpret_cast<uint32_t *>(scales + (row_tile * kTileRows + r) * groups + 2 * kt) = scale_bits[0] | (scale_bits[1] << 16);
    }
}

template <class Src>
__global__ __launch_bounds__(256) void unpack_kernel(const uint8_t *__restrict__ packed,
                                                     const half_t *__restrict__ scales, int M, int K,
                                                     half_t *__restrict__ W_out)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int KT = K / kTileK;
    const int64_t tile = (int64_t)blockIdx.x * 4 + wave;
    if (tile >= (int64_t)(M / kTileRows) * KT)
        return;
    // the waves of a block take neighbouring k-tiles of one row tile (2 KB of every row of W between them);
    // in the packed stream tiles are stored k-tile major
    const int64_t RT = M / kTileRows, row_tile = tile / KT, kt = tile % KT;
    const int r = lane & 15, q = lane >> 4;
    typename Src::Stream stream;
    stream.init(packed, scales, row_tile, (int)kt, 1, 1, RT, K, lane);
    typename Src::Tile t;
    stream.issue(t, 0);
    wait_loads<0>();
    Src::pin_tile(t);
    const float scale = Src::kHasScale ? (float)scales[row_tile * kTileRows + r] : 1.0f;  // else already applied
    half_t *out = W_out + (row_tile * kTileRows + r) * K + kt * kTileK + q * 8;
    half8_t frag[8];
    Src::template fragments<0>(t, frag[0], frag[1]);
    Src::template fragments<1>(t, frag[2], frag[3]);
    Src::template fragments<2>(t, frag[4], frag[5]);
    Src::template fragments<3>(t, frag[6], frag[7]);
#pragma unroll
    for (int f = 0; f < 8; ++f) {
        half8_t y;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            y[j] = (half_t)((float)frag[f][j] * scale);  // exact product in fp32, one rounding
        *reinterpret_cast<half8_t *>(out + f * 32) = y;
    }
}

// ---- diagnostics: empirical ceilings of the device, with the request patterns of the linear kernels ------
// probe_read_kernel: the buffer is cut into pieces of 8 KB; in step s wave w of the W waves reads piece
// s * W + w, so that the grid sweeps the buffer front to back (the way the linear kernels sweep packed
// weights; one contiguous range per wave is 10 % slower), with the non-temporal 128-bit loads of the weight
// path, sixteen in flight per wave (two sets of eight).  Nothing is computed except the XOR of what was loaded.
__global__ __launch_bounds__(256) void probe_read_kernel(const uint8_t *__restrict__ buffer, size_t bytes,
                                                         uint32_t *__restrict__ sink)
{
    const int lane = threadIdx.x & 63;
    const size_t wave = (size_t)blockIdx.x * 4 + (size_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const size_t n_waves = (size_t)gridDim.x * 4;
    const size_t steps = bytes / (n_waves * 8192) / 2 * 2;  // whole double steps; the host sizes the grid for >= 2
    u32x4 a[8], b[8];
    auto issue8 = [&](u32x4 (&v)[8], size_t step) {
        // a step past the end gets an empty range: its loads return zeros and fetch nothing
        const rsrc_t r = make_rsrc(buffer + (step < steps ? step * n_waves + wave : 0) * 8192, step < steps ? 8192u : 0u);
        const int off = lane * 16;
        v[0] = issue_load_b128<0, true>(r, off);
        v[1] = issue_load_b128<1024, true>(r, off);
        v[2] = issue_load_b128<2048, true>(r, off);
        v[3] = issue_load_b128<3072, true>(r, off);
        v[4] = issue_load_b128<0, true>(r, off + 4096);  // the immediate offset is a 12-bit field
        v[5] = issue_load_b128<1024, true>(r, off + 4096);
        v[6] = issue_load_b128<2048, true>(r, off + 4096);
        v[7] = issue_load_b128<3072, true>(r, off + 4096);
    };
    u32x4 x = {0u, 0u, 0u, 0u};  // running XOR of everything loaded: the data is touched, and checkable
    auto pin8 = [&](u32x4 (&v)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            pin(v[i]);
            x ^= v[i];
        }
        pin(x);  // the set is consumed here, before its registers are the target of the next loads
    };
    issue8(a, 0);
    for (size_t s = 0; s < steps; s += 2) {
        issue8(b, s + 1);
        wait_loads<8>();
        pin8(a);
        issue8(a, s + 2);
        wait_loads<8>();
        pin8(b);
    }
    wait_loads<0>();
    pin8(a);  // the look-ahead past the last step: zeros
    uint32_t w = x[0] ^ x[1] ^ x[2] ^ x[3];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1)
        w ^= (uint32_t)__shfl_xor((int)w, m, 64);
    if (lane == 0)
        sink[wave] = w;  // XOR of all 32-bit words of the wave's pieces
}

// probe_mfma_kernel: every wave issues iters x 4 independent v_mfma_f32_32x32x16_f16 on register operands.
__global__ __launch_bounds__(256) void probe_mfma_kernel(int iters, float *__restrict__ sink)
{
    const half_t one = (half_t)1.0f, tiny = (half_t)0.0009765625f;
    half8_t a = {one, tiny, one, tiny, one, tiny, one, tiny}, b = {tiny, one, tiny, one, tiny, one, tiny, one};
    float16_t acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j)
            acc[i][j] = (float)(i + j);
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, acc[i], 0, 0, 0);
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j)
            s += acc[i][j];
    sink[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = s;
}

__global__ void zero_fill_kernel(u32x4 *p, size_t n16)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n16)
        p[i] = (u32x4){0u, 0u, 0u, 0u};
}

}  // namespace fp6
