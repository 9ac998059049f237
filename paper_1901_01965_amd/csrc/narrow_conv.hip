// The whole hot path for layers with at most four input channels (a network's first layer),
// channels-last.  With so few channels the 64-deep reduction of the int8 matrix-core instructions would run
// nearly empty.  The products (Section 3.4: 16 real and 10 complex per tile and channel pair) are taken four channels deep
// instead, by `v_mfma_f32_4x4x4_16b_f16`, whose sixteen 4 x 4 blocks are laid out as 16 tiles x 16 filters.  This is integer
// arithmetic all the same: a transformed activation or filter is an integer of at most 2048 in magnitude, which a half holds
// exactly (no limb split, Section 3.1 is not needed), and a channel sum one of at most 2^24 (scaled mode 2^21), which a
// float holds exactly, as it does every partial sum of it.
//
// A workgroup of four waves takes 64 filters and up to kNarrowGroups x 16 tiles (chosen on the host so that the compute units
// finish together).  Phase 1: lane = (tile, two channels); the lane loads its 6x6 patch (all channels packed in one dword per
// pixel), runs the input transform of Section 3.3 in packed halves and leaves the 36 real numbers of the 26 free entries in
// LDS.  Phase 2: a wave holds its 16 filters' Winograd-domain numbers (from the blob's narrow table) in registers and walks
// over the groups of 16 tiles: channel sums, reverse scaling of Section 4.2 in scaled mode, output transform, and the
// outputs, int8 ones through LDS so that 64 filters of a pixel are stored together.
//
// It is bound by the vector ALU: per 16 tiles and a wave's 16 filters some 800 instructions (lossless 660), the reverse scaling (two
// for each of a lane's 144 sums) and the output transform (about 90 per tile) most of them.  Against narrow_wave_kernel, which needs
// twice as many (us, int8 outputs, 224x224x3 -> 64): N = 1 10.7 -> 7.9 scaled, 7.8 -> 7.1 lossless; N = 16 52.6 -> 38.1, 43.2 -> 34.2; N = 32 116.7 ->
// 62.7, 90.6 -> 54.4 (103 MB of outputs).
//
// narrow_wave_kernel has the layers of few tiles, and of filter counts that cannot be stored four at a time: a wave is a workgroup, lane = tile in the
// transform, then lane = filter, and one `v_dot2_i32_i16` multiplies two channels at a time.
#include "kernel_common.h"
#include "output_transform_core.h"
#include "wg_internal.h"
#include "write_through.h"

#include <algorithm>
#include <atomic>

namespace wg {
namespace {

constexpr int kWaveTiles = 32;                     // most tiles a wave takes (narrow_wave_kernel)
constexpr int kNarrowGroups = 7;                   // most groups of 16 tiles a workgroup takes: two workgroups' LDS fit a compute unit
constexpr int kNarrowPieces = kNarrowValues / 2;   // 16-byte pieces per tile or filter: two values x four channels
constexpr int kTileValuesBytes = 16 * kNarrowPieces + 16;   // in LDS; the 16 bytes keep sixteen tiles' pieces in different banks
constexpr int kStagedTileBytes = 16 * 64 + 16;     // 16 pixels x 64 filters of int8 outputs; four tiles apart is sixteen banks
constexpr int kStagedGroupBytes = 16 * kStagedTileBytes;

typedef _Float16 h16x4 __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// What makes it exact.  The 1-D rules' sums of |coefficients|, rows 0, 1, 2 and 5, and the real and imaginary part of row 3; two of them
// make an entry of 128 times their product.
constexpr int kActReach[4] = {2, 4, 4, 2}, kActRe = 2, kActIm = 2;          // B^T
constexpr int kFilterReach[4] = {4, 3, 3, 4}, kFilterRe = 2, kFilterIm = 1;   // 4 G
constexpr int largest_value() {
    int most = 0;
    for (int r = 0; r < 4; ++r)
        for (int c = 0; c < 4; ++c) most = std::max({most, kActReach[r] * kActReach[c], kFilterReach[r] * kFilterReach[c]});
    return 128 * std::max({most, kActRe * kActRe + kActIm * kActIm, kFilterRe * kFilterRe + kFilterIm * kFilterIm});   // (the other parts are smaller)
}
constexpr int largest_sum() {   // lossless; scaled filters are smaller
    int most = 0;
    for (int r = 0; r < 4; ++r) {
        const int row = kActReach[r] * kFilterReach[r];
        for (int c = 0; c < 4; ++c) most = std::max(most, row * kActReach[c] * kFilterReach[c]);
        most = std::max(most, row * (kActRe * kFilterRe + kActIm * kFilterIm));
    }
    const int act = kActRe * kActRe + kActIm * kActIm;   // either part of an entry of two complex rows
    most = std::max(most, act * (kFilterRe * kFilterRe + kFilterIm * kFilterIm) + act * 2 * kFilterRe * kFilterIm);
    return kNarrowChannels * 128 * 128 * most;
}
static_assert(largest_value() <= 2048, "transformed activations and filters are integers that a half holds");
static_assert(largest_sum() <= 1 << 24, "a float holds every channel sum, and every partial sum of it");

// ---- narrow_wave_kernel's pieces
// Receives the free entries from the input transform: value index = real entry p, or
// 16 + 2j (Re) and 17 + 2j (Im) of complex entry j, the order of the blob's narrow table.
struct QuadKeeper {
    Quad* v;
    __device__ inline void real_entry(int p, Quad q) const { v[p] = q; }
    __device__ inline void complex_entry(int j, Quad re, Quad im) const {
        v[16 + 2 * j] = re;
        v[17 + 2 * j] = im;
    }
};

// sum over the four channel slots of a (16-bit) x b (16-bit)
__device__ inline int dot4(uint32_t a01, uint32_t a23, uint32_t b01, uint32_t b23, int acc = 0) {
    return __builtin_amdgcn_sdot2(as_s16x2(a01), as_s16x2(b01), __builtin_amdgcn_sdot2(as_s16x2(a23), as_s16x2(b23), acc, false),
                                  false);
}

// Receives the free entries of two channels from the input transform: value index = real entry p, or
// 16 + 2j (Re) and 17 + 2j (Im) of complex entry j, the order of the blob's narrow table.
struct ValueKeeper {
    int8_t* base;   // of the tile's values, this pair of channels
    __device__ inline void put(int value, h16x2 v) const { *reinterpret_cast<uint32_t*>(base + 8 * value) = __builtin_bit_cast(uint32_t, v); }
    __device__ inline void real_entry(int p, h16x2 v) const { put(p, v); }
    __device__ inline void complex_entry(int j, h16x2 re, h16x2 im) const {
        put(16 + 2 * j, re);
        put(17 + 2 * j, im);
    }
};

// The 6x6 patch of tile (n, ty, tx), a pixel's C <= 4 channels in the low bytes of u[a][b], zeros above them: one unaligned
// dword per pixel.  It also brings what follows the pixel, which is masked off; where that lies beyond the tensor (a branch
// of the whole wave, near the tensor's end) the load begins earlier and is shifted.  A pixel's bytes one by one were four
// times the loads, 16 clocks each in the compute unit's memory path (one 224x224x3 image, 64 filters, lossless: 16.1 us instead of 8.9).
// Pixels outside the image are clamped into it (bias_patch replaces them).
__device__ inline void load_narrow_patch(const int8_t* __restrict__ x, const Problem& p, int n, int ty, int tx, uint32_t (&u)[6][6]) {
    const uint32_t total = (uint32_t)p.N * (uint32_t)p.H * (uint32_t)p.W * (uint32_t)p.C;
    if (total < 4) {
        load_patch<WG_NHWC, false>(x, p, n, ty, tx, 0, u);
        return;
    }
    uint32_t row_off[6], col_off[6];
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        row_off[a] = ((uint32_t)n * (uint32_t)p.H + (uint32_t)min(max(4 * ty - 1 + a, 0), p.H - 1)) * (uint32_t)p.W * (uint32_t)p.C;
        col_off[a] = (uint32_t)min(max(4 * tx - 1 + a, 0), p.W - 1) * (uint32_t)p.C;
    }
    const uint32_t channels = 0xffffffffu >> (32 - 8 * p.C);
    auto dword = [&](uint32_t at) {
        uint32_t v;
        __builtin_memcpy(&v, x + at, 4);
        return v;
    };
    if (__ballot(row_off[5] + col_off[5] > total - 4) == 0) {
#pragma unroll
        for (int i = 0; i < 36; ++i) u[i / 6][i % 6] = dword(row_off[i / 6] + col_off[i % 6]);
    } else {
#pragma unroll
        for (int i = 0; i < 36; ++i) {
            const uint32_t at = row_off[i / 6] + col_off[i % 6], from = min(at, total - 4);
            u[i / 6][i % 6] = dword(from) >> (8 * (at - from));
        }
    }
#pragma unroll
    for (int i = 0; i < 36; ++i) u[i / 6][i % 6] &= channels;
}

// The int8 epilogue on the output transform's 16 Y (before its rescale by 2^-4): the two nested
// floor divisions ((Y + rnd) >> 4, then (. + round) >> shift) are one, floor((Y + rnd + 16 round) /
// 2^(4 + shift)); then the clamp to [lo, 127].
// `add` = rnd + 16 round is in y16 already.
__device__ inline int requantise_y16(int y16, int shift, int lo, int most) {
    int v;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(v) : "v"(y16 >> shift), "s"(lo), "v"(most));
    return v;
}

// grid: (ceil(T/tiles_per_wave), Kp/64), 64 threads.
template <int MODE, bool Q8>
__global__ __launch_bounds__(64) void narrow_wave_kernel(const int8_t* __restrict__ x, WG_GEOMETRY_PARAMS, int tiles_per_wave,
                                                         const uint8_t* __restrict__ blob,
                                                         size_t table_off, size_t narrow_off, int32_t* __restrict__ y,
                                                         Problem p, Int8Epilogue q8) {
    WG_TAKE_GEOMETRY(p, 2);
    __shared__ uint4 values[kNarrowPieces * kWaveTiles];   // [piece][tile]
    const int lane = threadIdx.x;
    const int tile0 = blockIdx.x * tiles_per_wave;
    const BlobHeaderWords header = read_blob_header(blob);   // requested here, compared once the patch is on its way

    // ---- phase 1: lane = tile -----------------------------------------------------------------
    int my_n = 0, my_ty = 0, my_tx = 0;
    if (tile0 + lane < p.T) decode_tile(p, tile0 + lane, my_n, my_ty, my_tx);   // else tile (0,0,0): loaded, never used
    uint32_t u[6][6];
    if (lane < tiles_per_wave) load_narrow_patch(x, p, my_n, my_ty, my_tx, u);
    if (!blob_matches(header, p.K, p.C, MODE)) return;
    if (lane < tiles_per_wave) {
        bias_patch(p, my_ty, my_tx, 0, u);
        Quad v[kNarrowValues];
        transform_patch<ChannelPairs>(u, QuadKeeper{v});
#pragma unroll
        for (int i = 0; i < kNarrowPieces; ++i)
            values[i * kWaveTiles + lane] =
                make_uint4(as_u32(v[2 * i].a), as_u32(v[2 * i].b), as_u32(v[2 * i + 1].a), as_u32(v[2 * i + 1].b));
    }

    // ---- phase 2: lane = filter ----------------------------------------------------------------
    const int k = blockIdx.y * 64 + lane;   // < Kp: the blob's tables are padded to Kp
    uint4 w[kNarrowPieces];
    {
        const uint4* mine = reinterpret_cast<const uint4*>(blob + narrow_off) + (size_t)k * kNarrowPieces;
#pragma unroll
        for (int i = 0; i < kNarrowPieces; ++i) w[i] = mine[i];
    }
    // reverse scaling factors r | q << 8 of this filter's 26 entries (64 lines per load, which the compute unit's waves share in
    // its first-level cache: reading the table in order and handing it over through LDS was 14 % slower)
    uint32_t rq[MODE == WG_SCALED ? kEntries : 1];
    if constexpr (MODE == WG_SCALED) {
        const ScaleEntry* tk = reinterpret_cast<const ScaleEntry*>(blob + table_off) + (size_t)k * kEntries;
#pragma unroll
        for (int e = 0; e < kEntries; ++e) rq[e] = (uint32_t)tk[e].r | ((uint32_t)tk[e].q << 8);
    }
    auto unscale = [&](int e, int m) {
        if constexpr (MODE == WG_SCALED) {
            // at most four channels: |m| <= 4 * 2047 * 127 < 2^21, so m * r + 2^(q-1) fits 32 bits and
            // the product is a 24-bit multiply
            const int r = (int)(rq[e] & 0xff), q = (int)(rq[e] >> 8);
            static_assert(2LL * kNarrowChannels * 2047 * 127 * 255 + 64 < (1LL << 31), "m * r + rnd fits int32");
            return (__mul24(m, r) + ((1 << q) >> 1)) >> q;
        } else {
            return m;
        }
    };
    __syncthreads();

    // int8 output: 16-byte stores need K % 16 = 0 and an aligned buffer; two staging buffers so
    // that a tile's bytes are not overwritten while the previous tile's are being read
    __shared__ __attribute__((aligned(16))) int8_t staging[Q8 ? 2 : 1][Q8 ? 16 * 64 : 16];
    const bool vector_store = Q8 && ((p.K & 15) | (reinterpret_cast<uintptr_t>(q8.out) & 15)) == 0;

    const int count = min(tiles_per_wave, p.T - tile0);
    // With at most four input channels |y| < 2^21, so every shift from 22 on gives 0; capping it
    // at 24 changes no result and keeps 16 * round and 4 + shift within 32 bits for shifts up to 31.
    const int sh = Q8 ? min(q8.shift, 24) : 0, shift = 4 + sh;
    // what is added to every output before its final shift: M[1][1] enters each of the sixteen once, with weight one
    const int add = (MODE == WG_SCALED ? 8 : 0) + (sh > 0 ? 16 << (sh - 1) : 0);
    int most = 127;
    asm volatile("" : "+v"(most));
    for (int t = 0; t < count; ++t) {
        // all of the tile's numbers are requested before the first one is used, so the wave waits
        // for LDS once per tile
        uint4 v[kNarrowPieces];
#pragma unroll
        for (int i = 0; i < kNarrowPieces; ++i) v[i] = values[i * kWaveTiles + t];
        __builtin_amdgcn_sched_barrier(0);
        int re[16], cr[10], ci[10];
#pragma unroll
        for (int i = 0; i < 8; ++i) {   // pieces 0..7: real entries 2i, 2i+1
            re[2 * i] = unscale(2 * i, dot4(v[i].x, v[i].y, w[i].x, w[i].y));
            re[2 * i + 1] = unscale(2 * i + 1, dot4(v[i].z, v[i].w, w[i].z, w[i].w));
        }
#pragma unroll
        for (int j = 0; j < 10; ++j) {   // piece 8 + j: (Re, Im) of complex entry j
            const uint4 a = v[8 + j], b = w[8 + j];
            cr[j] = unscale(16 + j, dot4(a.x, a.y, b.x, b.y) - dot4(a.z, a.w, b.z, b.w));
            ci[j] = unscale(16 + j, dot4(a.z, a.w, b.x, b.y, dot4(a.x, a.y, b.z, b.w)));
        }
        re[5] += add;
        int out[4][4];   // out[j][i]: output row i, column j
        output_tile(re, cr, ci, out);

        const int n = __builtin_amdgcn_readlane(my_n, t);
        const int row = 4 * __builtin_amdgcn_readlane(my_ty, t), col = 4 * __builtin_amdgcn_readlane(my_tx, t);
        if constexpr (!Q8) {
            int32_t* dst = y + (((size_t)n * p.H + row) * p.W + col) * p.K + k;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (k < p.K && row + i < p.H && col + j < p.W) dst[(size_t)(i * p.W + j) * p.K] = out[j][i] >> 4;
        } else {
            // side x side output pixels per tile (2 x 2 after pooling), one byte per lane and pixel
            const int side = q8.pool ? 2 : 4, lg = q8.pool ? 1 : 2;
            const int Ho = p.H >> (q8.pool ? 1 : 0), Wo = p.W >> (q8.pool ? 1 : 0);
            const int orow = q8.pool ? row >> 1 : row, ocol = q8.pool ? col >> 1 : col;
            int8_t* tile_out = q8.out + (((size_t)n * Ho + orow) * Wo + ocol) * p.K;
            int8_t bytes[16];   // pixel (i, j) of the tile at 4 i + j; pooled: (pi, pj) at 2 pi + pj
            if (q8.pool) {
#pragma unroll
                for (int pi = 0; pi < 2; ++pi)
#pragma unroll
                    for (int pj = 0; pj < 2; ++pj) {
                        const int best = max(max(out[2 * pj][2 * pi], out[2 * pj + 1][2 * pi]), max(out[2 * pj][2 * pi + 1], out[2 * pj + 1][2 * pi + 1]));
                        bytes[2 * pi + pj] = (int8_t)requantise_y16(best, shift, q8.lo, most);   // monotonic: once, after the maximum
                    }
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) bytes[4 * i + j] = (int8_t)requantise_y16(out[j][i], shift, q8.lo, most);
            }
            if (vector_store) {
                // through LDS, so that a lane stores 16 consecutive filters of one pixel: stage[pixel][filter]
                int8_t* stage = staging[t & 1];
#pragma unroll
                for (int px = 0; px < 16; ++px)
                    if (px < side * side) stage[px * 64 + lane] = bytes[px];
                __syncthreads();   // one wave: orders the LDS writes before the reads
                const int px = lane >> 2, f0 = 16 * (lane & 3), i = px >> lg, j = px & (side - 1);
                if (px < side * side && orow + i < Ho && ocol + j < Wo && blockIdx.y * 64 + f0 < p.K)
                    *reinterpret_cast<uint4*>(tile_out + (size_t)(i * Wo + j) * p.K + blockIdx.y * 64 + f0) =
                        *reinterpret_cast<const uint4*>(stage + px * 64 + f0);
            } else {
#pragma unroll
                for (int px = 0; px < 16; ++px) {
                    const int i = px >> lg, j = px & (side - 1);
                    if (px < side * side && k < p.K && orow + i < Ho && ocol + j < Wo)
                        tile_out[(size_t)(i * Wo + j) * p.K + k] = bytes[px];
                }
            }
        }
    }
}

// Where a tile's outputs go.
struct TilePlace {
    uint32_t pixel;        // of the first output
    uint16_t rows, cols;   // that exist from there on
};
struct Factor {   // r, and q in the bits that a 24-bit multiply ignores; what is added before the shift
    int rq, addend;
};
constexpr int kFactorBytes = 64 * kEntries * (int)sizeof(Factor);   // [filter][entry]: 52 dwords apart, sixteen filters in different banks

// grid: (ceil(T / (16 groups)), Kp / 64), 256 threads.  THROUGH: 16-byte stores go through the L2 (write_out; which: first_layer_through).
template <int MODE, bool Q8, bool THROUGH>
__global__ __launch_bounds__(256, 2) void narrow_conv_kernel(const int8_t* __restrict__ x, WG_GEOMETRY_PARAMS, int groups,
                                                             const uint8_t* __restrict__ blob,
                                                             size_t table_off, size_t narrow_off, int32_t* __restrict__ y,
                                                             Problem p, Int8Epilogue q8) {
    WG_TAKE_GEOMETRY(p, 2);
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    int8_t* const values = lds;
    TilePlace* const places = reinterpret_cast<TilePlace*>(lds + groups * 16 * kTileValuesBytes);
    int8_t* const staging = reinterpret_cast<int8_t*>(places + groups * 16);
    Factor* const factors = reinterpret_cast<Factor*>(staging + 2 * kStagedGroupBytes);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tile0 = blockIdx.x * groups * 16;
    const BlobHeaderWords header = read_blob_header(blob);   // requested here, compared once the patch is on its way

    // ---- phase 1: lane = (tile, two channels) ---------------------------------------------------------------
    const int a_tile = tid >> 1;
    const bool mine = a_tile < groups * 16;
    int n = 0, ty = 0, tx = 0;
    if (tile0 + a_tile < p.T) decode_tile(p, tile0 + a_tile, n, ty, tx);   // else tile (0,0,0): loaded, never stored
    uint32_t u[6][6];
    if (mine) load_narrow_patch(x, p, n, ty, tx, u);
    if (!blob_matches(header, p.K, p.C, MODE)) return;
    // this wave's filters: lane l has filter l & 15 of them
    const int k0 = blockIdx.y * 64, k = k0 + 16 * wave + (lane & 15);   // < Kp: the blob's tables are padded to Kp
    uint4 raw[kNarrowPieces];
    {
        const uint4* from = reinterpret_cast<const uint4*>(blob + narrow_off) + (size_t)k * kNarrowPieces;
#pragma unroll
        for (int i = 0; i < kNarrowPieces; ++i) raw[i] = from[i];
    }
    constexpr int kFactorRounds = MODE == WG_SCALED ? (64 * kEntries + 255) / 256 : 1;
    int2 rq[kFactorRounds];
    if constexpr (MODE == WG_SCALED) {
        const ScaleEntry* tk = reinterpret_cast<const ScaleEntry*>(blob + table_off) + (size_t)k0 * kEntries;
#pragma unroll
        for (int i = 0; i < kFactorRounds; ++i)
            rq[i] = *reinterpret_cast<const int2*>(&tk[min(tid + 256 * i, 64 * kEntries - 1)].r);
    }
    if (mine) {
        bias_patch(p, ty, tx, 0, u);
        const uint32_t pair = tid & 1 ? HalfPairs::kSecondPair : HalfPairs::kFirstPair;
#pragma unroll
        for (int i = 0; i < 36; ++i) u[i / 6][i % 6] = HalfPairs::from_biased(u[i / 6][i % 6], pair);
        transform_patch<HalfPairs>(u, ValueKeeper{values + a_tile * kTileValuesBytes + 4 * (tid & 1)});
        const int half = Q8 && q8.pool ? 1 : 0, row = 4 * ty >> half, col = 4 * tx >> half;
        if ((tid & 1) == 0)
            places[a_tile] = TilePlace{((uint32_t)n * (uint32_t)(p.H >> half) + (uint32_t)row) * (uint32_t)(p.W >> half) + (uint32_t)col,
                                       (uint16_t)(tile0 + a_tile < p.T ? min((p.H >> half) - row, 4) : 0), (uint16_t)min((p.W >> half) - col, 4)};
    }

    // ---- phase 2 -----------------------------------------------------------------------------------------------
    // Reverse scaling of a sum m as floor((m r + 2^(q-1)) / 2^q).  The matrix-core sums of scaled mode begin at 1.5 x 2^23, so that
    // a sum's bits, read as an integer, end in 2^22 + m: a 24-bit multiply-add takes them as they are, with r 2^22 subtracted
    // from what it adds.  |m| <= 4 * 2047 * 127 < 2^21, so everything fits 32 bits.
    constexpr float kSumStart = MODE == WG_SCALED ? 12582912.0f : 0.0f;
    constexpr int kSumOffset = 1 << 22;
    static_assert(2LL * kNarrowChannels * 1024 * 127 < (1 << 21) && (3LL << 21) * 255 + 64 < (1LL << 31), "sums and products fit");
    if constexpr (MODE == WG_SCALED) {
#pragma unroll
        for (int i = 0; i < kFactorRounds; ++i) {
            const int r = rq[i].x & 0xff, q = rq[i].y & 0xff;
            if (tid + 256 * i < 64 * kEntries) factors[tid + 256 * i] = Factor{r | q << 24, ((1 << q) >> 1) - r * kSumOffset};
        }
    }
    h16x4 w[kNarrowValues];
    typedef short s16x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int i = 0; i < kNarrowPieces; ++i) {
        w[2 * i] = __builtin_convertvector(__builtin_bit_cast(s16x4, make_uint2(raw[i].x, raw[i].y)), h16x4);
        w[2 * i + 1] = __builtin_convertvector(__builtin_bit_cast(s16x4, make_uint2(raw[i].z, raw[i].w)), h16x4);
    }
    auto factor_of = [&](int e) { return MODE == WG_SCALED ? factors[(16 * wave + (lane & 15)) * kEntries + e] : Factor{0, 0}; };
    auto unscale = [&](v4f m, const Factor f) {
        v4i v;
        if constexpr (MODE == WG_SCALED) {
            const v4i bits = __builtin_bit_cast(v4i, m);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = (__mul24(bits[i], f.rq) + f.addend) >> ((uint32_t)f.rq >> 24);
        } else {
            v = __builtin_convertvector(m, v4i);
        }
        return v;
    };
    const v4f start = {kSumStart, kSumStart, kSumStart, kSumStart};
    auto product = [&](h16x4 a, h16x4 b, v4f c) { return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 0, 0, 0); };
    __syncthreads();

    // Outputs go through LDS to be stored four filters at a time or more (int8: 16 where K and the buffer allow it); two
    // staging buffers so that they are not overwritten while the previous ones are being read.
    const bool whole_pieces = Q8 && (((uint32_t)p.K | (uint32_t)reinterpret_cast<uintptr_t>(q8.out)) & 15) == 0;
    // With at most four input channels |y| < 2^21, so every shift from 22 on gives 0; capping it
    // at 24 changes no result and keeps 16 * round and 4 + shift within 32 bits for shifts up to 31.
    const int sh = Q8 ? min(q8.shift, 24) : 0, shift = 4 + sh;
    // what is added to every output before its final shift: M[1][1] enters each of the sixteen once, with weight one
    const int add = (MODE == WG_SCALED ? 8 : 0) + (16 << sh >> 1 & ~15);
    int most = 127;
    asm volatile("" : "+v"(most));
    const int side = Q8 && q8.pool ? 2 : 4, lg = Q8 && q8.pool ? 1 : 2, half = Q8 && q8.pool ? 1 : 0;
    const int Wo = p.W >> half;
    const int8_t* const my_values = values + (4 * (lane >> 4) + (lane & 3)) * kTileValuesBytes;   // as the first operand

    const int count = min(groups, (p.T - tile0 + 15) >> 4);
    for (int g = 0; g < count; ++g) {
        asm volatile("" ::: "memory");   // factors come from LDS each time (they would spill)
        const int8_t* const from = my_values + g * 16 * kTileValuesBytes;
        auto piece = [&](int i) { return *reinterpret_cast<const uint4*>(from + 16 * i); };
        v4i er[6], ei[6], Y[16];   // register i of a lane: tile 4 (lane / 16) + i, filter lane & 15
        auto real_pair = [&](int e, v4i& first, v4i& second) {   // entries e and e + 1
            const uint4 a = piece(e / 2);
            first = unscale(product(__builtin_bit_cast(h16x4, make_uint2(a.x, a.y)), w[e], start), factor_of(e));
            second = unscale(product(__builtin_bit_cast(h16x4, make_uint2(a.z, a.w)), w[e + 1], start), factor_of(e + 1));
        };
        auto complex_one = [&](int j, v4i& re, v4i& im) {
            const uint4 a = piece(8 + j);
            const h16x4 ar = __builtin_bit_cast(h16x4, make_uint2(a.x, a.y)), ai = __builtin_bit_cast(h16x4, make_uint2(a.z, a.w));
            const h16x4 minus = __builtin_bit_cast(h16x4, make_uint2(a.z ^ 0x80008000u, a.w ^ 0x80008000u));
            const Factor f = factor_of(16 + j);
            re = unscale(product(minus, w[17 + 2 * j], product(ar, w[16 + 2 * j], start)), f);
            im = unscale(product(ai, w[16 + 2 * j], product(ar, w[17 + 2 * j], start)), f);
        };
        static_for<4>([&](auto R) {
            constexpr int row = R;
            real_pair(4 * row, er[0], er[1]);
            real_pair(4 * row + 2, er[2], er[3]);
            complex_one(row, er[4], ei[4]);
            if constexpr (row == 1) er[1] += add;
            finish_row<row, (row < 3)>(er, ei, Y);
        });
#pragma unroll
        for (int j = 0; j < 6; ++j) complex_one(4 + j, er[j], ei[j]);
        finish_row<4, false>(er, ei, Y);   // Y[4 i + j]: output row i, column j
        // (the stores below are conditional: without this the last additions move into each of the conditions)
#pragma unroll
        for (int i = 0; i < 16; ++i) asm volatile("" : "+v"(Y[i]));

        if constexpr (!Q8) {
            // a row of the tiles' outputs at a time, so that 64 filters of a pixel are stored together
            static_for<4>([&](auto I) {
                int8_t* const stage = staging + (I & 1) * kStagedGroupBytes;
                int32_t* const put = reinterpret_cast<int32_t*>(stage + 4 * (lane >> 4) * kStagedTileBytes) + 16 * wave + (lane & 15);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) put[q * (kStagedTileBytes / 4) + 64 * j] = Y[4 * I + j][q] >> 4;
                __syncthreads();
                const int f0 = 4 * (tid & 15), j = (tid >> 4) & 3;
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const int tile = 4 * m + wave;
                    const TilePlace to = places[16 * g + tile];
                    if ((int)I < to.rows && j < to.cols && k0 + f0 < p.K) {
                        v4i* const at = reinterpret_cast<v4i*>(y + ((size_t)to.pixel + (int)I * Wo + j) * p.K + k0 + f0);
                        const v4i v = *reinterpret_cast<const v4i*>(stage + tile * kStagedTileBytes + 256 * j + 4 * f0);
                        write_as<THROUGH>(at, v);
                    }
                }
            });
        } else {
            // side x side output pixels per tile (2 x 2 after pooling), one byte per lane, tile and pixel
            if (q8.pool) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {   // monotonic: once, after the maximum
                    const int at = 8 * (i / 2) + 2 * (i % 2);
                    Y[i] = __builtin_elementwise_max(__builtin_elementwise_max(Y[at], Y[at + 1]), __builtin_elementwise_max(Y[at + 4], Y[at + 5]));
                }
            }
            // A dword takes the bytes of the lane's four tiles: [tiles / 4][pixel][filter], the sixteen filters of a wave turned by
            // the pixel in steps of four, so that neither side meets bank conflicts.  (Bytes stored one by one, four lanes to a
            // dword, take the LDS four times as long: 224x224x3 -> 64, lossless, N = 8 22.5 us instead of 21.6, N = 1 7.4 / 7.1.)
            int8_t* const stage = staging + (g & 1) * kStagedGroupBytes;
            uint32_t* const put = reinterpret_cast<uint32_t*>(stage + (lane >> 4) * (4 * kStagedTileBytes)) + 16 * wave + (lane & 3);
#pragma unroll
            for (int px = 0; px < 16; ++px)
                if (px < 4 || !q8.pool) {
                    v4i v;
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[q] = requantise_y16(Y[px][q], shift, q8.lo, most);
                    put[64 * px + ((lane + 4 * px) & 12)] = pack_bytes(v);
                }
            __syncthreads();
            // A thread stores 16 consecutive filters of one pixel: unpooled of four tiles, pooled of one.
            const int piece = tid & 3, px = (tid >> 2) & (q8.pool ? 3 : 15), quad = q8.pool ? (tid >> 4) & 3 : wave;
            const int8_t* const get = stage + quad * (4 * kStagedTileBytes) + 256 * px + 64 * piece;
            uint4 d[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) d[m] = *reinterpret_cast<const uint4*>(get + 16 * ((m + px) & 3));
            const int i = px >> lg, j = px & (side - 1);
            auto store = [&](int q, uint4 v) {
                const TilePlace to = places[16 * g + 4 * quad + q];
                const int left = p.K - k0 - 16 * piece;
                if (i < to.rows && j < to.cols && left > 0) {
                    int8_t* const at = q8.out + ((size_t)to.pixel + i * Wo + j) * p.K + k0 + 16 * piece;
                    if (whole_pieces) {
                        write_as<THROUGH>(reinterpret_cast<v4i*>(at), __builtin_bit_cast(v4i, v));
                    } else {
                        uint32_t* const dwords = reinterpret_cast<uint32_t*>(at);
                        dwords[0] = v.x;
                        if (left > 4) dwords[1] = v.y;
                        if (left > 8) dwords[2] = v.z;
                        if (left > 12) dwords[3] = v.w;
                    }
                }
            };
            if (q8.pool) {
                const uint32_t low = 0x0c0c0400u + 0x0101u * wave, high = 0x04000c0cu + 0x01010000u * wave;   // byte `wave` of two dwords
                auto byte_of = [&](uint4 v) { return __builtin_amdgcn_perm(v.y, v.x, low) | __builtin_amdgcn_perm(v.w, v.z, high); };
                store(wave, make_uint4(byte_of(d[0]), byte_of(d[1]), byte_of(d[2]), byte_of(d[3])));
            } else {
#pragma unroll
                for (int m = 0; m < 4; ++m) {   // four filters x four tiles -> four tiles x four filters
                    const uint32_t xy01 = __builtin_amdgcn_perm(d[m].y, d[m].x, 0x05010400u), xy23 = __builtin_amdgcn_perm(d[m].y, d[m].x, 0x07030602u);
                    const uint32_t zw01 = __builtin_amdgcn_perm(d[m].w, d[m].z, 0x05010400u), zw23 = __builtin_amdgcn_perm(d[m].w, d[m].z, 0x07030602u);
                    d[m] = make_uint4(__builtin_amdgcn_perm(zw01, xy01, 0x05040100u), __builtin_amdgcn_perm(zw01, xy01, 0x07060302u),
                                      __builtin_amdgcn_perm(zw23, xy23, 0x05040100u), __builtin_amdgcn_perm(zw23, xy23, 0x07060302u));
                }
                store(0, make_uint4(d[0].x, d[1].x, d[2].x, d[3].x));
                store(1, make_uint4(d[0].y, d[1].y, d[2].y, d[3].y));
                store(2, make_uint4(d[0].z, d[1].z, d[2].z, d[3].z));
                store(3, make_uint4(d[0].w, d[1].w, d[2].w, d[3].w));
            }
        }
    }
}

std::atomic<int> g_narrow_variant{0};

}  // namespace

void set_narrow_variant(int v) { g_narrow_variant.store(v, std::memory_order_relaxed); }

// Few tiles: 16 of them take a wave longer from the patch to the last store than the vector ALU's few.  64 groups of 16 tiles x 64
// filters are two waves of narrow_wave_kernel per compute unit, 128 four, one per SIMD: the next group costs it 6 - 8 %.  (us,
// narrow_wave_kernel and narrow_conv_kernel: scaled, int8 out, 49 groups 7.1, 7.9; 64 groups 7.3, 7.7, pooled 6.9, 7.1; 66 groups 8.0, 7.7, pooled
// 7.6, 7.0; 98 groups 8.6, 7.7; 196 groups, 224x224x3 -> 64 at N = 1, 10.7, 7.9.  Lossless, int8 out, 98 groups 6.5, 6.9; 128 groups 6.75, 6.95;
// 196 groups 7.8, 7.1.)  int32 outputs are four times the stores, which a lone workgroup does not hide (scaled, 66 groups 8.0, 8.1, 128 groups
// 9.4, 8.6; lossless, 224x224 -> 64, N = 2 12.2, 12.9; N = 8 24.7, 25.7; N = 16 41.9, 40.0; N = 32 107, 85).
bool narrow_on_matrix_cores(int tiles, int Kp, int mode, bool int8_out) {
    if (const int forced = g_narrow_variant.load(std::memory_order_relaxed)) return forced == 1;
    const long long groups = (long long)ceil_div(tiles, 16) * (Kp / 64);
    return groups > (mode == WG_SCALED ? (int8_out ? 64 : 70) : int8_out ? 128 : 1999);
}

namespace {

template <int MODE, bool Q8>
hipError_t launch(const int8_t* x, const uint8_t* blob, const BlobLayout& bl, int32_t* y, const Problem& p,
                  const Int8Epilogue& q8, hipStream_t s) {
    const int tile_groups = ceil_div(p.T, 16), blocks = p.Kp / 64;
    // Nor outputs that cannot be stored four filters at a time (K = 75, 224x224 N = 4, lossless, pooled 21.4, 24.8; K = 130, 100x120 N = 4, C = 4 10.7, 15.5).
    const uint32_t uneven = Q8 ? (uint32_t)p.K | (uint32_t)reinterpret_cast<uintptr_t>(q8.out) : 4u * (uint32_t)p.K | (uint32_t)reinterpret_cast<uintptr_t>(y);
    if ((uneven & (Q8 ? 3 : 15)) != 0 || !narrow_on_matrix_cores(p.T, p.Kp, MODE, Q8)) {
        // Tiles per wave: the kernel is bound by vector instructions, so the waves should fill every
        // SIMD evenly: two waves on each of the 1,024 SIMDs (two cover each other's LDS and memory
        // waits; a third would only add transform phases with mostly idle lanes).
        const long long work = (long long)p.T * (p.Kp / 64);
        const int tiles = (int)std::min<long long>(kWaveTiles, std::max<long long>(2, (work + 2047) / 2048));
        dim3 grid(ceil_div(p.T, tiles), p.Kp / 64);
        narrow_wave_kernel<MODE, Q8><<<grid, 64, 0, s>>>(x, WG_GEOMETRY(p), tiles, blob, bl.table_off, bl.narrow_off, y, p, q8);
        return hipGetLastError();
    }
    // Groups of 16 tiles per workgroup.  A compute unit takes two workgroups at a time, which then need 2.4 + 2 g times as long as a
    // group's share of it (1.7 us in scaled mode), a single one 1.45 + 1.31 g.  Measured with scaled, pooled outputs; the choice is within 0.3 % of
    // the best of the seven on average for every kind of int8 outputs (176 layers, 7 % at most), and 1.5 % for int32 ones, where one group
    // per workgroup is ahead of two just above a round (scaled, 280 groups 12.5, 13.1).  (Scaled, pooled, 224x224x3 -> 64, us for one to seven groups:
    // N = 4 17.2, 13.5, 16.7, 14.2, 16.5, 18.7, 21.1; N = 8 26.8, 23.4, 23.7, 20.4, 23.6, 26.8, 21.6; N = 32 85.5, 66.5, 61.9, 60.0, 53.0, 60.5, 56.0.)
    int groups = 1;
    double best = 1e300;
    for (int g = 1; g <= kNarrowGroups; ++g) {
        const long long workgroups = (long long)ceil_div(tile_groups, g) * blocks, each = (workgroups + compute_units() - 1) / compute_units();
        const double cost = (double)(each / 2) * (2.4 + 2 * g) + (double)(each % 2) * (1.45 + 1.31 * g);
        if (cost < best) { best = cost; groups = g; }
    }
    auto lds_bytes = [](int g) {
        return g * 16 * (kTileValuesBytes + (int)sizeof(TilePlace)) + 2 * kStagedGroupBytes + (MODE == WG_SCALED ? kFactorBytes : 0);
    };
    auto run = [&](auto THROUGH) -> hipError_t {
        static LdsLimitOnce lds_limit;   // per template instance
        if (hipError_t e = lds_limit.set(reinterpret_cast<const void*>(&narrow_conv_kernel<MODE, Q8, THROUGH>), lds_bytes(kNarrowGroups))) return e;
        dim3 grid(ceil_div(tile_groups, groups), blocks);
        narrow_conv_kernel<MODE, Q8, THROUGH><<<grid, 256, lds_bytes(groups), s>>>(x, WG_GEOMETRY(p), groups, blob, bl.table_off, bl.narrow_off, y, p, q8);
        return hipGetLastError();
    };
    const bool through = Q8 ? first_layer_through(p, q8.out, 1, q8.pool) : first_layer_through(p, y, 4, false);
    return through ? run(std::true_type{}) : run(std::false_type{});
}

}  // namespace

hipError_t launch_narrow_conv(const int8_t* x, const void* blob, int32_t* y, const Problem& p, int mode,
                              const Int8Epilogue& q8, hipStream_t s) {
    static_assert(kFilterPad % 64 == 0, "a wave covers 64 filters of the padded filter count");
    const BlobLayout bl = blob_layout(p.Kp, p.C, mode);
    const uint8_t* b = static_cast<const uint8_t*>(blob);
    if (mode == WG_LOSSLESS)
        return q8.out != nullptr ? launch<WG_LOSSLESS, true>(x, b, bl, y, p, q8, s) : launch<WG_LOSSLESS, false>(x, b, bl, y, p, q8, s);
    return q8.out != nullptr ? launch<WG_SCALED, true>(x, b, bl, y, p, q8, s) : launch<WG_SCALED, false>(x, b, bl, y, p, q8, s);
}

}  // namespace wg
