// Activations scaled per tile (complex F(4x4,3x3)): the factor table and the input transform's receivers, shared by the
// kernels that scale them.
#pragma once
#include "product_core.h"

namespace wg {
namespace {

// ---- activations scaled as well (the remark that closes Section 4.1) --------------------------------------------
// Section 4.1 ends by noting that the analysis of Section 4.2 applies to B^T d B too (12 bits here for int8 data).
// The rule used is that section's with a tile in the place of an output feature map: at each of a tile's 26 free
// entries the largest max(|Re|, |Im|) over the input channels decides one factor n/2^p, Re and Im of every channel's
// value there are multiplied by it (round half up), and the channel sums are multiplied back by its reciprocal r/2^q
// after the filter's.  Both operands are then single int8 values: one matrix-core instruction per real product, 36
// operand planes instead of 72, channel sums accumulated by the matrix cores themselves.
//
// (n, p, r, q) for every possible maximum of int8 data, one byte each (n = 0: within the range, nothing applied).
constexpr int kActMax = 16 * 128;
struct ActScaleTable {
    uint32_t v[kActMax + 1];
};
constexpr ActScaleTable make_act_scale_table() {
    ActScaleTable t = {};
    for (int mx = 0; mx <= kActMax; ++mx) {
        uint32_t n = 0, p = 0, r = 1, q = 0;
        if (mx > kWeightRange) {
            const int num = kWeightRange * 128;
            int y = 0;
            while ((mx << (y + 1)) <= num) ++y;
            n = (uint32_t)((num * 8) / (mx << y));
            p = (uint32_t)(10 - y);
            for (int qq = 7; qq >= 0; --qq) {
                const uint32_t rr = ((2u << (p + qq)) + n) / (2 * n);
                if (rr <= 255) { r = rr; q = (uint32_t)qq; break; }
            }
        }
        t.v[mx] = n | (p << 8) | (r << 16) | (q << 24);
    }
    return t;
}
constexpr uint32_t largest_act_shift() {
    const ActScaleTable t = make_act_scale_table();
    uint32_t p = 0;
    for (int mx = 0; mx <= kActMax; ++mx) p = ((t.v[mx] >> 8) & 255u) > p ? (t.v[mx] >> 8) & 255u : p;
    return p;
}
static_assert(largest_act_shift() <= 8, "act_factors");
__device__ const ActScaleTable kActScale = make_act_scale_table();

constexpr int kActPlanes = 36;                       // 16 real entries, then (Re, Im) of each complex entry
static_assert(kActPlanes * kPlaneBytes <= kLdsBytes, "the single-limb planes lie where the two-limb planes do");
constexpr int kActNpBytes = 16 * kEntries * 4;          // uint32 [tile][26]: act_factors
constexpr int kActRqBytes = kEntries * 16 * 4;         // uint32 [26][tile]: the table entry (r, q in its upper bytes)

__device__ inline s16x2 abs_max(Quad v) {
    const s16x2 zero = {0, 0};
    return __builtin_elementwise_max(__builtin_elementwise_max(v.a, zero - v.a), __builtin_elementwise_max(v.b, zero - v.b));
}
// transform_patch's receiver in the first pass: running maxima per free entry, two channels per register
struct MaxKeeper {
    s16x2* mx;
    __device__ inline void real_entry(int p, Quad v) const { mx[p] = __builtin_elementwise_max(mx[p], abs_max(v)); }
    __device__ inline void complex_entry(int j, Quad re, Quad im) const {
        mx[kRealEntries + j] = __builtin_elementwise_max(mx[kRealEntries + j], __builtin_elementwise_max(abs_max(re), abs_max(im)));
    }
};
// ... and in the second: every value times its tile's factor, rounded half up, as one int8 operand plane
struct ScaledPlanes {
    LdsPlaneSink sink;
    const uint32_t* np;   // this tile's 26 factors
    __device__ inline uint32_t scaled(int entry, Quad v) const {
        const s16x2 mul = as_s16x2(np[entry]), half = {128, 128};
        return pack_high_bytes(Quad{v.a * mul + half, v.b * mul + half});
    }
    __device__ inline void real_entry(int p, Quad v) const { sink.put(p, scaled(p, v)); }
    __device__ inline void complex_entry(int j, Quad re, Quad im) const {
        sink.put(kRealEntries + 2 * j, scaled(kRealEntries + j, re));
        sink.put(kRealEntries + 2 * j + 1, scaled(kRealEntries + j, im));
    }
};

// What a table entry means to the transform threads: n 2^(8-p) twice, in 16 bits each.  p <= 8, so (v n + 2^(p-1)) >> p is
// (v n 2^(8-p) + 128) >> 8, the upper byte of 16 bits (|v n| <= 127 2^p; unscaled, n = 1 and p = 0, |v| <= 127): one multiply-add per
// two channels and the permutation that packs the bytes anyway, one dword of LDS per entry.  With n, 2^(p-1) and p in three it
// took a shift more and a 16-byte read: 256 -> 256 at 14x14, N = 64, both kernels, 26.5 us.
__device__ inline uint32_t act_factors(uint32_t entry) {
    return (max(entry & 255u, 1u) << (8u - ((entry >> 8) & 255u))) * 0x00010001u;
}
// ... and (n, p, r, q) as the exported table has it.
__device__ inline v4i act_table_row(uint32_t entry) {
    return (v4i){(int)(entry & 255u), (int)((entry >> 8) & 255u), (int)((entry >> 16) & 255u), (int)(entry >> 24)};
}

}  // namespace
}  // namespace wg
