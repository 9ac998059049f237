// Products of the limb-pair filter operand (see lossless_conv.hip): a wave multiplies 8 filters with the 16 tiles whose operand planes
// (byte limbs) are in LDS, and reduces what it gets into 16 outputs of 2 filters x 1 tile per lane.
#pragma once
#include "kernel_common.h"

namespace wg {
namespace {
namespace pairs {

typedef int v2i __attribute__((ext_vector_type(2)));

// ---- which entries a wave multiplies, in order -------------------------------------------------
// A wave owns half or a quarter of the entries ("share").
// Half 0: rows 0, 1, 2 of M (five entries each: four real, then the complex M[row][3]) and M[3][0];
// half 1: M[3][1], M[3][2], M[3][5], M[3][3], M[3][4] and row 5.  56 matrix-core instructions each.
// Quarters (shares 2 .. 5): rows 0 and 1; row 2 and row 5; M[3][0], M[3][1], M[3][2]; M[3][5], M[3][3], M[3][4].  32, 32, 24 and 24 instructions.
// The whole (share 6): rows 0, 1, 2, 5, then 3.
// Entry numbering as in the blob: real entries 0..15 (4 RI + CI over rows/columns 0,1,2,5), complex
// 16..19 = M[RI][3], 20..23 = M[3][CI], 24 = M[3][3], 25 = M[3][4].
struct Slot {
    int entry, row, pos;   // row 0..3: real rows 0,1,2,5; row 4: the complex row 3; pos: place in finish_row's arrays
    bool ends;             // last entry of its row in this half
};
constexpr int kFirstQuarter = 2, kWhole = 6;
constexpr int half_slots(int half) { return half == kWhole ? 26 : half == 0 ? 16 : half < 4 ? 10 : 3; }
constexpr Slot half_slot(int half, int s) {
    if (half == kWhole) return s < 20 ? Slot{s % 5 < 4 ? 4 * (s / 5) + s % 5 : 16 + s / 5, s / 5, s % 5, s % 5 == 4} : Slot{s, 4, s - 20, s == 25};
    if (half == 3) return s < 5 ? Slot{s < 4 ? 8 + s : 18, 2, s, s == 4} : Slot{s < 9 ? 7 + s : 19, 3, s - 5, s == 9};
    if (half >= 4) return Slot{20 + 3 * (half - 4) + s, 4, 3 * (half - 4) + s, s == 2};
    if (half == 0 || half == 2) {
        if (s < 15) return Slot{s % 5 < 4 ? 4 * (s / 5) + s % 5 : 16 + s / 5, s / 5, s % 5, s % 5 == 4};
        return Slot{20, 4, 0, true};
    }
    // the complex row first: its reduction is the longest, and the last row's reduction has nothing to hide behind
    if (s < 5) return Slot{21 + s, 4, s + 1, s == 4};
    return Slot{s < 9 ? 7 + s : 19, 3, s - 5, s == 9};
}
constexpr bool real_entry(int e) { return e < kRealEntries; }
constexpr int entry_fragments(int e) { return real_entry(e) ? 1 : 2; }
constexpr int entry_value(int e) { return real_entry(e) ? e : 16 + 2 * (e - kRealEntries); }   // blob value index (Re; Im follows)
constexpr int entry_plane(int e) { return real_entry(e) ? 2 * e : 32 + 4 * (e - kRealEntries); }
constexpr int frag_start(int half, int s) {   // index of slot s's first fragment in the wave's fragment stream
    int n = 0;
    for (int i = 0; i < s; ++i) n += entry_fragments(half_slot(half, i).entry);
    return n;
}
constexpr int half_fragments(int half) { return frag_start(half, half_slots(half)); }
static_assert(half_fragments(0) + half_fragments(1) == kPairValues, "one fragment per Winograd-domain value");
static_assert(half_fragments(kWhole) == kPairValues, "and in the whole");
static_assert(half_fragments(2) + half_fragments(3) + half_fragments(4) + half_fragments(5) == kPairValues, "the same in quarters");
constexpr int frag_value(int half, int f) {   // blob value index of fragment f of the stream
    int s = 0;
    while (frag_start(half, s + 1) <= f) ++s;
    return entry_value(half_slot(half, s).entry) + (f - frag_start(half, s));
}

// value = 2^16 hh + 2^8 (lh + hl) + ll for the two filters of a lane: wd = W x Dh, wl = W x Dl,
// registers (Wh0, Wl0, Wh1, Wl1) x D.
__device__ inline v2i join_pair(v4i wd, v4i wl) {
    v2i out;
#pragma unroll
    for (int f = 0; f < 2; ++f) {
        int t = (wd[2 * f] << 8) + (wd[2 * f + 1] + wl[2 * f]);
        asm("" : "+v"(t));   // keeps the two shift-and-add instructions apart
        out[f] = (t << 8) + wl[2 * f + 1];
    }
    return out;
}

struct WaveContext {
    const int8_t* act;   // this lane's 16 bytes of activation plane 0 (LDS)
    const int8_t* flt;   // this lane's 16 bytes of filter fragment 0 of the current channel block (channels not split)
};

constexpr int kRing = 10;   // filter fragments in flight per wave

// Eight waves share what the compute unit takes in, some 57 bytes per clock, so a wave's 16 to 20 filter fragments per channel
// block are requested well ahead: the first kRing before the products, the others each time a ring slot has been used.
template <int HALF>
struct Products {
    static constexpr int NS = half_slots(HALF), NF = half_fragments(HALF);   // HALF: a share

    template <int F>
    __device__ inline static v4i fragment(const WaveContext& cx) {
        constexpr int offset = frag_value(HALF, F) * kFilterFragBytes;   // evaluated by the compiler
        return *reinterpret_cast<const v4i*>(cx.flt + offset);
    }
    // the same of a channel block given as a buffer, `lane16` = 16 x lane
    template <int F>
    __device__ inline static v4i fragment(__amdgpu_buffer_rsrc_t block, uint32_t lane16) {
        constexpr int offset = frag_value(HALF, F) * kFilterFragBytes;
        return buffer_fragment(block, lane16, offset);
    }
    template <int PLANE>
    __device__ inline static v4i activation(const WaveContext& cx) {
        return *reinterpret_cast<const v4i*>(cx.act + PLANE * kPlaneBytes);
    }
    // the first fragments, one per call (I = 0 .. kRing - 1), pinned where the caller puts them
    template <int I>
    __device__ inline static void prefetch_one(const WaveContext& cx, v4i (&ring)[kRing]) {
        __builtin_amdgcn_sched_barrier(0);
        ring[I] = fragment<I>(cx);
        __builtin_amdgcn_sched_barrier(0);
    }

    // One 64-channel block: entry s multiplies while entry s+1's activation fragments come from LDS,
    // the ring is refilled, and entry s-1 is joined and (at the end of a row of M) reduced into Y.
    // refill(F): fragment F has been used.
    template <class Refill>
    __device__ inline static void run(const WaveContext& cx, v4i (&ring)[kRing], v2i (&Y)[16], Refill&& refill) {
        v4i afr[2][4], acc[2][6];
        v2i er[6], ei[6];
        constexpr int e0 = half_slot(HALF, 0).entry;
        static_for<2 * entry_fragments(e0)>([&](auto I) { afr[0][I] = activation<entry_plane(e0) + I>(cx); });
        static_for<NS + 1>([&](auto S) {
            constexpr int s = S;
            if constexpr (s < NS) {
                constexpr int e = half_slot(HALF, s).entry, f0 = frag_start(HALF, s);
                if constexpr (s + 1 < NS) {
                    constexpr int en = half_slot(HALF, s + 1).entry;
                    static_for<2 * entry_fragments(en)>([&](auto I) { afr[(s + 1) & 1][I] = activation<entry_plane(en) + I>(cx); });
                }
                constexpr v4i zero = {0, 0, 0, 0};
                v4i (&a)[6] = acc[s & 1];
                const v4i (&d)[4] = afr[s & 1];
                const v4i w0 = ring[f0 % kRing];
                if constexpr (real_entry(e)) {
                    a[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w0, d[0], zero, 0, 0, 0);   // W x Dh
                    a[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w0, d[1], zero, 0, 0, 0);   // W x Dl
                } else {
                    // d = (Dr h, Dr l, Di h, Di l); Im = Wr Di + Wi Dr (a[0], a[1]), Re = Wr Dr (a[2], a[3]) - Wi Di (a[4], a[5]);
                    // instructions into the same accumulator are kept four apart
                    const v4i w1 = ring[(f0 + 1) % kRing];
                    a[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w0, d[2], zero, 0, 0, 0);
                    a[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w0, d[3], zero, 0, 0, 0);
                    a[2] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w0, d[0], zero, 0, 0, 0);
                    a[3] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w0, d[1], zero, 0, 0, 0);
                    a[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w1, d[0], a[0], 0, 0, 0);
                    a[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w1, d[1], a[1], 0, 0, 0);
                    a[4] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w1, d[2], zero, 0, 0, 0);
                    a[5] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w1, d[3], zero, 0, 0, 0);
                }
                static_for<entry_fragments(e)>([&](auto I) {
                    refill(std::integral_constant<int, f0 + I>{});
                });
            }
            if constexpr (s > 0) {
                constexpr Slot sl = half_slot(HALF, s - 1);
                const v4i (&a)[6] = acc[(s - 1) & 1];
                v2i re, im = {0, 0};
                if constexpr (real_entry(sl.entry)) {
                    re = join_pair(a[0], a[1]);
                } else {
                    re = join_pair(a[2] - a[4], a[3] - a[5]);
                    im = join_pair(a[0], a[1]);
                }
                if constexpr (HALF == 0 && sl.row == 4) {
                    // M[3][0] alone: in the row rule of A^T it only enters z0 = e0 + ..., which the column rule
                    // spreads as y0 += 2 Re z0, y1 -= 2 Im z0, y2 -= 2 Re z0, y3 += 2 Im z0 (first output column)
                    Y[0] += 2 * re;
                    Y[4] -= 2 * im;
                    Y[8] -= 2 * re;
                    Y[12] += 2 * im;
                } else {
                    er[sl.pos] = re;
                    ei[sl.pos] = im;
                    if constexpr (HALF == 1 && sl.row == 4 && sl.pos == 1) {   // M[3][0] belongs to the other half
                        er[0] = (v2i){0, 0};
                        ei[0] = (v2i){0, 0};
                    }
                    if constexpr (HALF >= 4 && s == 1) {   // and half of the row to the other quarter
#pragma unroll
                        for (int e = 0; e < 3; ++e) er[HALF == 4 ? 3 + e : e] = ei[HALF == 4 ? 3 + e : e] = (v2i){0, 0};
                    }
                    if constexpr (sl.ends) finish_row<sl.row, false>(er, ei, Y);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    }
};

// Every entry of one channel block in a wave that has 168 registers: 36 steps, one per Winograd-domain value, a complex entry's
// imaginary part (Wr Di + Wi Dr) before its real one, so that no more than 24 registers of limb products are alive; a step's products are
// joined behind the next one's matrix-core instructions.  RING filter fragments are in flight.
template <int RING>
struct WholeProducts {
    static constexpr int kSteps = kPairValues, NF = kPairValues;
    struct Step {
        int slot;
        bool imaginary;
    };
    static constexpr Step step(int v) {
        int s = 0;
        while (frag_start(kWhole, s + 1) <= v) ++s;
        return Step{s, !real_entry(half_slot(kWhole, s).entry) && v == frag_start(kWhole, s)};
    }
    template <int F>
    __device__ inline static v4i fragment(__amdgpu_buffer_rsrc_t block, uint32_t lane16) { return Products<kWhole>::template fragment<F>(block, lane16); }

    // act: this lane's 16 bytes of plane 0.  Y: the first outputs there are.
    template <class Refill>
    __device__ inline static void run(const int8_t* act, v4i (&ring)[RING], v2i (&Y)[16], Refill&& refill) {
        v4i d[2][4], acc[2][4];
        v2i er[6], ei[6];
        auto load = [&](auto S) {
            constexpr int e = half_slot(kWhole, S).entry;
            static_for<2 * entry_fragments(e)>([&](auto I) { d[S & 1][I] = *reinterpret_cast<const v4i*>(act + (entry_plane(e) + I) * kPlaneBytes); });
        };
        auto mul = [](v4i w, v4i x, v4i c) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(w, x, c, 0, 0, 0); };
        constexpr v4i zero = {0, 0, 0, 0};
        load(std::integral_constant<int, 0>{});
        static_for<kSteps + 1>([&](auto V) {
            constexpr int v = V;
            if constexpr (v < kSteps) {
                constexpr Step st = step(v);
                constexpr int s = st.slot, e = half_slot(kWhole, s).entry, f = frag_start(kWhole, s);
                if constexpr (!st.imaginary && s + 1 < 26) load(std::integral_constant<int, s + 1>{});
                const v4i (&x)[4] = d[s & 1];
                v4i (&a)[4] = acc[v & 1];
                const v4i w0 = ring[f % RING];
                if constexpr (real_entry(e)) {
                    a[0] = mul(w0, x[0], zero);   // W x Dh
                    a[1] = mul(w0, x[1], zero);   // W x Dl
                    refill(std::integral_constant<int, f>{});
                } else {   // x = (Dr h, Dr l, Di h, Di l)
                    const v4i w1 = ring[(f + 1) % RING];
                    if constexpr (st.imaginary) {
                        a[0] = mul(w0, x[2], zero);
                        a[1] = mul(w0, x[3], zero);
                        a[0] = mul(w1, x[0], a[0]);
                        a[1] = mul(w1, x[1], a[1]);
                    } else {
                        a[0] = mul(w0, x[0], zero);
                        a[1] = mul(w0, x[1], zero);
                        a[2] = mul(w1, x[2], zero);
                        a[3] = mul(w1, x[3], zero);
                        refill(std::integral_constant<int, f>{});
                        refill(std::integral_constant<int, f + 1>{});
                    }
                }
            }
            if constexpr (v > 0) {
                constexpr Step st = step(v - 1);
                constexpr Slot sl = half_slot(kWhole, st.slot);
                const v4i (&a)[4] = acc[(v - 1) & 1];
                if constexpr (st.imaginary) {
                    ei[sl.pos] = join_pair(a[0], a[1]);
                    asm volatile("" : "+v"(ei[sl.pos]));   // here, or the limb products of every step live to the end (see LeanProducts)
                } else {
                    if constexpr (real_entry(sl.entry)) er[sl.pos] = join_pair(a[0], a[1]);
                    else                                er[sl.pos] = join_pair(a[0] - a[2], a[1] - a[3]);
                    asm volatile("" : "+v"(er[sl.pos]));
                    if constexpr (sl.ends) {
                        finish_row<sl.row, (sl.row < 3)>(er, ei, Y);
                        if constexpr (sl.row >= 2)
#pragma unroll
                            for (int i = 0; i < 16; ++i) asm volatile("" : "+v"(Y[i]));
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    }
};

}  // namespace pairs
}  // namespace
}  // namespace wg
