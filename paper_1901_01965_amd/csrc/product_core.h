// Pieces shared by the single-kernel convolution variants: the per-entry matrix-core programs of the Winograd-domain
// products, the waves' share of them, the output staging and the stores.
#pragma once
#include <atomic>

#include "kernel_common.h"

namespace wg {
namespace {

constexpr int kFusedTiles = kTileBlock;   // tiles per workgroup (rows of the 16x16x64 matrix-core product)
constexpr int kFusedFilters = 32;   // filters per workgroup: two 16-wide column blocks
constexpr int kFusedPlanes = 72;    // two-limb activation planes (kSplitTwoLimb)
constexpr int kLdsBytes = kFusedPlanes * kPlaneBytes;
// How the activation patch reaches the transform threads (chosen on the host):
//   kLoadBytes:  one byte per load, any layout and channel count;
//   kLoadDwords: channels-last, C a multiple of 4: one 4-byte load per pixel and thread;
//   kLoadDirect: channels-last, C a multiple of 16, 16-byte aligned input: 16-byte pieces travel
//                from global memory straight into LDS (nine instructions per wave instead of
//                thirty-six), and the threads pick their four channels from there.
constexpr int kLoadBytes = 0, kLoadDwords = 1, kLoadDirect = 2;
constexpr int kRawWaveBytes = 4 * 36 * kCBlock;      // raw patches of a wave's four tiles: 36 pixels x 64 channels
constexpr int kRawBytes = 4 * kRawWaveBytes;

// Development aid (never compiled into the library): time spent in each part of a kernel's loop.
#ifdef WG_TIMESTAMPS
__device__ unsigned long long* g_roles_stamps = nullptr;
#define WG_CLOCK() __builtin_amdgcn_s_memtime()
#define WG_SPENT(i, since) do { const unsigned long long now_ = WG_CLOCK(); spent[i] += now_ - (since); (since) = now_; } while (0)
#else
#define WG_SPENT(i, since) do { } while (0)
#endif

// ---- per-entry programs ----------------------------------------------------------------
// An entry's product uses a few activation fragments (from LDS) and filter fragments (from
// the packed blob) and a short list of matrix-core instructions into a few accumulators.
//   lossless, real:    A = (h, l)  B = (h, l)          acc = (hh, hl+lh, ll)
//   lossless, complex: A = (Re h, Re l, Im h, Im l)  B = (Wr h, Wr l, Wi h, Wi l)
//                      acc 0-2: Dr*Wr, 3-5: Di*Wi, 6-8: Dr*Wi + Di*Wr, each as (hh, mid, ll)
//   scaled, real:      A = (h, l)  B = (W)             acc = (h, l)
//   scaled, complex:   B = (Wr, Wi, -Wi)               acc = (Re h, Re l, Im h, Im l)
//   scaled, complex, without the -Wi plane (kScaledTwoPlanes as MODE of the helpers below: a
//   third less filter traffic per complex entry for two subtractions per register):
//                      B = (Wr, Wi)                    acc = (Dr*Wr h, l, Im h, Im l, Di*Wi h, l)
constexpr int kScaledTwoPlanes = 2;
static_assert(kScaledTwoPlanes != WG_LOSSLESS && kScaledTwoPlanes != WG_SCALED, "a value of its own");
struct Op {
    int a, b, acc;
    bool init;   // first instruction into this accumulator (starts from zero)
};
constexpr bool is_real(int entry) { return entry < kRealEntries; }
template <int MODE> constexpr int num_a(int entry) { return is_real(entry) ? 2 : 4; }
template <int MODE> constexpr int num_b(int entry) {
    return MODE == WG_LOSSLESS ? (is_real(entry) ? 2 : 4) : (is_real(entry) ? 1 : (MODE == kScaledTwoPlanes ? 2 : 3));
}
template <int MODE> constexpr int num_ops(int entry) {
    return MODE == WG_LOSSLESS ? (is_real(entry) ? 4 : 16) : (is_real(entry) ? 2 : 8);
}
template <int MODE> constexpr int a_plane(int entry, int i) {
    return is_real(entry) ? 2 * entry + i : 32 + 4 * (entry - kRealEntries) + i;
}
template <int MODE> constexpr int b_plane(int entry, int i) {
    if (MODE == WG_LOSSLESS) {   // blob planes 3*value + {0: high limb, 1: low limb}
        if (is_real(entry)) return 3 * entry + i;
        const int value = 16 + 3 * (entry - kRealEntries) + (i >> 1);   // Re, then Im
        return 3 * value + (i & 1);
    }
    return is_real(entry) ? entry : 16 + 3 * (entry - kRealEntries) + i;
}
template <int MODE> constexpr Op entry_op(int entry, int i) {
    constexpr Op lossless_real[4] = {{0, 0, 0, true}, {0, 1, 1, true}, {1, 1, 2, true}, {1, 0, 1, false}};
    // dependent instructions into one accumulator are kept at least three apart
    constexpr Op lossless_complex[16] = {
        {0, 0, 0, true}, {0, 1, 1, true}, {1, 1, 2, true},    // Dr*Wr: hh, mid, ll
        {2, 2, 3, true}, {2, 3, 4, true}, {3, 3, 5, true},    // Di*Wi
        {0, 2, 6, true}, {0, 3, 7, true}, {1, 3, 8, true},    // Dr*Wi
        {1, 2, 7, false}, {1, 0, 1, false}, {3, 2, 4, false},
        {2, 1, 7, false}, {2, 0, 6, false}, {3, 1, 8, false}, {3, 0, 7, false}};
    constexpr Op scaled_real[2] = {{0, 0, 0, true}, {1, 0, 1, true}};
    constexpr Op scaled_complex[8] = {{0, 0, 0, true}, {1, 0, 1, true}, {0, 1, 2, true}, {1, 1, 3, true},
                                      {2, 2, 0, false}, {3, 2, 1, false}, {2, 0, 2, false}, {3, 0, 3, false}};
    constexpr Op two_planes_complex[8] = {{0, 0, 0, true}, {1, 0, 1, true}, {0, 1, 2, true}, {1, 1, 3, true},
                                          {2, 1, 4, true}, {3, 1, 5, true}, {2, 0, 2, false}, {3, 0, 3, false}};
    if (MODE == WG_LOSSLESS) return is_real(entry) ? lossless_real[i] : lossless_complex[i];
    if (MODE == kScaledTwoPlanes) return is_real(entry) ? scaled_real[i] : two_planes_complex[i];
    return is_real(entry) ? scaled_real[i] : scaled_complex[i];
}

// ---- which entries a wave owns, in order ---------------------------------------------------
// Half 0 owns rows 0,1,2 of M and M[3][0], half 1 row 5 and the rest of row 3, so that both have the same number of
// matrix-core instructions (scaled mode 56 and 56; by whole rows 48 and 64); "half" 2 is all five rows, for a wave that
// owns every entry.  A real row RI (rows 0,1,2,5) holds entries 4RI..4RI+3 and the complex
// entry 16+RI; the complex row holds entries 20..25.
constexpr int kAllRows = 2;
constexpr int row_entries(int row) { return row < 4 ? 5 : 6; }
constexpr int row_entry(int row, int pos) {
    return row < 4 ? (pos < 4 ? 4 * row + pos : kRealEntries + row) : kRealEntries + 4 + pos;
}
constexpr int half_entries(int half) { return half == 0 ? 16 : (half == 1 ? 10 : 26); }
constexpr bool fresh_row(int half, int row) { return row < 3 || half == 1; }   // see finish_row: no earlier row of this half
struct Slot {
    int entry, row, pos;
    bool last_in_row;   // of those this half has
};
constexpr Slot half_slot(int half, int i) {
    if (half == 0 && i == 15) return Slot{row_entry(4, 0), 4, 0, true};
    int n = 0;
    for (int r = half == 1 ? 3 : 0; r < 5; ++r) {   // half 1: row 5, then row 3 from its second entry on
        const int skip = half == 1 && r == 4 ? 1 : 0, entries = row_entries(r) - skip;
        if (i < n + entries) return Slot{row_entry(r, i - n + skip), r, i - n + skip, i - n == entries - 1};
        n += entries;
    }
    return Slot{0, 0, 0, false};
}
// The value of slot S of a half takes its place in the row being collected; the last of a row enters the outputs.
// ACCUMULATE: onto outputs that exist already.
template <int HALF, int S, bool ACCUMULATE = false>
__device__ inline void place_entry(const v4i re, const v4i im, v4i (&er)[6], v4i (&ei)[6], v4i (&Y)[16]) {
    constexpr Slot sl = half_slot(HALF, S);
    if constexpr (HALF == 0 && sl.row == 4) {   // M[3][0] alone: it only enters z0 = e0 + .. of finish_row
        Y[0] += 2 * re;
        Y[4] -= 2 * im;
        Y[8] -= 2 * re;
        Y[12] += 2 * im;
    } else {
        er[sl.pos] = re;
        ei[sl.pos] = im;
        if constexpr (HALF == 1 && sl.row == 4 && sl.pos == 1) er[0] = ei[0] = (v4i){0, 0, 0, 0};
        if constexpr (sl.last_in_row) finish_row<sl.row, !ACCUMULATE && fresh_row(HALF, sl.row)>(er, ei, Y);
    }
}
// index of the first filter fragment of slot i in the wave's fragment stream
template <int MODE> constexpr int b_start(int half, int i) {
    int n = 0;
    for (int s = 0; s < i; ++s) n += num_b<MODE>(half_slot(half, s).entry);
    return n;
}
// the slot that filter fragment f of the stream belongs to
template <int MODE> constexpr int b_slot_of(int half, int f) {
    int s = 0;
    while (b_start<MODE>(half, s + 1) <= f) ++s;
    return s;
}

// Direct global -> LDS transfer of the raw 6x6 patches of a wave's four tiles (one 64-channel
// block).  Instruction i (0..8) moves pixels 4i..4i+3 of the patch (pixel = 6 a + b): lane l
// carries 16 channels (piece l % 4) of tile (l % 16) / 4 at pixel 4i + l / 16, and the hardware
// puts lane l's piece at (wave-uniform destination) + 16 l.  The raw area of a wave is therefore
// [pixel][tile][64 channels], and transform thread (tile, channel quad) = lane reads its pixel
// p at p * 256 + 4 * lane: a wave reads 256 contiguous bytes.
struct DirectPatch {
    uint32_t pixel_off[9];   // byte offset of this lane's pixel (channel 0) for each instruction
    // (n, ty, tx): the tile this lane moves pieces of.  With j = lane / 16, instruction i covers
    // pixel 4i + j = 6a + b of the patch: a = {0,0,1,2,2,3,4,4,5}[i] + (i % 3 == 1 and j >= 2),
    // and b takes only three values per lane: j (i % 3 == 0), (j + 4) % 6 (i % 3 == 1) and j + 2
    // (i % 3 == 2).  Row terms follow each other by one clamped row step, so the whole table
    // costs four multiplications.
    __device__ inline void init(const Problem& p, int n, int ty, int tx, int lane) {
        const int h0 = 4 * ty - 1, w0 = 4 * tx - 1, j = lane >> 4;
        const uint32_t row_step = (uint32_t)(p.W * p.C);
        uint32_t row_term[6];
        row_term[0] = (uint32_t)(n * p.H + max(h0, 0)) * row_step;
#pragma unroll
        for (int a = 1; a < 6; ++a)   // rows clamp to [0, H-1]: the step is taken only inside the image
            row_term[a] = row_term[a - 1] + ((unsigned)(h0 + a - 1) < (unsigned)(p.H - 1) ? row_step : 0u);
        const int b1 = j < 2 ? j + 4 : j - 2;
        const uint32_t col_term[3] = {(uint32_t)(min(max(w0 + j, 0), p.W - 1) * p.C),
                                      (uint32_t)(min(max(w0 + b1, 0), p.W - 1) * p.C),
                                      (uint32_t)(min(max(w0 + j + 2, 0), p.W - 1) * p.C)};
        constexpr int a_base[9] = {0, 0, 1, 2, 2, 3, 4, 4, 5};
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            uint32_t row = row_term[a_base[i]];
            if (i % 3 == 1) row = j >= 2 ? row_term[a_base[i] + 1] : row;
            pixel_off[i] = row + col_term[i % 3];
        }
    }
    // Pieces beyond C (the last channel block of a C that is not a multiple of 64) re-read
    // channel 0; bias_patch() discards them.
    __device__ inline void issue(const int8_t* __restrict__ x, const Problem& p, int cb, int lane,
                                 int8_t* raw_wave) const {
        const int c = cb * kCBlock + (lane & 3) * 16;
        const int8_t* src = x + (c < p.C ? c : 0);
#pragma unroll
        for (int i = 0; i < 9; ++i) __builtin_amdgcn_global_load_lds(src + pixel_off[i], raw_wave + i * 1024, 16, 0, 0);
    }
    __device__ inline static void read(const int8_t* raw_wave, int lane, uint32_t u[6][6]) {
#pragma unroll
        for (int a = 0; a < 6; ++a)
#pragma unroll
            for (int b = 0; b < 6; ++b)
                u[a][b] = *reinterpret_cast<const uint32_t*>(raw_wave + (6 * a + b) * 256 + 4 * lane);
    }
};

struct LaneContext {
    const int8_t* a_lds;        // this lane's 16-byte slot in plane 0
    const int8_t* b_glob;       // filter plane 0 of the wave's 16 filters, current channel block; the same for the whole wave
    uint32_t b_lane;            // this lane's 16 bytes in a fragment: a scalar base and a 32-bit offset cost no address arithmetic
    const ScaleEntry* table_k;  // scaling table row of this lane's filter (scaled mode)
    const uint32_t* parked;     // role-specialised kernels, scaled mode: see park_scales
};

// The first fragment of the 16 filters from k (wave-uniform) on, channel block 0, and a lane's place in a fragment.
__device__ inline const int8_t* filter_fragments(const uint8_t* planes, int k, int Kp, int nplanes) {
    return reinterpret_cast<const int8_t*>(planes) + filter_plane_offset(0, 0, __builtin_amdgcn_readfirstlane(k), 0, Kp, nplanes);
}
__device__ inline uint32_t fragment_lane(int lane) { return (uint32_t)lane * 16u; }

constexpr int kFilterPrefetch = 16;   // filter fragments in flight per wave (covers L2 latency)

// value = 4096 hh + 64 mid + ll, modulo 2^32, as two shift-and-add instructions per register.
// The empty statement only pins the intermediate value, so that the compiler does not rewrite
// the expression as two shifts and a three-operand add.
__device__ inline v4i join_limbs(v4i hh, v4i mid, v4i ll) {
    v4i out;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        int t = (hh[q] << 6) + mid[q];
        asm("" : "+v"(t));
        out[q] = (t << 6) + ll[q];
    }
    return out;
}

template <int MODE, int HALF>
struct ProductPhase {
    static constexpr int NE = half_entries(HALF);
    static constexpr int NB = b_start<MODE>(HALF, NE);
    static constexpr int NPRE = NB < kFilterPrefetch ? NB : kFilterPrefetch;
    v4i bring[kFilterPrefetch];

    // F-th filter fragment of this wave's stream.  A workgroup that covers more than 32 filters
    // goes through its entries once per 32 (pass F / NB); the wave's 16-filter fragment of the
    // next pass lies two fragments (2 * planes KB) further on in the blob.
    // BUFFER: see load_fragment.
    template <int F, bool BUFFER = false>
    __device__ inline static v4i load_b(const LaneContext& cx) {
        constexpr int pass = F / NB, f = F % NB;
        constexpr int slot = b_slot_of<MODE>(HALF, f);
        constexpr int plane = b_plane<MODE>(half_slot(HALF, slot).entry, f - b_start<MODE>(HALF, slot));
        constexpr int planes = MODE == WG_LOSSLESS ? 138 : 46;
        constexpr int at = (pass * 2 * planes + plane) * kFilterFragBytes;
        if constexpr (BUFFER) return load_fragment(cx.b_glob, cx.b_lane, at);
        else return *reinterpret_cast<const v4i*>(cx.b_glob + at + cx.b_lane);
    }
    template <int SLOT, int I>
    __device__ inline static v4i load_a(const LaneContext& cx) {
        constexpr int plane = a_plane<MODE>(half_slot(HALF, SLOT).entry, I);
        return *reinterpret_cast<const v4i*>(cx.a_lds + plane * kPlaneBytes);
    }

    // Filter fragments do not depend on the transform phase: start them before it.
    __device__ inline void prefetch(const LaneContext& cx) {
        static_for<NPRE>([&](auto I) { bring[I] = load_b<I>(cx); });
    }
    static_assert(NB >= kFilterPrefetch || MODE != WG_LOSSLESS, "the ring is full from the first pass on");

    // One 64-channel block of this wave's rows.  Software pipeline over entries: while entry i's
    // matrix-core instructions run, entry i+1's activation fragments come from LDS, the filter
    // ring is refilled sixteen fragments ahead, and entry i-1's accumulators are joined,
    // (un)scaled and reduced into the outputs.
    // PASS of NPASS: which 32 of the workgroup's filters (see load_b).
    template <int PASS = 0, int NPASS = 1>
    __device__ inline void run(const LaneContext& cx, v4i (&Y)[16]) {
        constexpr int F0 = PASS * NB, FEND = NPASS * NB;   // this pass's place in the fragment stream
        v4i afr[2][4], acc[2][9], er[6], ei[6];
        static_for<num_a<MODE>(half_slot(HALF, 0).entry)>([&](auto I) { afr[0][I] = load_a<0, I>(cx); });
        static_for<NE + 1>([&](auto S) {
            constexpr int s = S;
            if constexpr (s < NE) {
                constexpr int entry = half_slot(HALF, s).entry;
                constexpr int b0 = b_start<MODE>(HALF, s);
                if constexpr (s + 1 < NE)
                    static_for<num_a<MODE>(half_slot(HALF, s + 1).entry)>(
                        [&](auto I) { afr[(s + 1) & 1][I] = load_a<s + 1, I>(cx); });
                static_for<num_ops<MODE>(entry)>([&](auto I) {
                    constexpr Op op = entry_op<MODE>(entry, I);
                    constexpr v4i zero = {0, 0, 0, 0};
                    acc[s & 1][op.acc] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                        afr[s & 1][op.a], bring[(F0 + b0 + op.b) % kFilterPrefetch],
                        op.init ? zero : acc[s & 1][op.acc], 0, 0, 0);
                });
                static_for<num_b<MODE>(entry)>([&](auto I) {
                    if constexpr (F0 + b0 + I + kFilterPrefetch < FEND)
                        bring[(F0 + b0 + I) % kFilterPrefetch] = load_b<F0 + b0 + I + kFilterPrefetch>(cx);
                });
            }
            if constexpr (s > 0) {
                constexpr Slot sl = half_slot(HALF, s - 1);
                const v4i(&a)[9] = acc[(s - 1) & 1];
                v4i re, im = {0, 0, 0, 0};
                if constexpr (MODE == WG_LOSSLESS) {
                    if constexpr (is_real(sl.entry)) {
                        re = join_limbs(a[0], a[1], a[2]);
                    } else {   // Re = Dr Wr - Di Wi,  Im = Dr Wi + Di Wr
                        re = join_limbs(a[0] - a[3], a[1] - a[4], a[2] - a[5]);
                        im = join_limbs(a[6], a[7], a[8]);
                    }
                } else {
                    re = (a[0] << kByteLimbShift) + a[1];
                    if constexpr (!is_real(sl.entry)) im = (a[2] << kByteLimbShift) + a[3];
                    const ReverseScale unscale(cx.table_k[PASS * kFusedFilters * kEntries + sl.entry]);   // Section 4.2
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        re[q] = unscale(re[q]);
                        if constexpr (!is_real(sl.entry)) im[q] = unscale(im[q]);
                    }
                }
                place_entry<HALF, s - 1, true>(re, im, er, ei, Y);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    }
};

// Role-specialised kernels, scaled mode: the reverse-scaling factors (r, q) of the entries a
// product wave owns, read once at the start of the kernel (while the wave would only wait for
// the first operand planes) and parked in LDS as rounding << 16 | q << 8 | r, [slot][filter of the wave], so that
// the reverse scaling after the last channel block does not begin with a trip to L2.  Lane
// group g = lane / 16 reads slots g, 4 + g, 8 + g, 12 + g of filter lane % 16: ask() issues the
// four loads, park() writes what they brought, and a caller puts its first filter prefetch
// between the two so that one wait covers both.  Each wave writes and later reads its own 1 KB
// (16 slots x 16 filters; 2 KB for a wave that owns all 26 entries), in program order: no barrier.
constexpr int kParkedScaleBytes = 16 * 16 * 4;
template <int HALF>
struct ParkedScales {
    static constexpr int NE = ProductPhase<WG_SCALED, HALF>::NE;
    static constexpr int kRounds = (NE + 3) / 4;   // a wave that owns every entry: seven loads per lane, 2 KB
    static constexpr int kBytes = kRounds * 4 * 16 * 4;
    int2 rq[kRounds];
    __device__ inline void ask(const LaneContext& cx, int lane) {
        const int g = lane >> 4;
        static_for<kRounds>([&](auto J) {
            int entry = half_slot(HALF, 4 * J).entry;   // slot 4 J + g, clamped to the last slot
            static_for<3>([&](auto G) {
                constexpr int slot = 4 * J + G + 1 < NE ? 4 * J + G + 1 : NE - 1;
                if (g > G) entry = half_slot(HALF, slot).entry;
            });
            rq[J] = *reinterpret_cast<const int2*>(&cx.table_k[entry].r);
        });
    }
    __device__ inline void park(LaneContext& cx, int8_t* area, int lane) {
        uint32_t* const base = reinterpret_cast<uint32_t*>(area) + (lane & 15);
        const int g = lane >> 4;
        static_for<kRounds>([&](auto J) {
            if (4 * J + g < NE)    // r <= 255, q <= 7
                base[(4 * J + g) * 16] = (((1u << rq[J].y) >> 1) << 16) | ((uint32_t)rq[J].y << 8) | (uint32_t)rq[J].x;
        });
        cx.parked = base;
    }
};
template <int SLOT>
__device__ inline ReverseScale parked_scale(const LaneContext& cx) {
    const uint32_t v = cx.parked[SLOT * 16];
    return ReverseScale((int)(v & 0xffu), (int)(v >> 8) & 31, (int)(v >> 16));
}

// Scaled mode over several channel blocks: the products of every entry a wave owns accumulate
// in registers across the blocks (run, once per block), and the reverse scaling and the output
// transform are applied to the finished channel sums (finish, once).
template <int HALF>
struct ScaledSums {
    static constexpr int MODE = WG_SCALED;
    using Phase = ProductPhase<MODE, HALF>;
    static constexpr int NE = Phase::NE, NB = Phase::NB;
    static constexpr int sum_start(int slot) {   // first sum of a slot: one per real entry, Re and Im per complex
        int n = 0;
        for (int s = 0; s < slot; ++s) n += is_real(half_slot(HALF, s).entry) ? 1 : 2;
        return n;
    }
    static constexpr int kSums = sum_start(NE);

    // One channel block: each entry's limb products are formed from zero, and its value
    // 256 * high + low (byte limbs) joins the entry's running sum one entry later.
    template <int PASS = 0, int NPASS = 1>
    __device__ inline static void run(const LaneContext& cx, v4i (&bring)[kFilterPrefetch], v4i* sums) {
        constexpr int F0 = PASS * NB, FEND = NPASS * NB;   // this pass's place in the fragment stream
        v4i afr[2][4], acc[2][4];
        static_for<num_a<MODE>(half_slot(HALF, 0).entry)>([&](auto I) { afr[0][I] = Phase::template load_a<0, I>(cx); });
        static_for<NE + 1>([&](auto S) {
            constexpr int s = S;
            if constexpr (s < NE) {
                constexpr int entry = half_slot(HALF, s).entry;
                constexpr int b0 = b_start<MODE>(HALF, s);
                if constexpr (s + 1 < NE)
                    static_for<num_a<MODE>(half_slot(HALF, s + 1).entry)>(
                        [&](auto I) { afr[(s + 1) & 1][I] = Phase::template load_a<s + 1, I>(cx); });
                static_for<num_ops<MODE>(entry)>([&](auto I) {
                    constexpr Op op = entry_op<MODE>(entry, I);
                    constexpr v4i zero = {0, 0, 0, 0};
                    acc[s & 1][op.acc] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                        afr[s & 1][op.a], bring[(F0 + b0 + op.b) % kFilterPrefetch],
                        op.init ? zero : acc[s & 1][op.acc], 0, 0, 0);
                });
                static_for<num_b<MODE>(entry)>([&](auto I) {
                    if constexpr (F0 + b0 + I + kFilterPrefetch < FEND)
                        bring[(F0 + b0 + I) % kFilterPrefetch] = Phase::template load_b<F0 + b0 + I + kFilterPrefetch>(cx);
                });
            }
            if constexpr (s > 0) {
                constexpr int v = sum_start(s - 1);
                const v4i(&a)[4] = acc[(s - 1) & 1];
                sums[v] += (a[0] << kByteLimbShift) + a[1];
                if constexpr (!is_real(half_slot(HALF, s - 1).entry)) sums[v + 1] += (a[2] << kByteLimbShift) + a[3];
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    }

    // After the last channel block: reverse scaling of the finished sums and the output transform.
    template <int PASS = 0, bool PARKED = false>
    __device__ inline static void finish(const LaneContext& cx, const v4i* sums, v4i (&Y)[16]) {
        v4i er[6], ei[6];
        static_for<NE>([&](auto S) {
            constexpr Slot sl = half_slot(HALF, S);
            constexpr int v = sum_start(S);
            v4i re = sums[v], im = {0, 0, 0, 0};
            if constexpr (!is_real(sl.entry)) im = sums[v + 1];
            const ReverseScale unscale = PARKED ? parked_scale<S>(cx)   // Section 4.2
                                                : ReverseScale(cx.table_k[PASS * kFusedFilters * kEntries + sl.entry]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                re[q] = unscale(re[q]);
                if constexpr (!is_real(sl.entry)) im[q] = unscale(im[q]);
            }
            place_entry<HALF, S>(re, im, er, ei, Y);
            if constexpr (sl.last_in_row) __builtin_amdgcn_sched_barrier(0);   // row by row: a row's sums are dead before the next row's work begins
        });
    }
};
constexpr int kChannelSums = 20;
static_assert(ScaledSums<0>::kSums == kChannelSums && ScaledSums<1>::kSums <= kChannelSums, "room for either half's sums");

// Who a thread is when 256 threads store the staged outputs of 16 tiles x 32 filters, and where its tile lies.
struct StoreContext {
    int8_t* lds;                                // the staged outputs
    int tid, lane;                              // within the four waves that store together
    int my_n, my_row, my_col, my_origin;        // of tile (lane & 15): image, first output row and column, offset in y (-1: none)
    int rnd;                                    // rounding added before the final >> 4
    int32_t* y;
};

// Outputs are staged filter-fastest, stage[half][output 4i+j][tile][36] (32 filters, rows padded to 36 dwords so that the
// four 16-lane groups of a wave land in different banks): wave (half, kblock) holds outputs of filters 16 kblock .. + 15.
constexpr int kStageRow = 36, kStageHalf = 16 * 16 * kStageRow;   // dwords
static_assert(2 * kStageHalf * 4 <= kLdsBytes, "staging fits the operand planes' LDS");
__device__ __forceinline__ void stage_outputs(int8_t* lds, int lane, int half, int kblock, const v4i (&Yp)[16]) {
    int* dst = reinterpret_cast<int*>(lds) + half * kStageHalf + (4 * (lane >> 4)) * kStageRow + kblock * 16 + (lane & 15);
#pragma unroll
    for (int o = 0; o < 16; ++o)
#pragma unroll
        for (int q = 0; q < 4; ++q) dst[(o * 16 + q) * kStageRow] = Yp[o][q];
}

// The same outputs of another wave's entries, added to what is staged.
__device__ __forceinline__ void add_staged_outputs(int8_t* lds, int lane, int half, int kblock, const v4i (&Yp)[16]) {
    int* dst = reinterpret_cast<int*>(lds) + half * kStageHalf + (4 * (lane >> 4)) * kStageRow + kblock * 16 + (lane & 15);
#pragma unroll
    for (int o = 0; o < 16; ++o)
#pragma unroll
        for (int q = 0; q < 4; ++q) __hip_atomic_fetch_add(&dst[(o * 16 + q) * kStageRow], Yp[o][q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Where tile (lane & 15) of tile block `tile0` starts in an output tensor of pixels (offsets fit 32 bits, checked on the
// host), into sc.
template <int LAYOUT>
__device__ __forceinline__ void locate_tile(StoreContext& sc, const Problem& p, int tile0) {
    const int t = tile0 + (sc.lane & 15);
    int n = 0, ty = 0, tx = 0;
    if (t < p.T) decode_tile(p, t, n, ty, tx);
    sc.my_n = n;
    sc.my_row = 4 * ty;
    sc.my_col = 4 * tx;
    sc.my_origin = t >= p.T ? -1 : LAYOUT == WG_NHWC ? ((n * p.H + 4 * ty) * p.W + 4 * tx) * p.K : (n * p.K * p.H + 4 * ty) * p.W + 4 * tx;
}

// Stores the 16 tiles x 32 filters (from kbase) that were staged (a barrier lies between): int32 to y, or requantised
// (and pooled) to int8 at q8.out.  ADD: two halves were staged and are added; otherwise one finished copy (half 0).
// Any K and either layout; 16-byte (int8: 4- or 16-byte) stores where K and the alignment allow.
template <int LAYOUT, int OUT, bool ADD>
__device__ __forceinline__ void store_staged(const StoreContext& sc, const Problem& p, const Int8Epilogue& q8, int kbase) {
    constexpr bool Q8 = OUT == kOutInt8, THROUGH = OUT == kOutThrough;
    const int tid = sc.tid, lane = sc.lane;
    const int* const parki = reinterpret_cast<const int*>(sc.lds);
    auto sixteen = [&](int o, int tile, int g) {   // 16 x the outputs of filters 4*g .. 4*g+3 of the block
        const int at = (o * 16 + tile) * kStageRow + 4 * g;
        v4i v = *reinterpret_cast<const v4i*>(parki + at);
        if constexpr (ADD) v += *reinterpret_cast<const v4i*>(parki + kStageHalf + at);
        return v;
    };
    auto staged = [&](int o, int tile, int g) { return (sixteen(o, tile, g) + sc.rnd) >> 4; };
    // the 2x2 maximum, requantised: rescale, requantisation and clamp are monotonic, so they come once, after the maximum
    // (112x112x128 N = 16 65.8 -> 62.4 us, 224x224x64 73.8 -> 66.5)
    auto best_of_window = [&](int tile, int pi, int pj, int g) {
        const v4i a = __builtin_elementwise_max(sixteen(4 * (2 * pi) + 2 * pj, tile, g), sixteen(4 * (2 * pi) + 2 * pj + 1, tile, g));
        const v4i b = __builtin_elementwise_max(sixteen(4 * (2 * pi + 1) + 2 * pj, tile, g), sixteen(4 * (2 * pi + 1) + 2 * pj + 1, tile, g));
        return requantise((__builtin_elementwise_max(a, b) + sc.rnd) >> 4, q8);
    };
    if constexpr (LAYOUT == WG_NCHW) {
        // A filter's outputs lie together: sixteen consecutive tiles of an image row are 64 consecutive pixels.
        if constexpr (!Q8) {
            // thread: output row i, column j of a tile; iteration: four filters, 256 contiguous bytes per wave and filter
            const int j = tid & 3, tile = (tid >> 2) & 15, i = tid >> 6;
            const int origin = __shfl(sc.my_origin, tile), h = __shfl(sc.my_row, tile) + i, w = __shfl(sc.my_col, tile) + j;
            const bool ok = origin >= 0 && h < p.H && w < p.W;
            int32_t* const first = sc.y + (size_t)(ok ? origin : 0) + i * p.W + j;
            const size_t plane = (size_t)p.H * p.W;
#pragma unroll
            for (int g = 0; g < 8; ++g) {
                const v4i v = staged(4 * i + j, tile, g);
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (ok && kbase + 4 * g + c < p.K) write_as<THROUGH>(first + (size_t)(kbase + 4 * g + c) * plane, (int32_t)v[c]);
            }
        } else if (q8.pool) {
            // thread: one pooled pixel of a tile; the four waves take two groups of four filters each
            const int pj = tid & 1, pi = (tid >> 1) & 1, tile = (tid >> 2) & 15, Ho = p.H >> 1, Wo = p.W >> 1;
            const int n = __shfl(sc.my_n, tile), row = __shfl(sc.my_row, tile), col = __shfl(sc.my_col, tile);
            const bool ok = __shfl(sc.my_origin, tile) >= 0 && row + 2 * pi < p.H && col + 2 * pj < p.W;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int g = 2 * (tid >> 6) + e;
                const v4i best = best_of_window(tile, pi, pj, g);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int kk = kbase + 4 * g + c;
                    if (ok && kk < p.K) q8.out[(((size_t)n * p.K + kk) * Ho + (row >> 1) + pi) * Wo + (col >> 1) + pj] = (int8_t)best[c];
                }
            }
        } else {
            // thread: output row i of a tile (four pixels: one dword where rows stay aligned), two groups of four filters
            const int i = tid & 3, tile = (tid >> 2) & 15;
            const int origin = __shfl(sc.my_origin, tile), row = __shfl(sc.my_row, tile) + i, col = __shfl(sc.my_col, tile);
            const bool ok = origin >= 0 && row < p.H;
            const bool word_store = ((p.W & 3) | (int)(reinterpret_cast<uintptr_t>(q8.out) & 3)) == 0;
            int8_t* const first = q8.out + (size_t)(ok ? origin : 0) + i * p.W;
            const size_t plane = (size_t)p.H * p.W;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int g = 2 * (tid >> 6) + e;
                v4i px[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) px[j] = requantise(staged(4 * i + j, tile, g), q8);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (!ok || kbase + 4 * g + c >= p.K) continue;
                    int8_t* at = first + (size_t)(kbase + 4 * g + c) * plane;
                    if (word_store) {
                        *reinterpret_cast<uint32_t*>(at) = pack_bytes((v4i){px[0][c], px[1][c], px[2][c], px[3][c]});
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (col + j < p.W) at[j] = (int8_t)px[j][c];
                    }
                }
            }
        }
        return;
    }
    // Channels-last.  Thread: filters 4*k4..4*k4+3, eight lanes cover the 128 contiguous bytes this block owns of a pixel;
    // pass ps: output row i = ps/2, tile = 8*(ps%2) + px/4, column j = px%4
    const int k4 = tid & 7, px = tid >> 3, j = px & 3;
    const int kk = kbase + 4 * k4;
    const bool quads = (p.K & 3) == 0;
    auto put4 = [&](int8_t* at, v4i v, int k_first) {   // four bytes of filters k_first ..
        if (quads) {
            if (k_first < p.K) *reinterpret_cast<uint32_t*>(at) = pack_bytes(v);
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (k_first + c < p.K) at[c] = (int8_t)v[c];
        }
    };
    if constexpr (Q8) {
        if (q8.pool) {
            // 16 tiles x 2x2 pooled pixels = 64 pixels; thread: four filters of pixels px and px + 32
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int pp = px + 32 * e, tile = pp >> 2, pi = (pp >> 1) & 1, pj = pp & 1;
                const v4i best = best_of_window(tile, pi, pj, k4);
                const int n = __shfl(sc.my_n, tile), row = __shfl(sc.my_row, tile), col = __shfl(sc.my_col, tile);
                const bool ok = __shfl(sc.my_origin, tile) >= 0 && row + 2 * pi < p.H && col + 2 * pj < p.W;
                const size_t at = (((size_t)n * (p.H >> 1) + (row >> 1) + pi) * (p.W >> 1) + (col >> 1) + pj) * p.K + kk;
                if (ok) put4(q8.out + at, best, kk);
            }
            return;
        }
        // thread: 16 filters (half h16 of the block) of its own tile (lane & 15) at outputs
        // tid/32 and tid/32 + 8: sixteen lanes read sixteen tiles' rows, which fall in
        // different banks, and a thread stores 16 bytes where the alignment allows
        const int h16 = (tid >> 4) & 1, kq = kbase + 16 * h16;
        const bool vector_store = ((p.K & 15) | (reinterpret_cast<uintptr_t>(q8.out) & 15)) == 0;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int o = (tid >> 5) + 8 * e, i = o >> 2, jj = o & 3;
            v4i v[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) v[g] = requantise(staged(o, lane & 15, 4 * h16 + g), q8);
            const bool ok = sc.my_origin >= 0 && sc.my_row + i < p.H && sc.my_col + jj < p.W;
            int8_t* dst = q8.out + (size_t)sc.my_origin + (size_t)(i * p.W + jj) * p.K + kq;
            if (ok && vector_store && kq < p.K) {
                *reinterpret_cast<uint4*>(dst) = make_uint4(pack_bytes(v[0]), pack_bytes(v[1]), pack_bytes(v[2]), pack_bytes(v[3]));
            } else if (ok) {
#pragma unroll
                for (int g = 0; g < 4; ++g) put4(dst + 4 * g, v[g], kq + 4 * g);
            }
        }
        return;
    }
    int32_t* first[2];   // output row 0 of the thread's two tiles (e = 0, 1); null where nothing is stored
    int rows[2];         // output rows of that tile inside the image
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int origin = __shfl(sc.my_origin, 8 * e + (px >> 2));
        const bool ok = origin >= 0 && __shfl(sc.my_col, 8 * e + (px >> 2)) + j < p.W && kk < p.K;
        first[e] = ok ? sc.y + (size_t)origin + j * p.K + kk : nullptr;
        rows[e] = p.H - __shfl(sc.my_row, 8 * e + (px >> 2));
    }
    const size_t row_pitch = (size_t)p.W * p.K;
    v4i v[8];
#pragma unroll
    for (int ps = 0; ps < 8; ++ps) v[ps] = staged(4 * (ps >> 1) + j, 8 * (ps & 1) + (px >> 2), k4);
#pragma unroll
    for (int ps = 0; ps < 8; ++ps) {
        const int i = ps >> 1, e = ps & 1;
        if (first[e] == nullptr || i >= rows[e]) continue;
        int32_t* at = first[e] + i * row_pitch;
        if (quads) {
            write_as<THROUGH>(reinterpret_cast<v4i*>(at), v[ps]);
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (kk + c < p.K) at[c] = v[ps][c];
        }
    }
}
// Product phase of the role-specialised kernels: the same arithmetic as ProductPhase / ScaledSums in the registers a product
// wave has there, with a filter ring of RING fragments.
//   Half of the entries (lossless mode only): channel sums of the joined values; one set of fragments and accumulators, no
//   software pipelining: such a wave's waits are covered by the other waves of its SIMD.
//   Every entry (kAllRows, either mode; scaled: one channel block): each block's products go through to the outputs at once.
//   These waves are the longer chain of the two roles, so the activation fragments of the next entry are asked for before
//   the current entry's matrix-core instructions, and an entry's vector work runs beside the next entry's matrix-core
//   instructions (a second set of fragments and of accumulators).
template <int MODE, int HALF, int RING>
struct LeanProducts {
    static constexpr bool WHOLE = HALF == kAllRows;
    static_assert(WHOLE || MODE == WG_LOSSLESS, "scaled mode keeps its channel sums in ChainedSums or ResidentScaled");
    static constexpr int PM = MODE == WG_SCALED ? kScaledTwoPlanes : MODE;   // complex entries without the -Wi plane
    using Phase = ProductPhase<PM, HALF>;
    using Target = std::conditional_t<WHOLE, v4i (&)[16], v4i*>;   // the outputs, or the channel sums in ScaledSums' order
    static constexpr int NE = Phase::NE, NB = Phase::NB;
    static constexpr int kSums = ScaledSums<HALF>::kSums;
    static_assert(NB >= RING, "the ring is full from the first channel block on");
    v4i ring[RING];

    __device__ inline void prefetch(const LaneContext& cx) {
        static_for<RING>([&](auto I) { ring[I] = Phase::template load_b<I, WHOLE>(cx); });
    }

    __device__ inline void run(const LaneContext& cx, Target to) {
        v4i er[6], ei[6];
        v4i afr2[WHOLE ? 2 : 1][4];
        if constexpr (WHOLE)
            static_for<num_a<PM>(half_slot(HALF, 0).entry)>([&](auto I) { afr2[0][I] = Phase::template load_a<0, I>(cx); });
        // the matrix-core part of slot S: activation fragments, products into acc, refill of the filter ring
        auto multiply = [&](auto S, v4i (&acc)[9]) {
            constexpr int s = S;
            constexpr int entry = half_slot(HALF, s).entry;
            constexpr int b0 = b_start<PM>(HALF, s);
            v4i (&afr)[4] = afr2[WHOLE ? (s & 1) : 0];
            if constexpr (!WHOLE) {
                static_for<num_a<PM>(entry)>([&](auto I) { afr[I] = Phase::template load_a<s, I>(cx); });
            } else if constexpr (s + 1 < NE) {
                static_for<num_a<PM>(half_slot(HALF, s + 1).entry)>(
                    [&](auto I) { afr2[(s + 1) & 1][I] = Phase::template load_a<s + 1, I>(cx); });
            }
            static_for<num_ops<PM>(entry)>([&](auto I) {
                constexpr Op op = entry_op<PM>(entry, I);
                constexpr v4i zero = {0, 0, 0, 0};
                acc[op.acc] = __builtin_amdgcn_mfma_i32_16x16x64_i8(afr[op.a], ring[(b0 + op.b) % RING],
                                                                    op.init ? zero : acc[op.acc], 0, 0, 0);
            });
            static_for<num_b<PM>(entry)>([&](auto I) {
                if constexpr (b0 + I + RING < NB) ring[(b0 + I) % RING] = Phase::template load_b<b0 + I + RING, WHOLE>(cx);
            });
        };
        // the vector part of slot S: limbs joined (Re = Dr Wr - Di Wi, Im = Dr Wi + Di Wr); then into the channel sums, or
        // reverse scaling and output transform
        auto reduce = [&](auto S, const v4i (&acc)[9]) {
            constexpr int s = S;
            constexpr Slot sl = half_slot(HALF, s);
            constexpr int entry = sl.entry;
            if constexpr (!WHOLE) {   // the output transform waits for finish_lossless()
                constexpr int v = ScaledSums<HALF>::sum_start(s);
                if constexpr (is_real(entry)) {
                    to[v] += join_limbs(acc[0], acc[1], acc[2]);
                } else {
                    to[v] += join_limbs(acc[0] - acc[3], acc[1] - acc[4], acc[2] - acc[5]);
                    to[v + 1] += join_limbs(acc[6], acc[7], acc[8]);
                }
                asm volatile("" : "+v"(to[v]));   // here, not in front of the next use of the sums with the limbs alive until then
                if constexpr (!is_real(entry)) asm volatile("" : "+v"(to[v + 1]));
            } else {
                v4i re, im = {0, 0, 0, 0};
                if constexpr (MODE == WG_LOSSLESS) {
                    if constexpr (is_real(entry)) {
                        re = join_limbs(acc[0], acc[1], acc[2]);
                    } else {
                        re = join_limbs(acc[0] - acc[3], acc[1] - acc[4], acc[2] - acc[5]);
                        im = join_limbs(acc[6], acc[7], acc[8]);
                    }
                } else {
                    if constexpr (is_real(entry)) {
                        re = (acc[0] << kByteLimbShift) + acc[1];
                    } else {
                        re = ((acc[0] - acc[4]) << kByteLimbShift) + (acc[1] - acc[5]);
                        im = (acc[2] << kByteLimbShift) + acc[3];
                    }
                    const ReverseScale unscale = parked_scale<s>(cx);   // Section 4.2
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        re[q] = unscale(re[q]);
                        if constexpr (!is_real(entry)) im[q] = unscale(im[q]);
                    }
                }
                place_entry<HALF, s, MODE != WG_SCALED>(re, im, er, ei, to);   // scaled mode: one channel block, these are the outputs' first values
                // Pins the entry's value, and a finished row's outputs, to this place.  Left alone, the compiler moves
                // the vector work of all 26 entries behind the last matrix-core instruction (into the block that
                // stages the outputs) and keeps every accumulator alive until then.
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    asm volatile("" ::"v"(re[q]));
                    if constexpr (!is_real(entry)) asm volatile("" ::"v"(im[q]));
                }
                if constexpr (sl.last_in_row) {
#pragma unroll
                    for (int i = 0; i < 16; ++i)
#pragma unroll
                        for (int q = 0; q < 4; ++q) asm volatile("" ::"v"(to[i][q]));
                }
            }
        };
        if constexpr (WHOLE) {
            // slot s + 1's matrix-core instructions are issued before slot s's vector work, which then runs beside them
            v4i acc2[2][9];
            static_for<NE + 1>([&](auto S) {
                if constexpr (S < NE) multiply(S, acc2[S & 1]);
                if constexpr (S > 0) reduce(std::integral_constant<int, S - 1>{}, acc2[(S - 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
            });
        } else {
            static_for<NE>([&](auto S) {
                v4i acc[9];
                multiply(S, acc);
                reduce(S, acc);
                __builtin_amdgcn_sched_barrier(0);
            });
        }
    }

    // Half of the entries, after the last channel block: the output transform of the channel sums
    // (it is linear, so it may as well run once on the sums as once per block).
    __device__ inline static void finish_lossless(const v4i* sums, v4i (&Y)[16]) {
        v4i er[6], ei[6];
        static_for<NE>([&](auto S) {
            constexpr Slot sl = half_slot(HALF, S);
            constexpr int v = ScaledSums<HALF>::sum_start(S);
            v4i im = {0, 0, 0, 0};
            if constexpr (!is_real(sl.entry)) im = sums[v + 1];
            place_entry<HALF, S>(sums[v], im, er, ei, Y);
            if constexpr (sl.last_in_row) __builtin_amdgcn_sched_barrier(0);   // row by row (see ScaledSums::finish)
        });
    }
};

// Lossless mode with joined channel sums (20 and 16 per half).
template <int HALF, int RING>
struct LosslessSums : LeanProducts<WG_LOSSLESS, HALF, RING> {
    using Lean = LeanProducts<WG_LOSSLESS, HALF, RING>;
    using Lean::kSums;
    __device__ inline void enter(LaneContext& cx, int8_t*, int) { Lean::prefetch(cx); }
    __device__ inline static void finish(const LaneContext&, const v4i* sums, v4i (&Y)[16]) { Lean::finish_lossless(sums, Y); }
};
// One object for a wave of either half.  (The two empty statements differ, so that the compiler does not join the ends of
// the branches: sums written through a choice of two addresses would live in memory.)
template <int RING>
struct EitherHalf {
    static constexpr int kSums = kChannelSums;
    int half;
    LosslessSums<0, RING> first;
    LosslessSums<1, RING> second;
    template <class F0, class F1>
    __device__ inline void choose(F0&& f0, F1&& f1) const {
        if (half == 0) { f0(); asm volatile("; half 0" ::: "memory"); }
        else           { f1(); asm volatile("; half 1" ::: "memory"); }
    }
    __device__ inline void prefetch(const LaneContext& cx) { choose([&]() { first.prefetch(cx); }, [&]() { second.prefetch(cx); }); }
    __device__ inline void enter(LaneContext& cx, int8_t*, int) { prefetch(cx); }
    __device__ inline void run(const LaneContext& cx, v4i* sums) { choose([&]() { first.run(cx, sums); }, [&]() { second.run(cx, sums); }); }
    __device__ inline void finish(const LaneContext& cx, const v4i* sums, v4i (&Y)[16]) const {
        choose([&]() { first.finish(cx, sums, Y); }, [&]() { second.finish(cx, sums, Y); });
    }
};

// Scaled mode over several channel blocks in a product wave of the role-specialised kernels: what it leaves to the vector
// ALU is what its SIMD has least of (the transform wave issues some 430 vector instructions per channel block there, each
// 4 clocks, and a matrix-core instruction keeps the vector ALU from other waves for 8 of its 16).  The low activation limb
// of every product accumulates over the channel blocks inside the matrix-core instructions; only the high limb starts from
// zero in each block, and one shift-and-add per register brings it in.  Re = Dr Wr - Di Wi keeps its two terms apart until
// finish().  24 / 22 vector instructions per accumulator register and half and channel block, where joining the limbs per
// block took 48 / 44 (56x56x256 N = 16 with int8 outputs 72.0 -> 64.9 us, together with the cheaper unpacking of StoredInt8).
// RING filter fragments and ARING activation fragments are in flight.  BUFFER: the former come by buffer loads (with eight product
// waves and signed int8: 56x56x256 N = 16 59.3 -> 57.3 us, 28x28x128 N = 32 13.35 -> 13.15, and every entry in one wave, 56x56x64 N = 256 94.7 -> 93.9; uint8 13.3 -> 13.55, the forms with
// resident accumulators 18.8 -> 19.3 at 14x14x512 N = 16, lossless 75.7 -> 76.5 at 56x56x256).
template <int HALF, int RING, int ARING, bool BUFFER>
struct ChainedSums {
    using Phase = ProductPhase<kScaledTwoPlanes, HALF>;
    static constexpr int PM = kScaledTwoPlanes;
    static constexpr int NE = Phase::NE, NB = Phase::NB;
    static constexpr int sum_start(int slot) {   // a real entry: one chain; complex: Dr Wr, Di Wi, Im
        int n = 0;
        for (int s = 0; s < slot; ++s) n += is_real(half_slot(HALF, s).entry) ? 1 : 3;
        return n;
    }
    static constexpr int a_start(int slot) {     // first activation fragment of a slot
        int n = 0;
        for (int s = 0; s < slot; ++s) n += num_a<PM>(half_slot(HALF, s).entry);
        return n;
    }
    static constexpr int kSums = sum_start(NE), NA = a_start(NE);
    static_assert(ARING >= 4 && NB >= RING, "an entry's fragments are there together");
    v4i ring[RING], aring[ARING];

    template <int F>
    __device__ inline static v4i load_a(const LaneContext& cx) {
        constexpr int slot = [] { int s = 0; while (a_start(s + 1) <= F) ++s; return s; }();
        return Phase::template load_a<slot, F - a_start(slot)>(cx);
    }
    __device__ inline void prefetch(const LaneContext& cx) {
        static_for<RING>([&](auto I) { ring[I] = Phase::template load_b<I, BUFFER>(cx); });
    }
    // The first block's prefetch, between the request for the reverse-scaling factors and their parking in `area`.
    __device__ inline void enter(LaneContext& cx, int8_t* area, int lane) {
        ParkedScales<HALF> scales;
        scales.ask(cx, lane);
        prefetch(cx);
        scales.park(cx, area, lane);
    }
    __device__ inline void run(const LaneContext& cx, v4i* sums) {
        static_for<ARING>([&](auto I) { aring[I] = load_a<I>(cx); });
        static_for<NE>([&](auto S) {
            constexpr int s = S;
            constexpr int entry = half_slot(HALF, s).entry;
            constexpr int b0 = b_start<PM>(HALF, s), a0 = a_start(s), v = sum_start(s);
            auto mul = [](v4i x, v4i w, v4i c) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(x, w, c, 0, 0, 0); };
            constexpr v4i zero = {0, 0, 0, 0};
            v4i high[3];
            if constexpr (is_real(entry)) {
                const v4i w = ring[b0 % RING];
                high[0] = mul(aring[a0 % ARING], w, zero);
                sums[v] = mul(aring[(a0 + 1) % ARING], w, sums[v]);
            } else {   // fragments: activations Re h, Re l, Im h, Im l; filters Re, Im
                const v4i wr = ring[b0 % RING], wi = ring[(b0 + 1) % RING];
                const v4i rh = aring[a0 % ARING], rl = aring[(a0 + 1) % ARING], ih = aring[(a0 + 2) % ARING], il = aring[(a0 + 3) % ARING];
                high[2] = mul(rh, wi, zero);
                high[0] = mul(rh, wr, zero);
                sums[v + 2] = mul(rl, wi, sums[v + 2]);
                sums[v] = mul(rl, wr, sums[v]);
                high[2] = mul(ih, wr, high[2]);
                high[1] = mul(ih, wi, zero);
                sums[v + 2] = mul(il, wr, sums[v + 2]);
                sums[v + 1] = mul(il, wi, sums[v + 1]);
            }
            static_for<num_a<PM>(entry)>([&](auto I) {
                if constexpr (a0 + I + ARING < NA) aring[(a0 + I) % ARING] = load_a<a0 + I + ARING>(cx);
            });
            static_for<num_b<PM>(entry)>([&](auto I) {
                if constexpr (b0 + I + RING < NB) ring[(b0 + I) % RING] = Phase::template load_b<b0 + I + RING, BUFFER>(cx);
            });
#pragma unroll
            for (int i = 0; i < (is_real(entry) ? 1 : 3); ++i) {
                sums[v + i] += high[i] << kByteLimbShift;
                asm volatile("" : "+v"(sums[v + i]));   // here, not in front of the next use of the sums with every high limb alive until then
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    // After the last channel block: the sums in the form ScaledSums<HALF>::finish takes.
    __device__ inline static void finish(const LaneContext& cx, const v4i* sums, v4i (&Y)[16]) {
        v4i joined[ScaledSums<HALF>::kSums];
        static_for<NE>([&](auto S) {
            constexpr int v = sum_start(S), o = ScaledSums<HALF>::sum_start(S);
            if constexpr (is_real(half_slot(HALF, S).entry)) {
                joined[o] = sums[v];
            } else {
                joined[o] = sums[v] - sums[v + 1];
                joined[o + 1] = sums[v + 2];
            }
        });
        ScaledSums<HALF>::template finish<0, true>(cx, joined, Y);
    }
};

// Scaled mode in the role-specialised kernel: every limb product of every entry a wave owns has
// its own matrix-core accumulator for the whole kernel (two per real entry: high and low
// activation limb; four per complex entry: Re and Im, each high and low; 36 per wave), so a
// channel block costs a product wave nothing but fragment loads and matrix-core instructions
// and the vector ALU is left to the transform wave.  The limbs are joined, the reverse scaling
// applied and the output transform run once, on the finished channel sums.
template <int HALF>
struct ResidentScaled {
    static constexpr int MODE = WG_SCALED;
    using Phase = ProductPhase<MODE, HALF>;
    static constexpr int NE = Phase::NE, NB = Phase::NB;
    static constexpr int kRing = 8;
    static constexpr int acc_start(int slot) {
        int n = 0;
        for (int s = 0; s < slot; ++s) n += is_real(half_slot(HALF, s).entry) ? 2 : 4;
        return n;
    }
    static constexpr int kSums = acc_start(NE);
    v4i ring[kRing];

    __device__ inline void prefetch(const LaneContext& cx) {
        static_for<(NB < kRing ? NB : kRing)>([&](auto I) { ring[I] = Phase::template load_b<I>(cx); });
    }
    // The first block's prefetch, between the request for the reverse-scaling factors and their parking in `area`.
    __device__ inline void enter(LaneContext& cx, int8_t* area, int lane) {
        ParkedScales<HALF> scales;
        scales.ask(cx, lane);
        prefetch(cx);
        scales.park(cx, area, lane);
    }
    __device__ inline void run(const LaneContext& cx, v4i* sums) {
        static_for<NE>([&](auto S) {
            constexpr int s = S;
            constexpr int entry = half_slot(HALF, s).entry;
            constexpr int b0 = b_start<MODE>(HALF, s);
            constexpr int v = acc_start(s);
            v4i afr[4];
            static_for<num_a<MODE>(entry)>([&](auto I) { afr[I] = Phase::template load_a<s, I>(cx); });
            static_for<num_ops<MODE>(entry)>([&](auto I) {
                constexpr Op op = entry_op<MODE>(entry, I);
                sums[v + op.acc] = __builtin_amdgcn_mfma_i32_16x16x64_i8(afr[op.a], ring[(b0 + op.b) % kRing], sums[v + op.acc], 0, 0, 0);
            });
            static_for<num_b<MODE>(entry)>([&](auto I) {
                if constexpr (b0 + I + kRing < NB) ring[(b0 + I) % kRing] = Phase::template load_b<b0 + I + kRing>(cx);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    __device__ inline static void finish(const LaneContext& cx, const v4i* sums, v4i (&Y)[16]) {
        v4i er[6], ei[6];
        static_for<NE>([&](auto S) {
            constexpr Slot sl = half_slot(HALF, S);
            constexpr int v = acc_start(S);
            v4i re = (sums[v] << kByteLimbShift) + sums[v + 1], im = {0, 0, 0, 0};
            if constexpr (!is_real(sl.entry)) im = (sums[v + 2] << kByteLimbShift) + sums[v + 3];
            const ReverseScale unscale = parked_scale<S>(cx);   // Section 4.2
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                re[q] = unscale(re[q]);
                if constexpr (!is_real(sl.entry)) im[q] = unscale(im[q]);
            }
            place_entry<HALF, S>(re, im, er, ei, Y);
        });
    }
};
}  // namespace
}  // namespace wg
