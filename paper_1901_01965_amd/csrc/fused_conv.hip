// The whole hot path in one kernel: input transform (Section 3.3-3.4) of a block
// of 16 tiles into int8 operand planes held in LDS, the Winograd-domain
// products of Section 3.4 against 32 filters on the int8 matrix cores, and the
// output transform accumulated on the fly, so neither the transformed
// activations nor the 36 accumulator planes ever travel through HBM.
//
// The output transform Y = A^T M A is linear in M, and M is a sum over input
// channels, so each finished row of M (for one 64-channel block) is reduced by
// the row rule of A^T at once and added into the 16 outputs of the tile.  That is
// valid for any number of channel blocks in lossless mode.  The reverse scaling of
// Section 4.2 is not linear (it rounds): with more than one channel block, scaled
// mode keeps the channel sums of all of a wave's entries in registers (18 sums of
// four registers per wave) across the channel blocks and scales and reduces them
// once at the end.
//
// This kernel is bound by vector ALU work (transform, limb re-assembly, output
// transform) and memory latency, not by the matrix cores, so it trades
// multiplications for vector work and traffic: a 12-bit x 12-bit
// product is taken as the four limb products hh, hl, lh, ll (two activation and
// two filter planes per value) and a complex product as its four real products,
// instead of the three-multiplication forms of Section 3.1 that the staged
// contraction kernel uses; those would need half again as many operand planes.
#include <algorithm>

#include "act_scale.h"
#include "product_core.h"
#include "roles_conv.h"

namespace wg {
namespace {

// grid: (ceil(T/16), ceil(K/32)), or ceil(K/64) for WIDE.  256 threads: in the transform phase one thread per (tile,
// four channels); in the product phase wave w owns filter block (w & 1) and half of the
// rows of M (w >> 1: rows 0,1,2 or rows 5,3); all four waves stage their partial outputs
// in LDS and the block stores the sums with full-line writes.
// SUMS: scaled mode keeps channel sums and scales them at the end (see ScaledSums): needed with
// more than one channel block, and used for every scaled WIDE workgroup.
// WIDE: the workgroup covers 64 filters instead of 32: the transform of a
// channel block is followed by two passes over the entries, one per 32 filters, each with its own
// outputs; used when there are more workgroups than compute units, where halving the number of
// repeated transforms outweighs the longer workgroup.
// Q8: the finished outputs are requantised (and pooled) to int8 at q8.out instead of stored to y.
// ENC: how the activation bytes are read (signed int8, or uint8 with a zero point: Section 4.1); the latter only
// with the load paths that select padding explicitly, and with blobs made from uint8 filters.
template <int LAYOUT, int LOAD, int MODE, bool SUMS, bool WIDE, bool Q8, class ENC = SignedInt8>
__device__ __forceinline__ void fused_conv_body(const int8_t* __restrict__ x, const uint8_t* __restrict__ blob,
                                                size_t table_off, size_t planes_off, int32_t* __restrict__ y,
                                                const Problem p, const Int8Epilogue q8, const GridOrder order, const ENC enc = ENC{}) {
    static_assert(LOAD != kLoadDirect || ENC::kMagic == kBlobMagic, "direct transfers deliver zero bytes for absent pixels");
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kblock = wave & 1, half = wave >> 1;
    int bx, by;
    order.place(bx, by);
    const int tile0 = bx * kFusedTiles;
    constexpr int NPASS = WIDE ? 2 : 1;
    const int k0 = by * (kFusedFilters * NPASS);
    const int k = k0 + kblock * 16 + (lane & 15);

    // The activation patch of the first channel block does not depend on the blob and is the
    // longest wait of the kernel: its requests go out before anything else.
    DirectPatch direct;
    int8_t* raw_wave = lds + kLdsBytes + wave * kRawWaveBytes;
    if constexpr (LOAD == kLoadDirect) {
        const int dt = tile0 + 4 * wave + ((lane & 15) >> 2);   // the tile this lane moves pieces of
        int dn = 0, dty = 0, dtx = 0;
        if (dt < p.T) decode_tile(p, dt, dn, dty, dtx);
        direct.init(p, dn, dty, dtx, lane);
        direct.issue(x, p, 0, lane, raw_wave);
    }

    // transform-phase identity
    // every lane decodes tile (lane & 15) of the block once; the transform phase fetches the
    // coordinates of its own tile (tid / 16) from that lane
    int my_n = 0, my_ty = 0, my_tx = 0;
    if (tile0 + (lane & 15) < p.T) decode_tile(p, tile0 + (lane & 15), my_n, my_ty, my_tx);
    const int a_tile = tid >> 4, a_cq = tid & 15;
    const int a_t = tile0 + a_tile;
    const int a_tx = __shfl(my_tx, a_tile), a_ty = __shfl(my_ty, a_tile), a_n = __shfl(my_n, a_tile);
    OperandSplitter<MODE == WG_SCALED ? kSplitByteLimbs : kSplitTwoLimb, LdsPlaneSink> out;
    out.sink.base = lds + lds_slot(a_cq >> 2, a_tile) * 16 + (a_cq & 3) * 4;

    LaneContext cx;
    cx.a_lds = lds + lds_slot(lane >> 4, lane & 15) * 16;
    cx.table_k = reinterpret_cast<const ScaleEntry*>(blob + table_off) + (size_t)k * kEntries;
    constexpr int NP = MODE == WG_LOSSLESS ? 138 : 46;
    const int8_t* const b_wave = filter_fragments(blob + planes_off, k - (lane & 15), p.Kp, NP);
    cx.b_lane = fragment_lane(lane);
    const size_t b_block_stride = (size_t)(p.Kp >> 4) * NP * kFilterFragBytes;

    v4i Yall[NPASS][16];
#pragma unroll
    for (int pass = 0; pass < NPASS; ++pass)
#pragma unroll
        for (int i = 0; i < 16; ++i) Yall[pass][i] = (v4i){0, 0, 0, 0};
    v4i (&Y)[16] = Yall[0];

    // The blob header is checked while the patch requests are in flight.
    constexpr bool VEC4 = LOAD == kLoadDwords;
    uint32_t patch[6][6];
    if constexpr (LOAD != kLoadDirect) {
        if (a_t < p.T) load_patch<LAYOUT, VEC4>(x, p, a_n, a_ty, a_tx, 4 * a_cq, patch, enc);
    }
    if (!blob_matches(reinterpret_cast<const BlobHeader*>(blob), p.K, p.Cf, MODE, ENC::kMagic)) return;

    ProductPhase<MODE, 0> phase0;
    ProductPhase<MODE, 1> phase1;
    static_assert(!SUMS || MODE == WG_SCALED, "channel sums are kept apart in scaled mode only");
    v4i sums[SUMS ? NPASS : 1][SUMS ? kChannelSums : 1];
    if constexpr (SUMS) {
#pragma unroll
        for (int pass = 0; pass < NPASS; ++pass)
#pragma unroll
            for (int i = 0; i < kChannelSums; ++i) sums[pass][i] = (v4i){0, 0, 0, 0};
    }
    static_assert(ProductPhase<MODE, 0>::NPRE == kFilterPrefetch && ProductPhase<MODE, 1>::NPRE == kFilterPrefetch,
                  "the wait for the direct patch transfer counts the filter fragments requested after it");
    for (int cb = 0; cb < p.CB; ++cb) {
        cx.b_glob = b_wave + cb * b_block_stride;
        if (half == 0) phase0.prefetch(cx); else phase1.prefetch(cx);
        if (cb > 0) {   // everyone is done reading the previous block's planes
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
        }
        if constexpr (LOAD == kLoadDirect) {
            // the patch pieces were requested before the sixteen filter fragments above, and
            // loads complete in order; the pieces a thread reads were moved by its own wave
            asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
            DirectPatch::read(raw_wave, lane, patch);
            if (cb + 1 < p.CB) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the raw area has been read
                direct.issue(x, p, cb + 1, lane, raw_wave);
            }
        }
        if (a_t < p.T) {
            bias_patch(p, a_ty, a_tx, cb * kCBlock + 4 * a_cq, patch, enc);
            transform_patch(patch, out, enc);
            if constexpr (LOAD != kLoadDirect) {
                if (cb + 1 < p.CB)   // next block's patch travels while this block's products run
                    load_patch<LAYOUT, VEC4>(x, p, a_n, a_ty, a_tx, (cb + 1) * kCBlock + 4 * a_cq, patch, enc);
            }
        }
        // the operand planes are complete once every wave's LDS writes have landed; global
        // requests (filter fragments, the next block's patch) stay in flight across the barrier
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        if constexpr (SUMS && WIDE) {
            if (half == 0) {
                ScaledSums<0>::template run<0, 2>(cx, phase0.bring, sums[0]);
                ScaledSums<0>::template run<1, 2>(cx, phase0.bring, sums[1]);
            } else {
                ScaledSums<1>::template run<0, 2>(cx, phase1.bring, sums[0]);
                ScaledSums<1>::template run<1, 2>(cx, phase1.bring, sums[1]);
            }
        } else if constexpr (SUMS) {
            if (half == 0) ScaledSums<0>::run(cx, phase0.bring, sums[0]); else ScaledSums<1>::run(cx, phase1.bring, sums[0]);
        } else if constexpr (WIDE) {
            if (half == 0) { phase0.template run<0, 2>(cx, Yall[0]); phase0.template run<1, 2>(cx, Yall[1]); }
            else           { phase1.template run<0, 2>(cx, Yall[0]); phase1.template run<1, 2>(cx, Yall[1]); }
        } else {
            if (half == 0) phase0.run(cx, Y); else phase1.run(cx, Y);
        }
    }
    if constexpr (SUMS) {
        if (half == 0) ScaledSums<0>::template finish<0>(cx, sums[0], Yall[0]);
        else           ScaledSums<1>::template finish<0>(cx, sums[0], Yall[0]);
        if constexpr (WIDE) {
            if (half == 0) ScaledSums<0>::template finish<1>(cx, sums[1], Yall[1]);
            else           ScaledSums<1>::template finish<1>(cx, sums[1], Yall[1]);
        }
    }

    // ---- add the two halves and store ------------------------------------------------------
    StoreContext sc;
    sc.lds = lds; sc.tid = tid; sc.lane = lane; sc.rnd = MODE == WG_SCALED ? 8 : 0; sc.y = y;
    locate_tile<LAYOUT>(sc, p, tile0);
#pragma unroll
    for (int pass = 0; pass < NPASS; ++pass) {
        __syncthreads();   // the operand planes (or the previous pass's staged outputs) are dead
        stage_outputs(lds, lane, half, kblock, Yall[pass]);
        __syncthreads();
        store_staged<LAYOUT, Q8 ? kOutInt8 : kOutInt32, true>(sc, p, q8, k0 + pass * kFusedFilters);
    }
}

template <int LAYOUT, int LOAD, int MODE, bool SUMS, bool WIDE>
__global__ __launch_bounds__(256) void fused_conv_kernel(const int8_t* __restrict__ x,
                                                         const uint8_t* __restrict__ blob, size_t table_off,
                                                         size_t planes_off, int32_t* __restrict__ y, Problem p, GridOrder order) {
    fused_conv_body<LAYOUT, LOAD, MODE, SUMS, WIDE, false>(x, blob, table_off, planes_off, y, p, Int8Epilogue{}, order);
}

template <int LAYOUT, int LOAD, int MODE, bool SUMS, bool WIDE>
__global__ __launch_bounds__(256) void fused_conv_int8_kernel(const int8_t* __restrict__ x,
                                                              const uint8_t* __restrict__ blob, size_t table_off,
                                                              size_t planes_off, Problem p, Int8Epilogue q8, GridOrder order) {
    fused_conv_body<LAYOUT, LOAD, MODE, SUMS, WIDE, true>(x, blob, table_off, planes_off, nullptr, p, q8, order);
}

template <int LAYOUT, int LOAD, int MODE, bool SUMS>
__global__ __launch_bounds__(256) void fused_conv_u8_kernel(const int8_t* __restrict__ x, ZeroPointU8 zero,
                                                            const uint8_t* __restrict__ blob, size_t table_off,
                                                            size_t planes_off, int32_t* __restrict__ y, Problem p, GridOrder order) {
    fused_conv_body<LAYOUT, LOAD, MODE, SUMS, false, false, ZeroPointU8>(x, blob, table_off, planes_off, y, p, Int8Epilogue{}, order, zero);
}

template <int LAYOUT, int LOAD, int MODE, bool SUMS, bool WIDE, bool Q8>
hipError_t launch(const int8_t* x, const uint8_t* blob, const BlobLayout& bl, int32_t* y, const Problem& p,
                  const Int8Epilogue& q8, hipStream_t s) {
    constexpr int lds_bytes = kLdsBytes + (LOAD == kLoadDirect ? kRawBytes : 0);
    const void* kernel = Q8 ? reinterpret_cast<const void*>(&fused_conv_int8_kernel<LAYOUT, LOAD, MODE, SUMS, WIDE>)
                            : reinterpret_cast<const void*>(&fused_conv_kernel<LAYOUT, LOAD, MODE, SUMS, WIDE>);
    static LdsLimitOnce lds_limit;   // per template instance
    if (hipError_t e = lds_limit.set(kernel, lds_bytes)) return e;
    dim3 grid(ceil_div(p.T, kFusedTiles), ceil_div(p.K, kFusedFilters * (WIDE ? 2 : 1)));
    const GridOrder order(grid, workgroup_order(p, MODE, kFusedFilters * (WIDE ? 2 : 1)));
    if constexpr (Q8)
        fused_conv_int8_kernel<LAYOUT, LOAD, MODE, SUMS, WIDE><<<grid, 256, lds_bytes, s>>>(x, blob, bl.table_off, bl.planes_off, p, q8, order);
    else
        fused_conv_kernel<LAYOUT, LOAD, MODE, SUMS, WIDE><<<grid, 256, lds_bytes, s>>>(x, blob, bl.table_off, bl.planes_off, y, p, order);
    return hipGetLastError();
}

template <int LAYOUT, int LOAD, bool Q8>
hipError_t launch_mode(const int8_t* x, const uint8_t* blob, const BlobLayout& bl, int32_t* y, const Problem& p,
                       int mode, const Int8Epilogue& q8, hipStream_t s) {
    // 64 filters per workgroup once the 32-filter grid would need more than one round of the
    // compute units (Kp is a multiple of 64).  Only the direct-transfer variants have the
    // registers for it (the others hold a patch in registers across the product phase).
    if constexpr (LOAD == kLoadDirect) {
        const long long workgroups = (long long)ceil_div(p.T, kFusedTiles) * ceil_div(p.K, kFusedFilters);
        if (workgroups > compute_units()) {
            if (mode == WG_LOSSLESS) return launch<LAYOUT, LOAD, WG_LOSSLESS, false, true, Q8>(x, blob, bl, y, p, q8, s);
            // scaled mode keeps channel sums here also for a single channel block: the variant that
            // reduces each entry at once needs more registers than a wave has when it covers 64 filters
            return launch<LAYOUT, LOAD, WG_SCALED, true, true, Q8>(x, blob, bl, y, p, q8, s);
        }
    }
    if (mode == WG_LOSSLESS) return launch<LAYOUT, LOAD, WG_LOSSLESS, false, false, Q8>(x, blob, bl, y, p, q8, s);
    if (p.CB == 1) return launch<LAYOUT, LOAD, WG_SCALED, false, false, Q8>(x, blob, bl, y, p, q8, s);
    return launch<LAYOUT, LOAD, WG_SCALED, true, false, Q8>(x, blob, bl, y, p, q8, s);
}

template <bool Q8>
hipError_t launch_layout(const int8_t* x, const uint8_t* b, const BlobLayout& bl, int32_t* y, const Problem& p,
                         int layout, int mode, const Int8Epilogue& q8, hipStream_t s) {
    if (layout == WG_NHWC && p.C % 16 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0)
        return launch_mode<WG_NHWC, kLoadDirect, Q8>(x, b, bl, y, p, mode, q8, s);
    if (layout == WG_NHWC && p.C % 4 == 0) return launch_mode<WG_NHWC, kLoadDwords, Q8>(x, b, bl, y, p, mode, q8, s);
    if (layout == WG_NHWC) return launch_mode<WG_NHWC, kLoadBytes, Q8>(x, b, bl, y, p, mode, q8, s);
    return launch_mode<WG_NCHW, kLoadBytes, Q8>(x, b, bl, y, p, mode, q8, s);
}

// ---- activations scaled as well (act_scale.h) in one kernel, for calls without scratch memory -------------------
constexpr int kActNpOff = kLdsBytes;
constexpr int kActRqOff = kActNpOff + kActNpBytes;
constexpr int kActLdsBytes = kActRqOff + kActRqBytes;

// Product phase: the channel sums of a wave's entries (18 of four registers) are the matrix cores' accumulators.
//   real:    sum += D W;    complex: Re += Dr Wr + Di (-Wi),  Im += Dr Wi + Di Wr
// Filter fragments come from the scaled blob in ProductPhase<WG_SCALED>'s order (W; Wr, Wi, -Wi).
template <int HALF>
struct BothScaledSums {
    using Phase = ProductPhase<WG_SCALED, HALF>;
    static constexpr int NE = Phase::NE, NB = Phase::NB;
    static constexpr int sum_start(int slot) { return ScaledSums<HALF>::sum_start(slot); }
    template <int SLOT, int I>
    __device__ inline static v4i load_a(const LaneContext& cx) {
        constexpr int entry = half_slot(HALF, SLOT).entry;
        constexpr int plane = is_real(entry) ? entry : kRealEntries + 2 * (entry - kRealEntries) + I;
        return *reinterpret_cast<const v4i*>(cx.a_lds + plane * kPlaneBytes);
    }
    __device__ inline static void run(const LaneContext& cx, v4i (&bring)[kFilterPrefetch], v4i (&sums)[kChannelSums]) {
        v4i afr[2][2];
        afr[0][0] = load_a<0, 0>(cx);
        if constexpr (!is_real(half_slot(HALF, 0).entry)) afr[0][1] = load_a<0, 1>(cx);
        static_for<NE>([&](auto S) {
            constexpr int s = S;
            constexpr int entry = half_slot(HALF, s).entry;
            constexpr int b0 = b_start<WG_SCALED>(HALF, s), v = sum_start(s);
            if constexpr (s + 1 < NE) {
                afr[(s + 1) & 1][0] = load_a<s + 1, 0>(cx);
                if constexpr (!is_real(half_slot(HALF, s + 1).entry)) afr[(s + 1) & 1][1] = load_a<s + 1, 1>(cx);
            }
            auto mac = [&](int a, int b, int sum) {
                sums[sum] = __builtin_amdgcn_mfma_i32_16x16x64_i8(afr[s & 1][a], bring[(b0 + b) % kFilterPrefetch], sums[sum], 0, 0, 0);
            };
            if constexpr (is_real(entry)) {
                mac(0, 0, v);
            } else {
                mac(0, 0, v);        // Dr Wr
                mac(0, 1, v + 1);    // Dr Wi
                mac(1, 2, v);        // Di (-Wi)
                mac(1, 0, v + 1);    // Di Wr
            }
            static_for<num_b<WG_SCALED>(entry)>([&](auto I) {
                if constexpr (b0 + I + kFilterPrefetch < NB)
                    bring[(b0 + I) % kFilterPrefetch] = Phase::template load_b<b0 + I + kFilterPrefetch>(cx);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    // After the last channel block: the filter's reverse scaling, then the tile's (register q of a lane belongs to
    // tile 4 (lane / 16) + q), and the output transform.
    __device__ inline static void finish(const LaneContext& cx, const uint32_t* rq_tab, int lane, const v4i (&sums)[kChannelSums],
                                         v4i (&Y)[16]) {
        v4i er[6], ei[6];
        static_for<NE>([&](auto S) {
            constexpr Slot sl = half_slot(HALF, S);
            constexpr int v = sum_start(S);
            v4i re = sums[v], im = {0, 0, 0, 0};
            if constexpr (!is_real(sl.entry)) im = sums[v + 1];
            const ReverseScale filter_side(cx.table_k[sl.entry]);
            const v4i rq = *reinterpret_cast<const v4i*>(rq_tab + sl.entry * 16 + 4 * (lane >> 4));
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const ReverseScale tile_side((int)(((uint32_t)rq[q] >> 16) & 255u), (int)((uint32_t)rq[q] >> 24));
                re[q] = tile_side(filter_side(re[q]));
                if constexpr (!is_real(sl.entry)) im[q] = tile_side(filter_side(im[q]));
            }
            place_entry<HALF, S>(re, im, er, ei, Y);
        });
    }
};

// grid (ceil(T/16), ceil(K/32)), 256 threads with the roles of fused_conv_body; the blob is a WG_SCALED one of signed int8
// filters.  Pass 1 transforms every channel block of the workgroup's 16 tiles and keeps the running maxima; each
// thread then looks up the factors of one or two (tile, entry) pairs; pass 2 transforms again (the patches now come
// from the caches), scales, and multiplies.  act_table (may be null) receives int32 [T][26][4] = (n, p, r, q).
template <int LAYOUT, int LOAD>
__global__ __launch_bounds__(256) void fused_conv_act_scaled_kernel(const int8_t* __restrict__ x, const uint8_t* __restrict__ blob,
                                                                    size_t table_off, size_t planes_off, int32_t* __restrict__ y,
                                                                    int32_t* __restrict__ act_table, const Problem p) {
    static_assert(LOAD != kLoadDirect, "the patch is held in registers");
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kblock = wave & 1, half = wave >> 1;
    const int tile0 = blockIdx.x * kFusedTiles, k0 = blockIdx.y * kFusedFilters;
    const int k = k0 + kblock * 16 + (lane & 15);
    if (!blob_matches(reinterpret_cast<const BlobHeader*>(blob), p.K, p.Cf, WG_SCALED)) return;

    int my_n = 0, my_ty = 0, my_tx = 0;
    if (tile0 + (lane & 15) < p.T) decode_tile(p, tile0 + (lane & 15), my_n, my_ty, my_tx);
    const int a_tile = tid >> 4, a_cq = tid & 15;
    const int a_t = tile0 + a_tile;
    const int a_tx = __shfl(my_tx, a_tile), a_ty = __shfl(my_ty, a_tile), a_n = __shfl(my_n, a_tile);
    uint32_t* np_tab = reinterpret_cast<uint32_t*>(lds + kActNpOff);
    uint32_t* rq_tab = reinterpret_cast<uint32_t*>(lds + kActRqOff);
    constexpr bool VEC4 = LOAD == kLoadDwords;
    uint32_t patch[6][6];

    // ---- pass 1: largest magnitude per (tile, entry) over all channels --------------------------------------
    s16x2 mx[kEntries];
#pragma unroll
    for (int e = 0; e < kEntries; ++e) mx[e] = (s16x2){0, 0};
    if (a_t < p.T) {
        load_patch<LAYOUT, VEC4>(x, p, a_n, a_ty, a_tx, 4 * a_cq, patch);
        for (int cb = 0; cb < p.CB; ++cb) {
            bias_patch(p, a_ty, a_tx, cb * kCBlock + 4 * a_cq, patch);
            uint32_t now[6][6];
#pragma unroll
            for (int i = 0; i < 36; ++i) now[i / 6][i % 6] = patch[i / 6][i % 6];
            // the next block's patch, or the first block's again for pass 2, travels meanwhile
            load_patch<LAYOUT, VEC4>(x, p, a_n, a_ty, a_tx, (cb + 1 < p.CB ? cb + 1 : 0) * kCBlock + 4 * a_cq, patch);
            transform_patch(now, MaxKeeper{mx});
        }
    }
    // over the sixteen threads of a tile (consecutive lanes), two entries per register
    s16x2 pm[kEntries / 2];
#pragma unroll
    for (int j = 0; j < kEntries / 2; ++j) {
        pm[j] = (s16x2){max(mx[2 * j].x, mx[2 * j].y), max(mx[2 * j + 1].x, mx[2 * j + 1].y)};
#pragma unroll
        for (int off = 1; off < 16; off <<= 1)
            pm[j] = __builtin_elementwise_max(pm[j], as_s16x2((uint32_t)__shfl_xor((int)as_u32(pm[j]), off)));
    }
    {   // thread (tile, cq) looks up entry cq of its tile, and entry 16 + cq if there is one
        int mine[2] = {0, 0};
#pragma unroll
        for (int e = 0; e < kEntries; ++e)
            if (a_cq == (e & 15)) mine[e >> 4] = (e & 1) ? pm[e / 2].y : pm[e / 2].x;
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            const int e = 16 * part + a_cq;
            if (e >= kEntries) break;
            const uint32_t entry = kActScale.v[min(mine[part], kActMax)];
            np_tab[a_tile * kEntries + e] = act_factors(entry);
            rq_tab[e * 16 + a_tile] = entry;
            if (act_table != nullptr && blockIdx.y == 0 && a_t < p.T)
                *reinterpret_cast<v4i*>(act_table + ((size_t)a_t * kEntries + e) * 4) = act_table_row(entry);
        }
    }
    __syncthreads();

    // ---- pass 2: scaled operands, products --------------------------------------------------------------------
    ScaledPlanes out;
    out.sink.base = lds + lds_slot(a_cq >> 2, a_tile) * 16 + (a_cq & 3) * 4;
    out.np = np_tab + a_tile * kEntries;
    LaneContext cx;
    cx.a_lds = lds + lds_slot(lane >> 4, lane & 15) * 16;
    cx.table_k = reinterpret_cast<const ScaleEntry*>(blob + table_off) + (size_t)k * kEntries;
    constexpr int NP = 46;
    const int8_t* const b_wave = filter_fragments(blob + planes_off, k - (lane & 15), p.Kp, NP);
    cx.b_lane = fragment_lane(lane);
    const size_t b_block_stride = (size_t)(p.Kp >> 4) * NP * kFilterFragBytes;
    ProductPhase<WG_SCALED, 0> phase0;
    ProductPhase<WG_SCALED, 1> phase1;
    v4i sums[kChannelSums];
#pragma unroll
    for (int i = 0; i < kChannelSums; ++i) sums[i] = (v4i){0, 0, 0, 0};
    for (int cb = 0; cb < p.CB; ++cb) {
        cx.b_glob = b_wave + cb * b_block_stride;
        if (half == 0) phase0.prefetch(cx); else phase1.prefetch(cx);
        if (cb > 0) {   // everyone is done reading the previous block's planes
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
        }
        if (a_t < p.T) {
            bias_patch(p, a_ty, a_tx, cb * kCBlock + 4 * a_cq, patch);
            transform_patch(patch, out);
            if (cb + 1 < p.CB) load_patch<LAYOUT, VEC4>(x, p, a_n, a_ty, a_tx, (cb + 1) * kCBlock + 4 * a_cq, patch);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        if (half == 0) BothScaledSums<0>::run(cx, phase0.bring, sums); else BothScaledSums<1>::run(cx, phase1.bring, sums);
    }
    v4i Y[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) Y[i] = (v4i){0, 0, 0, 0};
    if (half == 0) BothScaledSums<0>::finish(cx, rq_tab, lane, sums, Y); else BothScaledSums<1>::finish(cx, rq_tab, lane, sums, Y);

    StoreContext sc;
    sc.lds = lds; sc.tid = tid; sc.lane = lane; sc.rnd = 8; sc.y = y;
    locate_tile<LAYOUT>(sc, p, tile0);
    __syncthreads();   // the operand planes are dead (the tables lie behind them)
    stage_outputs(lds, lane, half, kblock, Y);
    __syncthreads();
    store_staged<LAYOUT, kOutInt32, true>(sc, p, Int8Epilogue{}, k0);
}

template <int LAYOUT, int LOAD>
hipError_t launch_act_scaled(const int8_t* x, const uint8_t* blob, const BlobLayout& bl, int32_t* y, int32_t* act_table, const Problem& p,
                             hipStream_t s) {
    static LdsLimitOnce lds_limit;   // per template instance
    if (hipError_t e = lds_limit.set(reinterpret_cast<const void*>(&fused_conv_act_scaled_kernel<LAYOUT, LOAD>), kActLdsBytes)) return e;
    dim3 grid(ceil_div(p.T, kFusedTiles), ceil_div(p.K, kFusedFilters));
    fused_conv_act_scaled_kernel<LAYOUT, LOAD><<<grid, 256, kActLdsBytes, s>>>(x, blob, bl.table_off, bl.planes_off, y, act_table, p);
    return hipGetLastError();
}

template <int LAYOUT, int LOAD, int MODE, bool SUMS>
hipError_t launch_u8(const int8_t* x, ZeroPointU8 zero, const uint8_t* blob, const BlobLayout& bl, int32_t* y, const Problem& p,
                     hipStream_t s) {
    static LdsLimitOnce lds_limit;   // per template instance
    if (hipError_t e = lds_limit.set(reinterpret_cast<const void*>(&fused_conv_u8_kernel<LAYOUT, LOAD, MODE, SUMS>), kLdsBytes)) return e;
    dim3 grid(ceil_div(p.T, kFusedTiles), ceil_div(p.K, kFusedFilters));
    fused_conv_u8_kernel<LAYOUT, LOAD, MODE, SUMS><<<grid, 256, kLdsBytes, s>>>(x, zero, blob, bl.table_off, bl.planes_off, y, p,
                                                                              GridOrder(grid, workgroup_order(p, MODE, kFusedFilters)));
    return hipGetLastError();
}

template <int LAYOUT, int LOAD>
hipError_t launch_u8_mode(const int8_t* x, ZeroPointU8 zero, const uint8_t* blob, const BlobLayout& bl, int32_t* y, const Problem& p,
                          int mode, hipStream_t s) {
    if (mode == WG_LOSSLESS) return launch_u8<LAYOUT, LOAD, WG_LOSSLESS, false>(x, zero, blob, bl, y, p, s);
    if (p.CB == 1) return launch_u8<LAYOUT, LOAD, WG_SCALED, false>(x, zero, blob, bl, y, p, s);
    return launch_u8<LAYOUT, LOAD, WG_SCALED, true>(x, zero, blob, bl, y, p, s);
}

// Test hooks (see winograd_c.h).
std::atomic<int> g_stream_workgroups{0}, g_stream_variant{0}, g_scaled_variant{0};

// How a convolution is run where the fast loads apply (channels-last, C % 4 = 0, as given or as a copy).
struct Plan {
    bool copies;         // through a channels-last copy in scratch memory
    bool planes;         // channel-major activations read as they are: split channels, or the limb-pair kernel
    int splits, blocks;  // > 1: the channel blocks are dealt to `splits` workgroups each, `blocks` per workgroup
};

// Deep layers with few tiles leave most of the chip idle while a workgroup walks through its channel blocks one after the
// other.  Dealing the blocks to several workgroups takes a second kernel that adds the splits and finishes.  CB channel blocks in
// one workgroup against b in each of W, whose partial sums are written and read (36 per tile and filter in scaled mode, 16
// otherwise).  Fitted to layers of 128 .. 896 channels and K = 16 .. 512 filters that fill at most half the chip, with filters
// that are not in the L2, as in a network (us; 248 layers in scaled mode, 226 in lossless mode, off by 4 - 8 % on average):
//   lossless: 4.3 + 3.3 b + W / 50 split; one kernel, which is the limb-pair form with 16 filters per workgroup there (lossless_conv.hip),
//             2.1 + 2.6 CB + W16 / 120 for W16 workgroups with 16-byte pieces, 1.6 + 3.3 CB with 4-byte loads, both + CB min(K, 256) / 1500 for the
//             filters that come from memory, unless filter blocks are dealt out first (split / one kernel: 256 -> 256 at 56x56, N = 1, 14.9, 13.8;
//             256 -> 512 at 28x28, N = 1, 12.1, 12.8; 128 -> 64 at 14x14, N = 1, 9.1, 7.7; 256 -> 256 at 14x14, N = 1, 9.1, 12.4; of 226 layers the choice
//             is 0.2 % from the better one on average, 12 % at most; with 4.0 it was 1.0 % and 26 %);
//             on channel-major tensors 4.0 + 4.4 b + W / 53 + 6.4 per million outputs split and 2.5 + 3.9 CB + W16 / 120 (112 -> 448 at 58x29,
//             N = 1: 18.5, 12.7); with a copy, where there are more than two blocks, 9.3 + 2.75 CB and 5.1 + 3.7 b + W / 68 + 7.1 per million
//             outputs split (256 -> 128 at 72x72, N = 1: 20.3, 19.2);
//             4.8 + 3.27 b + W / 50 + CB K / 2700 and 5.7 + 2.68 CB, both with a copy
//   scaled:   5.9 + 1.65 CB in one kernel, 7.4 + 3.0 b + W / 29 split, 0.5 more up to three blocks, where the fit is 1.2 too high for one kernel
//             (512 -> 512 at 17x12, N = 1: 18.8, 15.0; 256 -> 64 at 38x26, N = 2: 11.4, 12.4; 176 -> 64 at 8x8, N = 1: 9.1, 9.9);
//             on channel-major tensors 8.0 + 1.75 CB, with a copy, and 8.6 + 2.9 b + W / 24 (256 -> 16 at 42x17, N = 2: 14.8, 12.0; 192 -> 512 at 23x23,
//             N = 1: 13.7, 16.8; 118 layers after the finishing kernel reads 16 bytes at a time, off by 5 and 4 %; 0.3 in favour of one kernel)
// and 3.9 b - 2.2 more where the split kernels cannot read 16-byte pieces (N = 2, 324 -> 512 at 28x28, lossless: 21.6, 32.8).  The
// kernels that transform on waves of their own take 0.6 less with up to 32 filters (250 drawn layers; 272 -> 16 at 17x17, N = 10, scaled: 13.3, 14.1;
// 116 -> 16 at 64x7, N = 15, lossless: 10.4, 11.2), unless it needs a copy that the split kernels do without (`planes`; 480 -> 32 at
// 81x81, N = 1, scaled: 25.7, 21.2).
// pairs: one kernel would be the limb-pair form.
bool split_pays(int mode, const Problem& p, int b, int W, bool pieces, bool planes, bool pairs) {
    const double w16 = (double)ceil_div(p.T, kFusedTiles) * ceil_div(p.K, 16), outputs = (double)p.N * p.H * p.W * p.K / 1e6;
    double one = mode == WG_LOSSLESS ? (planes ? 9.3 + 2.75 * p.CB : 5.7 + 2.68 * p.CB)
                                     : (planes ? 8.0 + 1.75 * p.CB : 5.9 + 1.65 * p.CB);
    if (p.K <= kFusedFilters && !planes) one -= 0.6;
    if (pairs) one = (planes ? 2.5 + 3.9 * p.CB : pieces ? 2.1 + 2.6 * p.CB : 1.6 + 3.3 * p.CB) + w16 / 120.0 +
                     (planes || lossless_pair_filters_first(p) ? 0.0 : p.CB * std::min(p.Kp, 256) / 1500.0);
    const double split = mode != WG_LOSSLESS ? (planes ? 8.6 + 2.9 * b + W / 24.0 : (p.CB <= 3 ? 7.9 : 7.4) + 3.0 * b + W / 29.0)
                       : planes && !pairs    ? 5.1 + 3.7 * b + W / 68.0 + 7.1 * outputs
                       : planes              ? 4.0 + 4.4 * b + W / 53.0 + 6.4 * outputs
                       : pairs               ? 4.3 + 3.3 * b + W / 50.0
                                             : 4.8 + 3.27 * b + W / 50.0 + p.CB * p.Kp / 2700.0;
    return one > split + (pieces ? 0.0 : 3.9 * b - 2.2);
}

// Channel-major activations in lossless mode, not split: the limb-pair kernel with patches turned on their way into LDS, while
// its grid is one round of the compute units, against a copy and the forms of run_roles (fifty drawn layers, us: one
// channel block 7.9 - 8.9 against 10.1 - 12.4; two 12.3 - 13.5 / 12.8 - 15.4; three 16.9 - 18.7 / 15.4 - 23.5, seven 35 / 30 - 41; two
// rounds, one block 15.4 - 16.7 / 14.4 - 18.5).  Those are times of the halves; with quarters, where the grid allows them, three blocks that are
// not split would take 0.66 - 1.05 of what runs them (twelve layers, 0.89 on average), four and five 0.97 - 1.16 (eight).
bool pair_reads_planes(const Problem& p) {
    return p.CB <= 2 && (long long)ceil_div(p.T, kFusedTiles) * ceil_div(p.K, kFusedFilters) <= compute_units();
}

Plan plan_conv(const Problem& p, int layout, int mode, bool is_unsigned, size_t scratch_bytes) {
    Plan plan = {false, false, 1, p.CB};
    size_t left = scratch_bytes;
    // a test hook asks for one kernel (lossless mode: the split is the limb-pair form as well)
    const bool hooked = g_stream_workgroups.load(std::memory_order_relaxed) > 0 || g_stream_variant.load(std::memory_order_relaxed) != 0 ||
                        g_scaled_variant.load(std::memory_order_relaxed) != 0 || (mode == WG_LOSSLESS && lossless_variant() != 0);
    const int workgroups = ceil_div(p.T, kFusedTiles) * ceil_div(p.K, kFusedFilters);
    const bool may_split = p.CB >= 2 && 2 * workgroups <= compute_units() && !is_unsigned && !hooked;
    const int blocks = may_split ? ceil_div(p.CB, std::min(p.CB, compute_units() / workgroups)) : p.CB, splits = ceil_div(p.CB, blocks);
    auto split = [&](bool pieces, bool planes, bool pairs) {
        if (!may_split || !split_pays(mode, p, blocks, splits * workgroups, pieces, planes, pairs) || split_partial_bytes(p, mode, splits) > left) return false;
        plan.splits = splits;
        plan.blocks = blocks;
        return true;
    };
    if (layout == WG_NCHW && !is_unsigned && plane_patches_hold(p)) {
        // The split kernels read channel-major patches as well, at 1.1 us more per further block, while a copy is a launch: with up to two blocks
        // per workgroup what would be split after a copy is split without (us, split after a copy / without: 224 -> 32 at 82x98, N = 3, lossless,
        // 25.2 / 20.1; 208 -> 48 at 16x16, N = 59, 23.7 / 20.3; 196 -> 92 at 63x63, N = 2, 19.9 / 19.2).
        const bool pairs = mode == WG_LOSSLESS && pair_reads_planes(p);
        plan.planes = (blocks <= 2 && (split(true, true, pairs) || (!pairs && split(true, false, false)))) ||
                      (mode == WG_LOSSLESS && (lossless_variant() == 1 || (!hooked && pairs)));
        if (plan.planes) return plan;
    }
    if (layout != WG_NHWC || p.C % 4 != 0) {
        // (the copy is addressed with 32-bit offsets)
        plan.copies = left >= channels_last_bytes(p) && (long long)p.N * p.H * p.W * padded_channels(p.C) <= 0x7fffffffll;
        if (!plan.copies) return plan;
        left -= channels_last_bytes(p);
    }
    const bool pieces = plan.copies ? padded_channels(p.C) % 16 == 0 : p.C % 16 == 0;
    split(pieces, false, mode == WG_LOSSLESS && layout == WG_NHWC && lossless_pair_takes(p, pieces));   // (a caller's view may still start off a boundary)
    return plan;
}

}  // namespace

void set_scaled_variant(int v) { g_scaled_variant.store(v, std::memory_order_relaxed); }
void set_stream_variant(int v) { g_stream_variant.store(v, std::memory_order_relaxed); }
void set_stream_workgroups(int n) { g_stream_workgroups.store(n > 0 ? n : 0, std::memory_order_relaxed); }

int stream_workgroups(int tile_blocks, int filter_blocks) {
    const int forced = g_stream_workgroups.load(std::memory_order_relaxed);
    if (forced > 0) return std::max(1, std::min(tile_blocks, forced));
    // as many as the compute units allow, then as few as still finish in the same number of rounds
    const int wanted = std::max(1, compute_units() / filter_blocks);
    const int rounds = ceil_div(tile_blocks, wanted);
    return std::max(1, ceil_div(tile_blocks, rounds));
}

size_t fused_conv_scratch_wanted(const Problem& p, int layout, int mode, bool is_unsigned) {
    if (!is_unsigned && layout == WG_NHWC && p.C <= kNarrowChannels) return 0;
    const Plan plan = plan_conv(p, layout, mode, is_unsigned, ~(size_t)0 >> 1);
    return (plan.copies ? channels_last_bytes(p) : 0) + (plan.splits > 1 ? split_partial_bytes(p, mode, plan.splits) : 0);
}

namespace {

// The streaming kernel's 64-filter form without halves of the entries: in lossless mode and with one channel block four product waves with
// 16 filters each or eight with 8 (kStreamPairs).  The latter's chain per tile block is half as long, but they read the activation
// planes twice as often; they are ahead where a workgroup has few tile blocks and the store takes long.  us, four waves / eight, 64 -> 64
// at 56x56, one tile block per workgroup (N = 16): int8 out 10.4 / 9.4, pooled 9.9 / 8.9, channel-major int32 18.3 / 15.9, int32 11.1 / 10.8,
// uint8 11.2 / 11.0; two (N = 32) 16.6 / 16.0, 15.6 / 15.0, 27.5 / 26.6, 18.1 / 18.6, 17.6 / 17.8; three (N = 48) 22.6 / 21.8, 20.9 / 20.4, 35.7 / 35.5,
// 23.5 / 24.3, 23.7 / 24.7; four (N = 64, int8 out) 26.0 / 26.6.
StreamForm whole_form(const RolesCall& c, int mode) {
    const int variant = g_stream_variant.load(std::memory_order_relaxed);
    if (mode != WG_LOSSLESS || c.p.CB != 1 || variant == 1) return kStreamWhole;
    const int tile_blocks = ceil_div(c.p.T, kFusedTiles), each = ceil_div(tile_blocks, stream_workgroups(tile_blocks, ceil_div(c.p.K, 2 * kFusedFilters)));
    const bool planes32 = c.layout == WG_NCHW && c.q8.out == nullptr;
    return variant == 4 || each <= (c.q8.out != nullptr ? 3 : planes32 ? 2 : 1) ? kStreamPairs : kStreamWhole;
}

// Runs c through one of the role-specialised forms, which read channels-last activations with C % 4 = 0.  False: another
// kernel is the better one (it is left to the caller).
bool run_roles(const RolesCall& c, int mode, const Plan& plan, int32_t* partial, hipStream_t s, hipError_t& status) {
    const Problem& p = c.p;
    if (plan.splits > 1) {
        const int layout = plan.planes ? WG_NCHW : WG_NHWC;   // of the activations, as given or as a copy
        status = mode == WG_LOSSLESS ? launch_lossless_pair_sums(c.x, c.blob, partial, p, layout, plan.blocks, plan.splits, s)
                                     : launch_scaled_sums(c.x, c.blob, partial, p, layout, plan.blocks, plan.splits, s);
        if (status == hipSuccess)
            status = mode == WG_LOSSLESS ? launch_sums_finish(c, partial, plan.splits, s) : launch_split_finish(c, partial, plan.splits, s);
        return true;
    }
    // The streaming form when every workgroup gets at least six tile blocks to stream over (measured: +10-17 % on the
    // large layers; with fewer, the fill and drain of its pipeline cost more than the overlap saves), or when a test asks
    // for it.
    const int tile_blocks = ceil_div(p.T, kFusedTiles), filter_blocks = ceil_div(p.K, kFusedFilters);
    // The 64-filter form of that kernel (see below for when it applies) is also the fastest form for a layer with one
    // channel block as soon as the 32-filter grid exceeds one round of the compute units, whatever the number of tile
    // blocks per workgroup (56x56x64 at N = 12 .. 48: 8-30 % ahead of the limb-pair and 64-filter four-wave kernels).
    const int stream_variant = g_stream_variant.load(std::memory_order_relaxed);
    const bool whole64 = (p.K & 63) == 0 || (p.K & 63) > 32;   // padding to 64 filters adds no 32-filter block of nothing
    const int variant = g_scaled_variant.load(std::memory_order_relaxed);
    const long long cus = compute_units(), w32 = (long long)tile_blocks * filter_blocks;
    const long long wide_grid = (long long)tile_blocks * ceil_div(p.K, 2 * kFusedFilters);
    const bool wide_one_block = p.CB == 1 && whole64 && stream_variant == 0 && (long long)tile_blocks * filter_blocks > compute_units();
    // One channel block, a 32-filter grid of at most one round: the streaming kernel's 32-filter form with one tile block
    // per workgroup (its eight waves: four transform, four multiply) is 10-14 % ahead of the four-wave kernel in scaled
    // mode (56x56x64 at N = 8: 9.3 -> 8.5 us).  Lossless mode has the limb-pair kernel for signed channels-last layers of
    // this kind; the others come here, too.
    const bool forced_stream = g_stream_workgroups.load(std::memory_order_relaxed) > 0;
    const bool pair_layer = mode == WG_LOSSLESS && c.zero == nullptr && c.layout == WG_NHWC;
    // K mod 64 = 1 .. 32 and more than one round of 32-filter workgroups: 64-filter workgroups multiply a 32-filter block of
    // nothing in every tile block, 32-filter ones transform twice as often.  Which costs more is a matter of rounds: the streaming
    // forms take, for one channel block, us (K = 32 .. 288, 14 - 2500 workgroups, off by 5 % at most)
    //   32 filters, r rounds: 5.0 + 3.65 r scaled, 4.4 + 4.25 r lossless; 64 filters: 4.8 + 5.5 r, 4.3 + 6.15 r;
    //   the limb-pair kernel 1.0 + 5.9 r; the form with eight product waves, scaled, a single round: 9
    // and with several blocks 32-filter rounds take 1 / 1.34 of those with eight product waves (C = 128, scaled: 32 filters 15.6
    // and 22.0 for two and three rounds, 64 filters 11.4, 20.4, 30.4 for one to three; lossless 18.0, 25.3 / 13.8, 23.5, 33.8).
    // (64 -> 32 filters, 28x28, N = 162, scaled: 34 -> 15.6 us, lossless N = 490 60 -> 30; 128 -> 32, N = 162, 30.2 -> 22.0.)
    // Not where int8 outputs are stored byte by byte (not pooled, K no multiple of four): the four waves that store take up to 8 us a
    // round of 32 filters and 13 one of 64, the limb-pair kernel's eight no longer than otherwise (62 -> 334 at 86x86, N = 2, 25.1 us against
    // 35.8, 21 -> 138 at 43x43, N = 16, 24.3 / 32.4; 40 drawn layers 0.68 - 1.03 of what they took).
    if (!whole64 && w32 > cus && stream_variant == 0 && variant == 0 && !forced_stream && lossless_variant() != 1) {
        const int r32 = ceil_div(tile_blocks, std::max(1, (int)cus / filter_blocks)), r64 = (int)((wide_grid + cus - 1) / cus);
        if (p.CB > 1) {
            if (100 * r32 < 134 * r64) {
                status = launch_stream(c, mode, kStreamHalves, s);
                return true;
            }
        } else {
            const bool scaled = mode == WG_SCALED;
            const double halves = scaled ? 5.0 + 3.65 * r32 : 4.4 + 4.25 * r32, whole = scaled ? 4.8 + 5.5 * r64 : 4.3 + 6.15 * r64;
            const bool pairs = pair_layer && lossless_pair_conv_choice(c.x, p, c.layout) != 0;
            const bool by_bytes = c.q8.out != nullptr && !c.q8.pool && (p.K & 3) != 0;
            const double pair_cost = by_bytes ? 0.0 : 1.0 + 5.9 * (double)((w32 + cus - 1) / cus);
            const double other = scaled ? (r64 == 1 ? 9.0 : 1e9) : pairs ? pair_cost : 1e9;
            if (other < halves && other < whole) status = scaled ? launch_roles(c, mode, true, s) : launch_lossless_pair_conv(c.x, c.blob, c.y, p, c.layout, c.q8, s);
            else                                 status = launch_stream(c, mode, halves < whole ? kStreamHalves : whole_form(c, mode), s);
            return true;
        }
    }
    const bool narrow_one_round = !pair_layer && p.CB == 1 && stream_variant == 0 && !forced_stream &&
                                  (long long)tile_blocks * filter_blocks <= compute_units();
    const bool streams = forced_stream || wide_one_block || narrow_one_round ||
                         tile_blocks >= 6 * stream_workgroups(tile_blocks, filter_blocks);
    // Lossless mode, channels-last, one channel block, at most one round of 32-filter workgroups (layers with more are streamed): the
    // limb-pair form (eight waves per 16 tiles x 32 filters, lossless_conv.hip), 6.9 us a round on 56x56x64 layers, against
    // 7.4 for the four-wave form of this file.  Several channel blocks: see lossless_pair_takes.
    if (pair_layer && !streams) {
        const int form = lossless_pair_conv_choice(c.x, p, c.layout);   // 0: not applicable or switched off, 1: the library decides, 2: forced
        const bool others_asked_for = variant != 0 || stream_variant != 0;
        if (form == 2 || (form == 1 && (p.CB == 1 ? w32 <= cus : !others_asked_for && lossless_pair_takes(p, p.C % 16 == 0 && reinterpret_cast<uintptr_t>(c.x) % 16 == 0)))) {
            status = launch_lossless_pair_conv(c.x, c.blob, c.y, p, c.layout, c.q8, s);
            return true;
        }
    }
    // Several channel blocks: the role-specialised kernel with eight product waves and 64 filters per workgroup, as soon as
    // the 32-filter grid would need more than one round of the compute units (with a 64-filter grid of at most half the
    // compute units the 32-filter form, which then fills the chip in one round, stays ahead).
    // Measured on the layers of the VGG-16-shaped stack at N = 16 and on the 128-, 256- and 512-channel configurations.
    // Scaled mode: 15-30 % faster than the streaming, 64-filter four-wave and 32-filter role-specialised forms wherever
    // there are two or more channel blocks.  Lossless mode (twice the matrix-core work and filter bytes per product):
    // +10-25 % with two or more channel blocks where the layer is too small to stream; where it streams, the streaming
    // kernel's 64-filter form is level (two blocks) or 4 % ahead (four blocks) and takes the layer.
    // scaled mode also with one channel block, where the 64-filter grid is a single round and the 32-filter grid is not
    // (56x56x64 at N = 16: 11.4 -> 10.9 us against the streaming kernel's 64-filter form)
    const bool deep_enough = (p.CB >= 2 && (mode == WG_SCALED || !streams)) || (mode == WG_SCALED && wide_grid <= compute_units());
    // Several channel blocks and several tile blocks for every workgroup (scaled mode: three): the streaming kernel with eight
    // product waves.  Scaled: 112x112x128 N = 16 69.4 -> 65.2 us, 56x56x256 61.7 -> 59.4; with two tile blocks per workgroup it
    // is 2-5 % behind the form below (28x28x128 N = 64 23.0 -> 24.2).  Lossless: 56x56x256 N = 16 84.2 -> 75.9, 112x112x128
    // 78.7 -> 74.5, 28x28x128 N = 64 27.1 -> 26.2.  Not with channel-major int32 outputs, which are written in 64-byte rows of 32
    // planes and spill registers here (stream_kernel.h).  Scaled, the form below against this one: 56x56x256 N = 16 81.2 us
    // against 87.7, 112x112x128 N = 16 98.9 / 105.4 (uint8 99.5 / 114.4), 56x56x128 N = 32 60.0 / 67.4 (uint8 60.5 / 73.0); lossless,
    // whole entries: 96.9 / 102.3, 97.8 / 113.7 (99.2 / 114.4), 62.0 / 69.4 (62.8 / 69.7), and 28x28x128 N = 64 (the form below)
    // 38.7 / 41.1.  Channel-major int8 outputs are level or ahead here (scaled 72.6 against 76.6, 87.3 / 89.6, 56.3 / 56.1).
    const bool planes32 = c.layout == WG_NCHW && c.q8.out == nullptr;
    const bool long_streams = p.CB >= 2 && !planes32 && wide_grid > (mode == WG_SCALED ? 2LL : 1LL) * compute_units();
    if (stream_variant == 3 || (stream_variant == 0 && variant == 0 && !forced_stream && long_streams)) {
        status = launch_stream(c, mode, kStreamEight, s);
        return true;
    }
    if (variant == 1 || (variant == 0 && deep_enough && w32 > cus)) {
        status = launch_roles(c, mode, true, s);
        return true;
    }
    if (streams) {
        // the 64-filter form: lossless mode, or one channel block (see the kernel), unless the padding to 64 filters
        // would add a 32-filter block of nothing
        const bool wide = !narrow_one_round && (mode == WG_LOSSLESS || p.CB == 1) &&
                          (stream_variant == 1 || stream_variant == 4 || (stream_variant == 0 && whole64));
        status = launch_stream(c, mode, wide ? whole_form(c, mode) : kStreamHalves, s);
        return true;
    }
    // Transform and products on separate waves: with several channel blocks and no more 32-filter workgroups than compute
    // units (where the 64-filter variant would leave units idle), and in scaled mode from four channel blocks on
    // when the grid is at least three rounds of the compute units (there the product waves do no
    // vector work per block; measured on 256- and 512-channel layers: 10 % faster than the
    // 64-filter variant, while in lossless mode, with two channel blocks, or with a grid of one
    // or two rounds the 64-filter variant stays ahead).  Outputs and encodings that the four-wave kernel reaches only
    // through its slow loads take it with any grid.
    const long long workgroups = (long long)tile_blocks * filter_blocks;
    const bool others = c.zero != nullptr || c.layout != WG_NHWC;
    if ((p.CB >= 2 && (workgroups <= compute_units() || (mode == WG_SCALED && p.CB >= 4 && workgroups >= 3 * compute_units()))) || others) {
        status = launch_roles(c, mode, false, s);
        return true;
    }
    return false;
}

// The call with its activations channels-last, C % 4 = 0: as given, or copied into scratch memory, where the channel
// sums of a split follow.  False where the layout would need a copy and there is no memory for it.
bool make_fast_call(RolesCall& c, const Plan& plan, int layout, const Scratch& scratch, int32_t*& partial, hipStream_t s, hipError_t& status) {
    partial = static_cast<int32_t*>(scratch.p);
    status = hipSuccess;
    if (plan.planes || (layout == WG_NHWC && c.p.C % 4 == 0)) return true;
    if (!plan.copies) return false;
    int8_t* const copy = static_cast<int8_t*>(scratch.p);
    const int padded = padded_channels(c.p.C);
    status = launch_channels_last(c.x, copy, c.p, layout, padded, c.zero ? (uint8_t)c.zero->zero_bytes : 0, s);
    partial = reinterpret_cast<int32_t*>(copy + channels_last_bytes(c.p));
    c.x = copy;
    c.p.C = padded;
    return true;
}

}  // namespace

// uint8 activations with a zero point: the role-specialised forms; without the scratch memory for a channels-last copy
// the four-wave kernel's byte loads.
hipError_t launch_fused_conv_u8(const uint8_t* x_u8, int zero_point, const void* blob, int32_t* y, const Problem& p, int layout,
                                int mode, const Scratch& scratch, hipStream_t s) {
    const BlobLayout bl = blob_layout(p.Kp, p.Cf, mode);
    const uint8_t* b = static_cast<const uint8_t*>(blob);
    const int8_t* x = reinterpret_cast<const int8_t*>(x_u8);
    const ZeroPointU8 zero = make_zero_point(zero_point);
    const Plan plan = plan_conv(p, layout, mode, true, scratch.bytes);
    RolesCall c = {x, &zero, b, bl, y, p, layout, no_int8_epilogue()};
    int32_t* partial;
    hipError_t status;
    if (make_fast_call(c, plan, layout, scratch, partial, s, status)) {
        if (status == hipSuccess) run_roles(c, mode, plan, partial, s, status);
        return status;
    }
    if (layout == WG_NHWC) return launch_u8_mode<WG_NHWC, kLoadBytes>(x, zero, b, bl, y, p, mode, s);
    return launch_u8_mode<WG_NCHW, kLoadBytes>(x, zero, b, bl, y, p, mode, s);
}

// With scratch memory: factors first, then a role-specialised kernel (act_scaled_conv.hip), through a channels-last copy where
// the layout asks for one.  Without: both passes in the four-wave kernel.  So, too, where that reads the activations as they
// are, its 32-filter grid is a single round of the compute units and it has at most two channel blocks: what the two
// kernels save there is less than a launch (a grid of one round, one block 11.5 - 13 us in one kernel, 15 - 16.5 in two, two
// blocks 16.4 / 17.8, three 21 / 20; one block and 1.2 - 1.5 rounds 23 / 19).
static bool one_act_scaled_kernel(const Problem& p, int layout) {
    return layout == WG_NHWC && p.C % 4 == 0 && p.CB <= 2 && (long long)ceil_div(p.T, kFusedTiles) * ceil_div(p.K, kFusedFilters) <= compute_units();
}

static Plan plan_act_scaled(const Problem& p, int layout, size_t scratch_bytes) {
    Plan plan = {false, false, 1, p.CB};
    if (layout != WG_NHWC || p.C % 4 != 0)
        plan.copies = scratch_bytes >= channels_last_bytes(p) && (long long)p.N * p.H * p.W * padded_channels(p.C) <= 0x7fffffffll;
    return plan;
}

size_t act_scaled_scratch_wanted(const Problem& p, int layout) {
    if (one_act_scaled_kernel(p, layout)) return 0;
    return (plan_act_scaled(p, layout, ~(size_t)0 >> 1).copies ? channels_last_bytes(p) : 0) + act_factor_bytes(p);
}

hipError_t launch_fused_conv_act_scaled(const int8_t* x, const void* blob, int32_t* y, int32_t* act_table, const Problem& p,
                                        int layout, const Scratch& scratch, hipStream_t s) {
    const BlobLayout bl = blob_layout(p.Kp, p.Cf, WG_SCALED);
    const uint8_t* b = static_cast<const uint8_t*>(blob);
    if (!one_act_scaled_kernel(p, layout) && scratch.bytes >= act_scaled_scratch_wanted(p, layout)) {
        RolesCall c = {x, nullptr, b, bl, y, p, layout, no_int8_epilogue()};
        int32_t* rest;
        hipError_t status;
        if (make_fast_call(c, plan_act_scaled(p, layout, scratch.bytes), layout, scratch, rest, s, status)) {
            if (status == hipSuccess) status = launch_act_factors(c, reinterpret_cast<uint32_t*>(rest), act_table, s);
            if (status == hipSuccess) status = launch_act_scaled_roles(c, reinterpret_cast<const uint32_t*>(rest), s);
            return status;
        }
    }
    if (layout == WG_NHWC && p.C % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 4 == 0)
        return launch_act_scaled<WG_NHWC, kLoadDwords>(x, b, bl, y, act_table, p, s);
    if (layout == WG_NHWC) return launch_act_scaled<WG_NHWC, kLoadBytes>(x, b, bl, y, act_table, p, s);
    return launch_act_scaled<WG_NCHW, kLoadBytes>(x, b, bl, y, act_table, p, s);
}

hipError_t launch_fused_conv(const int8_t* x, const void* blob, int32_t* y, const Problem& p, int layout, int mode,
                             const Int8Epilogue& q8, const Scratch& scratch, hipStream_t s) {
    if (layout == WG_NHWC && p.C <= kNarrowChannels) return launch_narrow_conv(x, blob, y, p, mode, q8, s);
    const BlobLayout bl = blob_layout(p.Kp, p.Cf, mode);
    const uint8_t* b = static_cast<const uint8_t*>(blob);
    const Plan plan = plan_conv(p, layout, mode, false, scratch.bytes);
    if (plan.planes && plan.splits == 1) return launch_lossless_pair_conv(x, b, y, p, layout, q8, s);
    RolesCall c = {x, nullptr, b, bl, y, p, layout, q8};
    int32_t* partial;
    hipError_t status;
    if (make_fast_call(c, plan, layout, scratch, partial, s, status) && (status != hipSuccess || run_roles(c, mode, plan, partial, s, status)))
        return status;
    return q8.out != nullptr ? launch_layout<true>(c.x, b, bl, y, c.p, layout, mode, q8, s)
                             : launch_layout<false>(c.x, b, bl, y, c.p, layout, mode, q8, s);
}

}  // namespace wg
