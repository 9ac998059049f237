// fused_conv_roles_kernel: the single-kernel convolution with transform and products on different waves, one tile block
// per workgroup.  See fused_conv.hip for the method and the dispatch.
#pragma once
#include "product_core.h"
#include "roles_conv.h"
#include "write_through.h"

namespace wg {
namespace {

// The same computation for layers with several channel blocks, with the two kinds of work on
// different waves.  Eight waves: waves 0-3 only transform (vector ALU), waves 4-7 only multiply
// (matrix cores, joins, output transform); each SIMD hosts one of each, so the transform of
// channel block cb + 1 runs under the products of block cb instead of before them, and a
// product wave's waits are filled with the transform wave's work.  The operand planes are
// double-buffered in LDS (2 x 72 KB); patches come through 4-byte or byte loads into the
// transform threads' registers, one channel block ahead.  One barrier per channel block:
// barrier j (j = 1..CB) publishes the planes of block j - 1 and frees the buffer that the
// products of block j - 2 were reading.  32 filters per workgroup (a second pass would not fit
// the 256 registers a wave has when two share a SIMD).
// PW = 8: eight product waves, twelve waves in all, 64 filters per workgroup: with two product waves per SIMD one
// transform (and one set of patch loads) serves twice the filters.  Product wave pw owns filter block pw % 4 and half
// pw / 4 of the entries.  Three waves per SIMD leave a wave 168 registers, so in scaled mode the product waves keep the low
// limbs' chains (ChainedSums) instead of the 32 to 40 resident limb accumulators.  The two 32-filter halves stage their
// outputs in one operand buffer each and store at the same time.
// What bounds a further channel block of that form in scaled mode (14x14, K = 256, N = 64, one round: 2.66 us, 5,600 clocks; 4,900
// in the streaming kernel's form with eight product waves): a SIMD's vector ALU, 431 instructions of the transform wave and
// 2 x 110 of the product waves at 4.4 clocks + 8 for each of 112 matrix-core instructions = 3,800 (counted: 645 + 112); filter
// fragments and patches through the memory path, 2,500 + up to 2,300; LDS, 288 fragment reads and 288 writes, some 4,000; and the
// transform wave's own chain, an instruction per 5 clocks, 2,650.  (Four product waves and 32 filters: 1.76 us, 3,700 clocks.)

template <int LAYOUT, int MODE, int OUT, int PW, class ENC>
__global__ __launch_bounds__(64 * (4 + PW)) void fused_conv_roles_kernel(const int8_t* __restrict__ x, WG_GEOMETRY_PARAMS,
                                                                         WG_ORDER_PARAMS, const uint8_t* __restrict__ blob,
                                                                         size_t table_off, size_t planes_off, int32_t* __restrict__ y,
                                                                         Problem p, Int8Epilogue q8, ENC enc) {
    WG_TAKE_GEOMETRY(p, 2);
    const GridOrder order = WG_TAKE_ORDER;
    static_assert(PW == 4 || PW == 8, "one or two product waves per SIMD");
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    const int lane = threadIdx.x & 63, wave8 = threadIdx.x >> 6;
    const bool transforms = wave8 < 4;
    const int tid = threadIdx.x & 255, wave = wave8 & 3;   // within the role (PW = 8: within the four waves that store together)
    int bx, by;
    order.place(bx, by);
    const int tile0 = bx * kFusedTiles, k0 = by * (kFusedFilters * (PW / 4));
    // requested first, compared by either role before it goes on from what does not depend on the blob (uniform: nobody reaches a
    // barrier otherwise): compared up here, field by field, it stood before the first patch (28x28x128 N = 32 13.60 -> 13.21 us,
    // 16 channels at 16x16 10.28 -> 9.92)
    const BlobHeaderWords header = read_blob_header(blob);
    auto matches = [&] { return blob_matches(header, p.K, p.Cf, MODE, ENC::kMagic); };
    // (uint8 with eight product waves: here all the same, twelve layers of one channel block 1.4 % faster, deeper ones level; with four,
    // 144 -> 29 at 94x7, N = 3, 11.0 us, here 11.3)
    if (PW == 8 && !std::is_same_v<ENC, SignedInt8> && !matches()) return;
    int my_n = 0, my_ty = 0, my_tx = 0;
    if (tile0 + (lane & 15) < p.T) decode_tile(p, tile0 + (lane & 15), my_n, my_ty, my_tx);
#ifdef WG_TIMESTAMPS
    unsigned long long spent[4] = {0, 0, 0, 0}, mark = WG_CLOCK();
    const unsigned long long entered = mark;
    auto report = [&]() {
        if (g_roles_stamps != nullptr && lane == 0) {
            unsigned long long* o = g_roles_stamps + ((size_t)(blockIdx.y * gridDim.x + blockIdx.x) * 12 + wave8) * 8;
            o[0] = spent[0]; o[1] = spent[1]; o[2] = spent[2]; o[3] = spent[3]; o[4] = WG_CLOCK() - entered; o[6] = entered;
        }
    };
#endif

    if (transforms) {
        const int a_tile = PatchLoader::tile_of(wave, lane), a_cq = PatchLoader::quad_of(lane);
        const int a_tx = __shfl(my_tx, a_tile), a_ty = __shfl(my_ty, a_tile), a_n = __shfl(my_n, a_tile);
        OperandSplitter<MODE == WG_SCALED ? kSplitByteLimbs : kSplitTwoLimb, LdsPlaneSink> out;
        int8_t* const slot = lds + lds_slot(a_cq >> 2, a_tile) * 16 + (a_cq & 3) * 4;
        const __amdgpu_buffer_rsrc_t xbuf = activation_buffer(x, p);
        PatchBias<ENC> bias;
        bias.enter(p, a_ty, a_tx, enc);
        PatchLoader loader;
        loader.enter(p, a_n, a_ty, a_tx, lane);
        loader.drop_absent_channels(p, 0, lane);
        loader.request(xbuf, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (!matches()) return;
        WG_SPENT(3, mark);
        for (int cb = 0; cb < p.CB; ++cb) {
            if (cb > 0) {   // barrier cb
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
            }
            WG_SPENT(0, mark);   // LDS writes landed + barrier
            out.sink.base = slot + (cb & 1) * kLdsBytes;
#ifdef WG_TIMESTAMPS
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            WG_SPENT(1, mark);   // wait for the patch
#endif
            bias.apply(loader.patch);
            if (cb + 1 < p.CB) {
                loader.drop_absent_channels(p, cb + 1, lane);
                transform_patch<typename PatchBias<ENC>::Bytes>(loader.patch, out, enc, NextColumns{loader, xbuf, cb + 1});
            } else {
                transform_patch<typename PatchBias<ENC>::Bytes>(loader.patch, out, enc);
            }
            WG_SPENT(2, mark);   // transform and requests
        }
#ifdef WG_TIMESTAMPS
        report();
#endif
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();   // barrier CB: the last block's planes are published
        __syncthreads();                // the two barriers of the product waves' store
        __syncthreads();
        return;
    }

    // PW = 4: wave = 2 half + kblock.  PW = 8: product wave pw = wave8 - 4 owns filter block pw % 4 and half pw / 4; the
    // waves of filter blocks 2 group, 2 group + 1 store together (`wave` counts within that group, as store_staged expects)
    if (!matches()) return;
    const int pw = wave8 - 4;
    const int kblock4 = PW == 8 ? (pw & 3) : (wave & 1), half = PW == 8 ? (pw >> 2) : (wave >> 1);
    const int kblock = kblock4 & 1, group = kblock4 >> 1;
    const int k = k0 + kblock4 * 16 + (lane & 15);
    LaneContext cx;
    cx.table_k = reinterpret_cast<const ScaleEntry*>(blob + table_off) + (size_t)k * kEntries;
    cx.parked = nullptr;
    int8_t* const scale_area = lds + 2 * kLdsBytes + pw * kParkedScaleBytes;   // behind the two plane buffers: 1 KB per product wave
    constexpr int NP = MODE == WG_LOSSLESS ? 138 : 46;
    const int8_t* const b_wave = filter_fragments(blob + planes_off, k - (lane & 15), p.Kp, NP);
    cx.b_lane = fragment_lane(lane);
    const size_t b_block_stride = (size_t)(p.Kp >> 4) * NP * kFilterFragBytes;
    v4i Y[16];
    // The product waves do no output transform per block.  Scaled: all 36 limb-product accumulators of a half stay
    // resident (PW = 4), or the low limbs' chains do (PW = 8: 168 registers per wave); lossless: joined channel sums.
    // One loop per half (the same barriers in both), so that each is allocated registers on its own.
    auto blocks = [&](auto H) {
        using Phase = std::conditional_t<MODE == WG_LOSSLESS, LosslessSums<H, PW == 8 ? 6 : 8>,
                                         std::conditional_t<PW == 4, ResidentScaled<H>, ChainedSums<H, H == 0 ? 6 : 7, 4, std::is_same_v<ENC, SignedInt8>>>>;
        Phase phase;
        v4i sums[Phase::kSums];
#pragma unroll
        for (int i = 0; i < Phase::kSums; ++i) sums[i] = (v4i){0, 0, 0, 0};
        cx.b_glob = b_wave;
        phase.enter(cx, scale_area, lane);
        for (int cb = 0; cb < p.CB; ++cb) {
            if (cb > 0) {
                cx.b_glob = b_wave + cb * b_block_stride;
                phase.prefetch(cx);
            }
            WG_SPENT(3, mark);   // ring prefetch issue
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();   // barrier cb + 1
            WG_SPENT(0, mark);   // barrier
            cx.a_lds = lds + (cb & 1) * kLdsBytes + lds_slot(lane >> 4, lane & 15) * 16;
            // (512 -> 512 at 7x7, N = 32, scaled, at a multiple of eight / four behind 18.8 / 19.2 us, int8 out, 14x14, N = 16, 19.0 / 18.7;
            // 192 -> 32 at 28x28, N = 16, uint8, 10.5 / 10.8, 128 -> 128, N = 32, 12.5 / 12.3; lossless 14.4 / 14.2)
            place_loop(std::integral_constant<bool, OUT == kOutInt8 || MODE == WG_LOSSLESS || (PW == 8 && !std::is_same_v<ENC, SignedInt8>)>{});
            phase.run(cx, sums);
            WG_SPENT(2, mark);   // products
        }
#ifdef WG_TIMESTAMPS
        report();
#endif
        Phase::finish(cx, sums, Y);
    };
    if (half == 0) blocks(std::integral_constant<int, 0>{}); else blocks(std::integral_constant<int, 1>{});
    // PW = 8: the two 32-filter halves of the workgroup stage in one operand buffer each and store side by side
    StoreContext sc;
    sc.lds = lds + group * kLdsBytes;
    sc.tid = PW == 8 ? (2 * half + kblock) * 64 + lane : tid;
    sc.lane = lane; sc.rnd = MODE == WG_SCALED ? 8 : 0; sc.y = y;
    locate_tile<LAYOUT>(sc, p, tile0);
    __syncthreads();   // the operand planes are dead
    stage_outputs(sc.lds, lane, half, kblock, Y);
    __syncthreads();
    store_staged<LAYOUT, OUT, true>(sc, p, q8, k0 + group * kFusedFilters);
#ifdef WG_TIMESTAMPS
    if (g_roles_stamps != nullptr && lane == 0)
        g_roles_stamps[((size_t)(blockIdx.y * gridDim.x + blockIdx.x) * 12 + wave8) * 8 + 5] = WG_CLOCK() - entered;
#endif
}

template <int LAYOUT, int MODE, int OUT, int PW, class ENC>
hipError_t launch_roles(const int8_t* x, const ENC& enc, const uint8_t* blob, const BlobLayout& bl, int32_t* y, const Problem& p,
                        const Int8Epilogue& q8, hipStream_t s) {
    constexpr int lds_bytes = 2 * kLdsBytes + PW * kParkedScaleBytes;   // two plane buffers, the parked reverse-scaling factors
    static_assert(lds_bytes <= 160 * 1024, "fits the LDS of a compute unit");
    static LdsLimitOnce lds_limit;   // per template instance
    if (hipError_t e = lds_limit.set(reinterpret_cast<const void*>(&fused_conv_roles_kernel<LAYOUT, MODE, OUT, PW, ENC>), lds_bytes)) return e;
    dim3 grid(ceil_div(p.T, kFusedTiles), ceil_div(p.K, kFusedFilters * (PW / 4)));
    const GridOrder order(grid, workgroup_order(p, MODE, kFusedFilters * (PW / 4)));
    fused_conv_roles_kernel<LAYOUT, MODE, OUT, PW, ENC><<<grid, 64 * (4 + PW), lds_bytes, s>>>(
        x, WG_GEOMETRY(p), WG_ORDER(order), blob, bl.table_off, bl.planes_off, y, p, q8, enc);
    return hipGetLastError();
}

// One mode's launches (each mode is compiled in a file of its own).
template <int MODE>
hipError_t launch_roles_mode(const RolesCall& c, bool wide, hipStream_t s) {
    using std::integral_constant;
    const bool through = f4_through(c.p, c.y, c.layout);
    auto go = [&](auto L, auto Q8, auto PW, const auto& enc) {
        auto launch = [&](auto OUT) { return launch_roles<L, MODE, OUT, PW>(c.x, enc, c.blob, c.bl, c.y, c.p, c.q8, s); };
        if constexpr (Q8) return launch(integral_constant<int, kOutInt8>{});
        else return through ? launch(integral_constant<int, kOutThrough>{}) : launch(integral_constant<int, kOutInt32>{});
    };
    auto form = [&](auto L, auto Q8, const auto& enc) {
        return wide ? go(L, Q8, integral_constant<int, 8>{}, enc) : go(L, Q8, integral_constant<int, 4>{}, enc);
    };
    constexpr integral_constant<int, WG_NHWC> nhwc{};
    constexpr integral_constant<int, WG_NCHW> nchw{};
    if (c.zero != nullptr)   // uint8 tensors: int32 outputs only
        return c.layout == WG_NHWC ? form(nhwc, std::false_type{}, *c.zero) : form(nchw, std::false_type{}, *c.zero);
    if (c.q8.out != nullptr)
        return c.layout == WG_NHWC ? form(nhwc, std::true_type{}, SignedInt8{}) : form(nchw, std::true_type{}, SignedInt8{});
    return c.layout == WG_NHWC ? form(nhwc, std::false_type{}, SignedInt8{}) : form(nchw, std::false_type{}, SignedInt8{});
}

}  // namespace
}  // namespace wg
