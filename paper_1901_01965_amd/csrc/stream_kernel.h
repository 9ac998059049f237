// fused_conv_stream_kernel: the role-specialised convolution as a stream over tile blocks.  See fused_conv.hip for the
// method and the dispatch.
#pragma once
#include "product_core.h"
#include "roles_conv.h"

namespace wg {
namespace {

// Barrier among the four transform waves of the streaming kernel (s_barrier would stop the product
// waves as well): a counter in LDS that only grows, four arrivals per use.  A wave arrives once its
// own LDS reads have returned and leaves when all four have arrived, so no wave writes the shared
// buffer while another still reads it.  Every transform wave runs the same (workgroup-uniform)
// sequence of uses, and all four are resident together, so the wait ends.
struct TransformWavesBarrier {
    uint32_t* counter;
    uint32_t arrivals;   // what the counter reads once everyone has arrived at the current use
    __device__ inline void sync(int lane) {
        arrivals += 4;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (lane == 0) __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        while ((int)(__hip_atomic_load(counter, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) - arrivals) < 0)
            __builtin_amdgcn_s_sleep(1);
        asm volatile("" ::: "memory");
    }
};

// The role-specialised kernel as a stream over tile blocks: a workgroup owns one 32-filter block
// and walks over many tile blocks (grid: about one workgroup per compute unit), so that the two
// roles also overlap across tile blocks and layers with a single channel block are pipelined
// too.  A unit u is one (tile block, channel block); the transform waves are one unit ahead of
// the product waves, and they also take over the second half of the store: at the end of a
// tile block the product waves only stage their outputs in LDS (in the buffer whose planes
// they have just consumed), and the transform waves add the halves and write them out while
// the product waves already multiply the next unit.
// Barriers, in the same order on both roles: U_u (u = 1..U) publishes the planes of unit u - 1 and
// frees the buffer of unit u - 2; after the last channel block of a tile block, D_u (every product
// wave has finished reading the planes) and S_u (the outputs are staged).
// The staged outputs of unit u - 2 and the planes of unit u share a buffer, and the four transform
// waves both read the former (each thread reads rows that other waves' plane writes cover) and
// write the latter: between the two they meet at a barrier of their own (TransformWavesBarrier;
// the product waves, which are multiplying unit u - 1 in the other buffer, do not take part).
// Channels-last, C % 4 = 0 (4-byte pixel loads), K % 4 = 0 (16-byte stores).
// WIDE: 64 filters per workgroup.  Each product wave owns every entry of its 16 filters (and keeps no
// channel sums: see the product side), so one transform serves twice the filters, no halves are added, and
// the workgroup stages one finished copy of its outputs (32 filters in the place of each half), which the
// transform waves write out.
template <int LAYOUT, int MODE, bool Q8, bool WIDE, class ENC>
__global__ __launch_bounds__(512) void fused_conv_stream_kernel(const int8_t* __restrict__ x, const uint8_t* __restrict__ blob,
                                                                size_t table_off, size_t planes_off, int32_t* __restrict__ y,
                                                                Problem p, Int8Epilogue q8, int tile_blocks, ENC enc) {
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    const int lane = threadIdx.x & 63, wave8 = threadIdx.x >> 6;
    const bool transforms = wave8 < 4;
    const int tid = threadIdx.x & 255, wave = wave8 & 3;   // within the role
    const int k0 = blockIdx.y * kFusedFilters * (WIDE ? 2 : 1);
    if (!blob_matches(reinterpret_cast<const BlobHeader*>(blob), p.K, p.Cf, MODE, ENC::kMagic)) return;
    // this workgroup's tile blocks: blockIdx.x, blockIdx.x + gridDim.x, ...
    const int my_blocks = (tile_blocks - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
    const int units = my_blocks * p.CB;
    const int rnd = MODE == WG_SCALED ? 8 : 0;
#ifdef WG_TIMESTAMPS
    // ticks per part of the unit loop, summed per wave: 8 numbers per wave, 12 wave slots per workgroup
    unsigned long long spent[6] = {0, 0, 0, 0, 0, 0}, mark = WG_CLOCK();
    const unsigned long long entered = mark;
    auto report = [&]() {
        if (g_roles_stamps != nullptr && lane == 0) {
            unsigned long long* o = g_roles_stamps + ((size_t)(blockIdx.y * gridDim.x + blockIdx.x) * 12 + wave8) * 8;
            for (int i = 0; i < 6; ++i) o[i] = spent[i];
            o[6] = WG_CLOCK() - entered;
            o[7] = (unsigned long long)units;
        }
    };
#endif

    if (transforms) {
        const int a_tile = PatchLoader::tile_of(wave, lane), a_cq = PatchLoader::quad_of(lane);
        OperandSplitter<MODE == WG_SCALED ? kSplitByteLimbs : kSplitTwoLimb, LdsPlaneSink> out;
        int8_t* const slot = lds + lds_slot(a_cq >> 2, a_tile) * 16 + (a_cq & 3) * 4;
        PatchBias<ENC> bias, next_bias;   // of the patch being transformed, of the one in flight
        PatchLoader loader;
        auto enter_tile_block = [&](int tb) {
            const int t = tb * kFusedTiles + a_tile;
            int n = 0, ty = 0, tx = 0;
            if (t < p.T) decode_tile(p, t, n, ty, tx);
            loader.enter(p, n, ty, tx, lane);
            next_bias.enter(p, ty, tx, enc);
        };
        const __amdgpu_buffer_rsrc_t xbuf = activation_buffer(x, p);
        // adds the two halves staged in `buffer` for tile block tb and writes them out
        auto flush = [&](int tb, int buffer) {
            StoreContext sc;
            sc.lds = lds + buffer * kLdsBytes; sc.tid = tid; sc.lane = lane; sc.rnd = rnd; sc.y = y;
            locate_tile<LAYOUT>(sc, p, tb * kFusedTiles);
            if constexpr (WIDE) {   // one finished copy per 32 filters
                store_staged<LAYOUT, Q8, false>(sc, p, q8, k0);
                sc.lds += kStageHalf * 4;
                store_staged<LAYOUT, Q8, false>(sc, p, q8, k0 + kFusedFilters);
            } else {
                store_staged<LAYOUT, Q8, true>(sc, p, q8, k0);
            }
        };
        TransformWavesBarrier among_us = {reinterpret_cast<uint32_t*>(lds + 2 * kLdsBytes), 0u};
        if (tid == 0) *among_us.counter = 0u;   // lands before the first s_barrier, long before the first use
        int cb = 0, jb = 0;   // unit u = (tile block number jb of this workgroup, channel block cb)
        if (units > 0) {
            enter_tile_block(blockIdx.x);
            loader.drop_absent_channels(p, 0, lane);
            loader.request(xbuf, 0);
        }
        // was unit v the last channel block of its tile block?  v % CB == CB - 1, tracked without division:
        // last1 = for unit u - 1, last2 = for unit u - 2; tb1 / tb2 = their tile blocks
        bool last1 = false, last2 = false;
        int tb1 = 0, tb2 = 0;
        for (int u = 0; u <= units; ++u) {
            WG_SPENT(5, mark);   // requests
            if (u > 0) {   // U_u
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
            }
            WG_SPENT(0, mark);   // barrier U
            if (last2) {   // staged in the buffer of unit u - 2, which unit u is about to overwrite
                flush(tb2, u & 1);
                among_us.sync(lane);   // every transform wave has read its share before any of them writes planes
            }
            WG_SPENT(1, mark);   // flush
            const int tb = (int)blockIdx.x + jb * (int)gridDim.x;
            const bool last0 = u < units && cb == p.CB - 1;
            if (u < units) {
                out.sink.base = slot + (u & 1) * kLdsBytes;
#ifdef WG_TIMESTAMPS
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                WG_SPENT(2, mark);   // wait for the patch
#endif
                // the next unit's patch is asked for as the registers of this one become free
                const bool more = u + 1 < units;
                if (++cb == p.CB) { cb = 0; ++jb; }
                bias = next_bias;
                if (more) {
                    if (cb == 0) enter_tile_block((int)blockIdx.x + jb * (int)gridDim.x);
                    loader.drop_absent_channels(p, cb, lane);
                }
                bias.apply(loader.patch);
                WG_SPENT(5, mark);   // offsets
                if (more) transform_patch<typename PatchBias<ENC>::Bytes>(loader.patch, out, enc, NextColumns{loader, xbuf, cb});
                else      transform_patch<typename PatchBias<ENC>::Bytes>(loader.patch, out, enc);
            }
            WG_SPENT(3, mark);   // transform
            if (last1) {   // D_{u-1}, S_{u-1}
                __syncthreads();
                __syncthreads();
            }
            WG_SPENT(4, mark);   // barriers D and S
            last2 = last1; tb2 = tb1;
            last1 = last0; tb1 = tb;
        }
        if (last2) flush(tb2, (units + 1) & 1);   // the last tile block, staged in the buffer of unit U - 1
#ifdef WG_TIMESTAMPS
        report();
#endif
        return;
    }

    // WIDE: wave w owns filters 16 w .. 16 w + 15 of the 64 and every entry; in the staging it stands where wave
    // (half = w / 2, kblock = w % 2) of a 32-filter workgroup stands, so that copy w / 2 holds filters 32 (w / 2) ..
    const int kblock = wave & 1, half = wave >> 1;
    const int k = k0 + (WIDE ? wave : kblock) * 16 + (lane & 15);
    LaneContext cx;
    cx.table_k = reinterpret_cast<const ScaleEntry*>(blob + table_off) + (size_t)k * kEntries;
    cx.parked = nullptr;
    // behind the plane buffers and the barrier counter
    int8_t* const scale_area = lds + 2 * kLdsBytes + 64 + wave * (WIDE ? ParkedScales<kAllRows>::kBytes : kParkedScaleBytes);
    constexpr int NP = MODE == WG_LOSSLESS ? 138 : 46;
    const int8_t* const b_wave = filter_fragments(blob + planes_off, k - (lane & 15), p.Kp, NP);
    cx.b_lane = fragment_lane(lane);
    const size_t b_block_stride = (size_t)(p.Kp >> 4) * NP * kFilterFragBytes;
    if constexpr (WIDE) {
        // Every entry of 16 filters in one wave.  36 joined channel sums next to the fragments would not fit the registers,
        // so each channel block's products go through the reverse scaling and the output transform at once and the
        // outputs accumulate: exact in lossless mode (the transform is linear); in scaled mode the reverse scaling applies
        // to the channel sum (Section 4.2), so there the host uses this form for one-block layers only.
        // filter ring: lossless mode has twice the fragments per entry and the registers for twelve in flight
        LeanProducts<MODE, kAllRows, false, MODE == WG_SCALED ? 8 : 12, true, true> all;
        v4i unused[1];
        v4i Y[16];
        int cb = 0;
        if (units > 0) {
            cx.b_glob = b_wave;
            ParkedScales<kAllRows> scales;
            if constexpr (MODE == WG_SCALED) scales.ask(cx, lane);
            all.prefetch(cx);
            if constexpr (MODE == WG_SCALED) scales.park(cx, scale_area, lane);
        }
        for (int u = 0; u < units; ++u) {
            if (cb == 0) {
#pragma unroll
                for (int i = 0; i < 16; ++i) Y[i] = (v4i){0, 0, 0, 0};
            }
            WG_SPENT(5, mark);   // clearing the outputs
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();   // U_{u+1}
            WG_SPENT(0, mark);   // barrier U
            cx.a_lds = lds + (u & 1) * kLdsBytes + lds_slot(lane >> 4, lane & 15) * 16;
            all.run(cx, unused, Y);
            WG_SPENT(1, mark);   // products
            const bool last = cb == p.CB - 1;
            cb = last ? 0 : cb + 1;
            if (u + 1 < units) {   // the next unit's first filter fragments travel while this one is staged
                cx.b_glob = b_wave + cb * b_block_stride;
                all.prefetch(cx);
            }
            if (last) {
                WG_SPENT(2, mark);   // prefetch issue
                __syncthreads();   // D_u: every product wave has finished reading this unit's planes
                WG_SPENT(3, mark);   // barrier D
                stage_outputs(lds + (u & 1) * kLdsBytes, lane, half, kblock, Y);
                __syncthreads();   // S_u: staged
                WG_SPENT(4, mark);   // staging and barrier S
            }
        }
#ifdef WG_TIMESTAMPS
        report();
#endif
        return;
    }
    // Channel sums per wave (all 36 accumulators next to the outputs would not fit the 256 registers here).  Scaled mode: a
    // loop per half, whose sums differ in number; lossless mode: one loop for both halves (a loop each would spill).
    auto stream = [&](auto& phase) {
        v4i sums[std::remove_reference_t<decltype(phase)>::kSums];
        int cb = 0;
        if (units > 0) {
            cx.b_glob = b_wave;
            phase.enter(cx, scale_area, lane);
        }
        for (int u = 0; u < units; ++u) {
            if (cb == 0) {
#pragma unroll
                for (int i = 0; i < (int)(sizeof(sums) / sizeof(v4i)); ++i) sums[i] = (v4i){0, 0, 0, 0};
            }
            WG_SPENT(5, mark);   // clearing the sums
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();   // U_{u+1}
            WG_SPENT(0, mark);   // barrier U
            cx.a_lds = lds + (u & 1) * kLdsBytes + lds_slot(lane >> 4, lane & 15) * 16;
            phase.run(cx, sums);
            WG_SPENT(1, mark);   // products
            const bool last = cb == p.CB - 1;
            cb = last ? 0 : cb + 1;
            if (u + 1 < units) {   // the next unit's first filter fragments travel while this one is finished and staged
                cx.b_glob = b_wave + cb * b_block_stride;
                phase.prefetch(cx);
            }
            if (last) {
                v4i Y[16];
                phase.finish(cx, sums, Y);
                WG_SPENT(2, mark);   // finish
                __syncthreads();   // D_u: every product wave has finished reading this unit's planes
                WG_SPENT(3, mark);   // barrier D
                stage_outputs(lds + (u & 1) * kLdsBytes, lane, half, kblock, Y);
                __syncthreads();   // S_u: staged
                WG_SPENT(4, mark);   // staging and barrier S
            }
        }
    };
    if constexpr (MODE == WG_SCALED) {
        if (half == 0) {
            ChainedSums<0, 6, 8> phase;
            stream(phase);
        } else {
            ChainedSums<1, 6, 6> phase;
            stream(phase);
        }
    } else {
        EitherHalf<8> phase{half};
        stream(phase);
    }
#ifdef WG_TIMESTAMPS
    report();
#endif
}

template <int LAYOUT, int MODE, bool Q8, bool WIDE, class ENC>
hipError_t launch_stream(const RolesCall& c, const ENC& enc, hipStream_t s) {
    // two plane buffers, the transform waves' barrier counter, the parked reverse-scaling factors
    constexpr int lds_bytes = 2 * kLdsBytes + 64 + 4 * (WIDE ? ParkedScales<kAllRows>::kBytes : kParkedScaleBytes);
    static_assert(lds_bytes <= 160 * 1024, "fits the LDS of a compute unit");
    static LdsLimitOnce lds_limit;   // per template instance
    if (hipError_t e = lds_limit.set(reinterpret_cast<const void*>(&fused_conv_stream_kernel<LAYOUT, MODE, Q8, WIDE, ENC>), lds_bytes)) return e;
    const int tile_blocks = ceil_div(c.p.T, kFusedTiles), filter_blocks = c.p.Kp / (kFusedFilters * (WIDE ? 2 : 1));   // Kp is a multiple of 64
    const int gx = stream_workgroups(tile_blocks, filter_blocks);
    fused_conv_stream_kernel<LAYOUT, MODE, Q8, WIDE, ENC><<<dim3(gx, filter_blocks), 512, lds_bytes, s>>>(
        c.x, c.blob, c.bl.table_off, c.bl.planes_off, c.y, c.p, c.q8, tile_blocks, enc);
    return hipGetLastError();
}

// One mode's launches (each mode is compiled in a file of its own).
template <int MODE>
hipError_t launch_stream_mode(const RolesCall& c, bool wide, hipStream_t s) {
    auto form = [&](auto L, auto Q8, const auto& enc) {
        return wide ? launch_stream<L, MODE, Q8, true>(c, enc, s) : launch_stream<L, MODE, Q8, false>(c, enc, s);
    };
    constexpr std::integral_constant<int, WG_NHWC> nhwc{};
    constexpr std::integral_constant<int, WG_NCHW> nchw{};
    if (c.zero != nullptr)   // uint8 tensors: int32 outputs only
        return c.layout == WG_NHWC ? form(nhwc, std::false_type{}, *c.zero) : form(nchw, std::false_type{}, *c.zero);
    if (c.q8.out != nullptr)
        return c.layout == WG_NHWC ? form(nhwc, std::true_type{}, SignedInt8{}) : form(nchw, std::true_type{}, SignedInt8{});
    return c.layout == WG_NHWC ? form(nhwc, std::false_type{}, SignedInt8{}) : form(nchw, std::false_type{}, SignedInt8{});
}

}  // namespace
}  // namespace wg
