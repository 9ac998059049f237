// fused_conv_stream_kernel: the role-specialised convolution as a stream over tile blocks.  See fused_conv.hip for the
// method and the dispatch.
#pragma once
#include "pair_products.h"
#include "product_core.h"
#include "roles_conv.h"
#include "write_through.h"

namespace wg {
namespace {

// Barrier among the waves of one role (s_barrier would stop the other role as well): a counter in LDS that only grows,
// one arrival per wave and use.  A wave arrives once its own LDS accesses have completed and leaves when all have arrived.
// Every wave of the role runs the same (workgroup-uniform) sequence of uses, and all are resident together, so the wait ends.
template <int WAVES>
struct RoleBarrier {
    uint32_t* counter;
    uint32_t arrivals;   // what the counter reads once everyone has arrived at the current use
    __device__ inline void sync(int lane) {
        arrivals += WAVES;
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
// Barriers of both roles, in the same order: U_u (u = 1 .. U) publishes the planes of unit u - 1 and frees the buffer of unit
// u - 2; after the last channel block of a tile block, D_u (every product wave has finished reading the planes) and S_u (the
// outputs are staged).  kStreamEight: the product waves meet at a barrier of their own instead of D_u and again between the two
// stagings, and U_{u+2} (there is a U_{U+1}) stands for S_u, so that the transform waves wait for neither; with four product
// waves, whose chain is the longer one, that barrier's polling cost more than it gave (2-3 %).  kStreamPairs: likewise, and the product
// waves store what they staged themselves, before U_{u+2}.
// The staged outputs of unit u - 2 and the planes of unit u share a buffer, and the four transform waves both read the former
// (each thread reads rows that other waves' plane writes cover) and write the latter: between the two they meet at a barrier
// of their own.
// Activations channels-last, C % 4 = 0 (4-byte pixel loads).
// Forms, by who owns what:
//   kStreamHalves:  32 filters per workgroup; four product waves, each half of the entries of 16 filters.
//   kStreamWhole:   64 filters; four product waves, each every entry of its 16 filters, so that one transform serves twice the
//                   filters and no halves are added.  36 joined channel sums next to the fragments would not fit the
//                   registers: each channel block's products go through the output transform at once and the outputs
//                   accumulate, exact in lossless mode (the transform is linear); in scaled mode the reverse scaling applies
//                   to the channel sum (Section 4.2), so there the host uses this form for one-block layers only.
//   kStreamEight:   64 filters; eight product waves, each half of the entries of 16 filters: the tile blocks' fill and finish of
//                   fused_conv_roles_kernel<PW = 8>, a third of its time at two channel blocks, run beside other tile blocks'
//                   work.  The two halves would need twice the staging: the first writes, the second adds to it in LDS, a
//                   longer chain per tile block, which one channel block does not pay for (56x56x64 N = 256 scaled: 77 us
//                   with whole entries, 80 here).  Twelve waves leave 168 registers each: enough with signed channels-last
//                   tensors and with int8 outputs, one or two spilled with uint8, 6 - 12 with channel-major int32 outputs, whose
//                   32 plane offsets also spill 82 - 237 scalar registers (in every form).  It is the fastest form where
//                   fused_conv.hip chooses it, which it does not for those outputs.
//   kStreamPairs:   64 filters, lossless mode, one channel block; eight product waves, each every entry of 8 filters by way of the
//                   limb-pair operand (pair_products.h), whose outputs take half the registers: enough with twelve waves.  Half the chain per
//                   tile block of kStreamWhole, no halves to add, and all eight waves store: ahead where a workgroup has few tile
//                   blocks, so that this chain is not hidden behind others (see fused_conv.hip).  In a long stream twice as many waves read the
//                   activation planes (576 KB a tile block), and with the transform left out the products alone take 5.1 of a tile block's 7.3 us (kStreamWhole):
//                   56x56x64 N = 256 102 us, int8 out 84, with kStreamWhole 94.5 and 80; with the stores left to the transform
//                   waves 98 and 81, and nothing gained in short ones.
// What bounds kStreamWhole (56x56x64, N = 256, clocks per tile block of 64 filters, lossless / scaled): the product wave's chain,
// 13,500 / 12,400 = products with their joins, reverse scaling and output transform 10,700 / 9,800 + staging 880 + from
// there to the next unit's barrier 800 / 1,000 (lossless mode clears the outputs in it, 64 instructions; what the rest waits for, and
// all of it in scaled mode, which clears nothing, is not known) + barriers, waits and prefetch 1,060 / 650.  It issues some 1,200 instructions, an instruction per 5
// clocks alone; but the transform wave on its SIMD (transform 4,300, flush of the staged tile block 4,000, waiting 4,000)
// is the older one and goes first, and their vector instructions together occupy the SIMD for 1,764 x 4.4 + 224 x 8 = 9,600
// (scaled 1,831 x 4.4 + 112 x 8 = 9,000) of those clocks.
template <int FORM> constexpr int stream_filters() { return FORM == kStreamHalves ? 32 : 64; }
template <int FORM> constexpr bool twelve_waves() { return FORM == kStreamEight || FORM == kStreamPairs; }
template <int FORM> constexpr int stream_product_waves() { return twelve_waves<FORM>() ? 8 : 4; }

template <int LAYOUT, int MODE, int OUT, int FORM, class ENC>
__global__ __launch_bounds__(64 * (4 + stream_product_waves<FORM>())) void fused_conv_stream_kernel(
    const int8_t* __restrict__ x, WG_GEOMETRY_PARAMS, WG_ORDER_PARAMS, const uint8_t* __restrict__ blob, size_t table_off,
    size_t planes_off, int32_t* __restrict__ y, Problem p, Int8Epilogue q8, ENC enc) {
    WG_TAKE_GEOMETRY(p, 2);
    const GridOrder order = WG_TAKE_ORDER;
    const int tile_blocks = (p.T + kFusedTiles - 1) / kFusedTiles;
    constexpr int PW = stream_product_waves<FORM>();
    constexpr bool OWN_BARRIER = twelve_waves<FORM>();
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    const int lane = threadIdx.x & 63, wave8 = twelve_waves<FORM>() ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : threadIdx.x >> 6;
    const bool transforms = wave8 < 4;
    const int wave = wave8 & 3;   // within the role
    // Twelve waves have no registers to spare: what follows from the lane is formed where it is needed.  Spilled, it came back behind
    // the loads in flight, in every unit: scaled, 128 -> 128 at 112x112 N = 16, formed 66.4 us, spilled 68.9; 40 mixed
    // layers 1.2 % faster.  (With eight waves, nothing is spilled either way: 16 -> 16 lossless layers lost 11 % to the extra work.)
    auto my_lane = [&] { if constexpr (twelve_waves<FORM>()) return lane_again(); else return lane; };
    int bx, by;
    order.place(bx, by);
    const int k0 = by * stream_filters<FORM>();
    // looked at by either role before it goes on from what does not depend on the blob (see fused_conv_roles_kernel; held in
    // scalar registers from the start, as there, it cost 56x56x64 N = 256 two of 95 us)
    auto matches = [&] { return blob_matches(reinterpret_cast<const BlobHeader*>(blob), p.K, p.Cf, MODE, ENC::kMagic); };
    // this workgroup's tile blocks: bx, bx + gridDim.x, ...
    const int my_blocks = (tile_blocks - bx + order.across - 1) / order.across;
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
        OperandSplitter<MODE == WG_SCALED || FORM == kStreamPairs ? kSplitByteLimbs : kSplitTwoLimb, LdsPlaneSink> out;
        auto slot_of = [&](int l) {   // a lane's four bytes of an operand plane
            const int cq = PatchLoader::quad_of(l);
            return lds + lds_slot(cq >> 2, PatchLoader::tile_of(wave, l)) * 16 + (cq & 3) * 4;
        };
        int8_t* const slot = slot_of(lane);
        PatchBias<ENC> bias, next_bias;   // of the patch being transformed, of the one in flight
        PatchLoader loader;
        auto enter_tile_block = [&](int tb) {
            const int l = my_lane(), t = tb * kFusedTiles + PatchLoader::tile_of(wave, l);
            int n = 0, ty = 0, tx = 0;
            if (t < p.T) decode_tile(p, t, n, ty, tx);
            loader.enter(p, n, ty, tx, l);
            next_bias.enter(p, ty, tx, enc);
        };
        const __amdgpu_buffer_rsrc_t xbuf = activation_buffer(x, p);
        // writes out what is staged in `buffer` for tile block tb
        auto flush = [&](int tb, int buffer) {
            StoreContext sc;
            sc.lds = lds + buffer * kLdsBytes; sc.lane = my_lane(); sc.tid = twelve_waves<FORM>() ? wave * 64 + sc.lane : threadIdx.x & 255; sc.rnd = rnd; sc.y = y;
            // (opaque: what follows from these is formed here, not ahead of the loop: registers are scarce)
            if constexpr (twelve_waves<FORM>() || LAYOUT == WG_NCHW) asm volatile("" : "+v"(sc.tid), "+v"(sc.lane));
            locate_tile<LAYOUT>(sc, p, tb * kFusedTiles);
            if constexpr (FORM != kStreamHalves) {   // one finished copy per 32 filters
                store_staged<LAYOUT, OUT, false>(sc, p, q8, k0);
                sc.lds += kStageHalf * 4;
                store_staged<LAYOUT, OUT, false>(sc, p, q8, k0 + kFusedFilters);
            } else {
                store_staged<LAYOUT, OUT, true>(sc, p, q8, k0);
            }
        };
        RoleBarrier<4> among_us = {reinterpret_cast<uint32_t*>(lds + 2 * kLdsBytes), 0u};
        if (threadIdx.x < 2) among_us.counter[threadIdx.x] = 0u;   // this role's counter and the other's: land before the first s_barrier, long before the first use
        int cb = 0, jb = 0;   // unit u = (tile block number jb of this workgroup, channel block cb)
        if (units > 0) {
            enter_tile_block(bx);
            loader.drop_absent_channels(p, 0, my_lane());
            loader.request(xbuf, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (!matches()) return;
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
            if (FORM != kStreamPairs && last2) {   // staged in the buffer of unit u - 2, which unit u is about to overwrite
                flush(tb2, u & 1);
                among_us.sync(lane);   // every transform wave has read its share before any of them writes planes
            }
            WG_SPENT(1, mark);   // flush
            const int tb = bx + jb * order.across;
            const bool last0 = u < units && cb == p.CB - 1;
            if (u < units) {
                out.sink.base = (twelve_waves<FORM>() ? slot_of(my_lane()) : slot) + (u & 1) * kLdsBytes;
#ifdef WG_TIMESTAMPS
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                WG_SPENT(2, mark);   // wait for the patch
#endif
                // the next unit's patch is asked for as the registers of this one become free
                const bool more = u + 1 < units;
                if (++cb == p.CB) { cb = 0; ++jb; }
                bias = next_bias;
                if (more) {
                    if (cb == 0) enter_tile_block(bx + jb * order.across);
                    loader.drop_absent_channels(p, cb, my_lane());
                }
                place_loop(std::integral_constant<bool, FORM != kStreamWhole || MODE != WG_SCALED>{});
                bias.apply(loader.patch);
                WG_SPENT(5, mark);   // offsets
                if constexpr (FORM == kStreamPairs) {   // one copy of the transform (two spill): what comes after the last unit is asked for in a buffer of nothing
                    const __amdgpu_buffer_rsrc_t next = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(x), 0, more ? p.N * p.H * p.W * p.C : 0, kRawBufferWord3);
                    transform_patch<typename PatchBias<ENC>::Bytes>(loader.patch, out, enc, NextColumns{loader, next, cb});
                } else if (more) {
                    transform_patch<typename PatchBias<ENC>::Bytes>(loader.patch, out, enc, NextColumns{loader, xbuf, cb});
                } else {
                    transform_patch<typename PatchBias<ENC>::Bytes>(loader.patch, out, enc);
                }
            }
            WG_SPENT(3, mark);   // transform
            if (!OWN_BARRIER && last1) {   // D_{u-1}, S_{u-1}
                __syncthreads();
                __syncthreads();
            }
            WG_SPENT(4, mark);   // barriers D and S
            last2 = last1; tb2 = tb1;
            last1 = last0; tb1 = tb;
        }
        if (FORM != kStreamPairs && units > 0) {   // the last unit ends a tile block, staged in its buffer
            if (OWN_BARRIER) {   // U_{U+1}
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
            }
            flush(tb2, (units + 1) & 1);
        }
#ifdef WG_TIMESTAMPS
        report();
#endif
        return;
    }

    if (!matches()) return;
    // 64 filters: those of the workgroup's second 32 are staged as a copy of their own
    const int pw = wave8 - 4;
    const int kblock4 = FORM == kStreamHalves ? (pw & 1) : (pw & 3), half = FORM == kStreamHalves ? (pw >> 1) : (FORM == kStreamWhole ? 0 : pw >> 2);
    const int kblock = kblock4 & 1, copy = FORM == kStreamHalves ? half : kblock4 >> 1;
    const int k = k0 + kblock4 * 16 + (lane & 15);
    RoleBarrier<PW> among_us = {reinterpret_cast<uint32_t*>(lds + 2 * kLdsBytes) + 1, 0u};
    LaneContext cx;
    cx.table_k = reinterpret_cast<const ScaleEntry*>(blob + table_off) + (size_t)k * kEntries;
    cx.parked = nullptr;
    // behind the plane buffers and the barrier counters
    int8_t* const scale_area = lds + 2 * kLdsBytes + 64 + pw * (FORM == kStreamWhole ? ParkedScales<kAllRows>::kBytes : kParkedScaleBytes);
    constexpr int NP = MODE == WG_LOSSLESS ? 138 : 46;
    const int8_t* const b_wave = filter_fragments(blob + planes_off, k - (lane & 15), p.Kp, NP);
    cx.b_lane = fragment_lane(lane);
    const size_t b_block_stride = (size_t)(p.Kp >> 4) * NP * kFilterFragBytes;
    // (lossless mode: 56x56x256 N = 16 takes 76.5 us with it, 75.8 without, which spills others)
    auto lane_here = [&] { if constexpr (FORM == kStreamEight && MODE == WG_SCALED) return lane_again(); else return lane; };
    auto fragment_slot = [&] { const int l = lane_here(); return lds_slot(l >> 4, l & 15) * 16; };
    // stages a tile block's outputs once every product wave is done with the planes of unit u
    auto stage = [&](int u, const v4i (&Y)[16]) {
        int8_t* const at = lds + (u & 1) * kLdsBytes;
        if constexpr (OWN_BARRIER) among_us.sync(lane); else __syncthreads();
        WG_SPENT(3, mark);   // everyone is done with the planes
        if (FORM != kStreamEight || half == 0) stage_outputs(at, lane_here(), copy, kblock, Y);
        if constexpr (FORM == kStreamEight) {
            among_us.sync(lane);
            if (half == 1) add_staged_outputs(at, lane_here(), copy, kblock, Y);
        } else {
            __syncthreads();
        }
        WG_SPENT(4, mark);   // staging
    };
    auto published = [&]() {   // U_{u+1}
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
    };
    if constexpr (FORM == kStreamPairs) {
        // one channel block: a unit is a tile block; `planes_off` is that of the limb-pair planes
        constexpr int RING = 6;
        using All = pairs::WholeProducts<RING>;
        const __amdgpu_buffer_rsrc_t filters = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<int8_t*>(reinterpret_cast<const int8_t*>(blob + planes_off) + filter_pair_offset(0, 0, k0 + kPairFilters * pw, 0, 0, p.Kp)), 0,
            kPairValues * kFilterFragBytes, kRawBufferWord3);
        v4i ring[RING];
        const uint32_t lane16 = fragment_lane(lane);
        static_for<RING>([&](auto F) { ring[F] = All::template fragment<F>(filters, lane16); });
        for (int u = 0; u < units; ++u) {
            published();
            place_loop(std::false_type{});
            pairs::v2i Y[16];
            // (the next unit's first fragments travel while this one is staged)
            All::run(lds + (u & 1) * kLdsBytes + fragment_slot(), ring, Y, [&](auto F) { ring[F % RING] = All::template fragment<(F + RING < All::NF ? F + RING : F % RING)>(filters, lane16); });
            among_us.sync(lane);   // every product wave is done with the planes
            // lane = tile (lane & 15) x filters 8 pw + 2 (lane / 16), + 1
            const int l = lane_here();
            int* const to = reinterpret_cast<int*>(lds + (u & 1) * kLdsBytes) + (pw >> 2) * kStageHalf + (l & 15) * kStageRow + kPairFilters * (pw & 3) + 2 * (l >> 4);
#pragma unroll
            for (int o = 0; o < 16; ++o) *reinterpret_cast<pairs::v2i*>(to + o * 16 * kStageRow) = Y[o];
            among_us.sync(lane);   // staged
            StoreContext sc;
            sc.lds = lds + (u & 1) * kLdsBytes + (pw >> 2) * kStageHalf * 4;
            sc.lane = lane_again(); sc.tid = (pw & 3) * 64 + sc.lane; sc.rnd = rnd; sc.y = y;
            asm volatile("" : "+v"(sc.tid));
            locate_tile<LAYOUT>(sc, p, (bx + u * order.across) * kFusedTiles);
            store_staged<LAYOUT, OUT, false>(sc, p, q8, k0 + (pw >> 2) * kFusedFilters);
        }
    } else if constexpr (FORM == kStreamWhole) {
        // filter ring: lossless mode has twice the fragments per entry and the registers for twelve in flight
        LeanProducts<MODE, kAllRows, MODE == WG_SCALED ? 8 : 12> all;
        v4i Y[16];
        int cb = 0;
        cx.b_glob = b_wave;
        if (units > 0) {
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
            WG_SPENT(5, mark);   // from the staging on: clearing the outputs (lossless)
            published();
            WG_SPENT(0, mark);   // barrier U
            cx.a_lds = lds + (u & 1) * kLdsBytes + fragment_slot();
            place_loop(std::false_type{});
            all.run(cx, Y);
            WG_SPENT(1, mark);   // products
            const bool last = cb == p.CB - 1;
            cb = last ? 0 : cb + 1;
            if (u + 1 < units) {   // the next unit's first filter fragments travel while this one is staged
                cx.b_glob = b_wave + cb * b_block_stride;
                all.prefetch(cx);
            }
            WG_SPENT(2, mark);   // prefetch issue
            if (last) stage(u, Y);
        }
    } else {
        // Channel sums per wave.  A loop per half, whose sums differ in number; lossless mode with four product waves: one loop
        // for both halves (a loop each would spill).
        auto stream = [&](auto& phase) {
            v4i sums[std::remove_reference_t<decltype(phase)>::kSums];
            auto clear = [&]() {
#pragma unroll
                for (int i = 0; i < (int)(sizeof(sums) / sizeof(v4i)); ++i) sums[i] = (v4i){0, 0, 0, 0};
            };
            int cb = 0;
            cx.b_glob = b_wave;
            if (units > 0) phase.enter(cx, scale_area, lane);
            clear();
            for (int u = 0; u < units; ++u) {
                WG_SPENT(5, mark);
                published();
                WG_SPENT(0, mark);   // barrier U
                cx.a_lds = lds + (u & 1) * kLdsBytes + fragment_slot();
                place_loop(std::integral_constant<bool, FORM == kStreamEight>{});
                phase.run(cx, sums);
                WG_SPENT(1, mark);   // products
                const bool last = cb == p.CB - 1;
                cb = last ? 0 : cb + 1;
                // the next unit's first filter fragments travel while this one is finished and staged (eight product waves: while
                // it is staged, for want of registers)
                cx.b_glob = b_wave + cb * b_block_stride;
                if (u + 1 < units && (PW == 4 || !last)) phase.prefetch(cx);
                if (last) {
                    v4i Y[16];
                    phase.finish(cx, sums, Y);
                    // (pinned: left alone, the compiler moves the outputs' arithmetic behind the waits of the staging)
#pragma unroll
                    for (int i = 0; i < 16; ++i) asm volatile("" : "+v"(Y[i]));
                    WG_SPENT(2, mark);   // finish
                    if constexpr (PW == 8) {
                        __builtin_amdgcn_sched_barrier(0);
                        if (u + 1 < units) phase.prefetch(cx);
                    }
                    stage(u, Y);
                    clear();   // (here, so that their registers are free while the outputs are formed)
                }
            }
        };
        if constexpr (MODE == WG_SCALED) {
            if (half == 0) {
                ChainedSums<0, 6, PW == 8 ? 4 : 8, PW == 8> phase;
                stream(phase);
            } else {
                ChainedSums<1, 6, PW == 8 ? 4 : 6, PW == 8> phase;
                stream(phase);
            }
        } else if constexpr (PW == 8) {
            if (half == 0) {
                LosslessSums<0, 6> phase;
                stream(phase);
            } else {
                LosslessSums<1, 6> phase;
                stream(phase);
            }
        } else {
            EitherHalf<8> phase{half};
            stream(phase);
        }
    }
    if (FORM == kStreamEight && units > 0) published();   // U_{U+1}
#ifdef WG_TIMESTAMPS
    report();
#endif
}

template <int LAYOUT, int MODE, int OUT, int FORM, class ENC>
hipError_t launch_stream(const RolesCall& c, const ENC& enc, hipStream_t s) {
    // two plane buffers, the roles' barrier counters, the parked reverse-scaling factors
    constexpr int lds_bytes = 2 * kLdsBytes + 64 + (FORM == kStreamPairs ? 0 : FORM == kStreamWhole ? 4 * ParkedScales<kAllRows>::kBytes : stream_product_waves<FORM>() * kParkedScaleBytes);
    static_assert(lds_bytes <= 160 * 1024, "fits the LDS of a compute unit");
    static LdsLimitOnce lds_limit;   // per template instance
    if (hipError_t e = lds_limit.set(reinterpret_cast<const void*>(&fused_conv_stream_kernel<LAYOUT, MODE, OUT, FORM, ENC>), lds_bytes)) return e;
    const int tile_blocks = ceil_div(c.p.T, kFusedTiles), filter_blocks = ceil_div(c.p.K, stream_filters<FORM>());
    const dim3 grid(stream_workgroups(tile_blocks, filter_blocks), filter_blocks);
    const GridOrder order(grid, workgroup_order(c.p, MODE, stream_filters<FORM>()));
    fused_conv_stream_kernel<LAYOUT, MODE, OUT, FORM, ENC><<<grid, 64 * (4 + stream_product_waves<FORM>()), lds_bytes, s>>>(
        c.x, WG_GEOMETRY(c.p), WG_ORDER(order), c.blob, c.bl.table_off, FORM == kStreamPairs ? c.bl.pairs_off : c.bl.planes_off, c.y, c.p, c.q8, enc);
    return hipGetLastError();
}

// One mode's launches (each mode is compiled in a file of its own).
template <int MODE>
hipError_t launch_stream_mode(const RolesCall& c, StreamForm which, hipStream_t s) {
    auto form = [&](auto L, auto Q8, const auto& enc) {
        auto go = [&](auto FORM) {
            if constexpr (Q8) {
                return launch_stream<L, MODE, kOutInt8, FORM>(c, enc, s);
            } else {
                // in a longer stream the stores are spread over it already (64 -> 64 at 56x56, four tile blocks per workgroup, N = 64, scaled 29.2 us,
                // through 27.0; seven and thirteen level)
                const int tile_blocks = ceil_div(c.p.T, kFusedTiles);
                const bool few = FORM == kStreamEight || tile_blocks <= 4 * stream_workgroups(tile_blocks, ceil_div(c.p.K, stream_filters<FORM>()));
                return few && f4_through(c.p, c.y, c.layout) ? launch_stream<L, MODE, kOutThrough, FORM>(c, enc, s)
                                                                      : launch_stream<L, MODE, kOutInt32, FORM>(c, enc, s);
            }
        };
        using std::integral_constant;
        if constexpr (MODE == WG_LOSSLESS)
            if (which == kStreamPairs) return go(integral_constant<int, kStreamPairs>{});
        if (which == kStreamEight) return go(integral_constant<int, kStreamEight>{});
        if (which == kStreamWhole) return go(integral_constant<int, kStreamWhole>{});
        return go(integral_constant<int, kStreamHalves>{});
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
