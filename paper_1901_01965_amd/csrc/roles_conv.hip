// The single-kernel convolution with the two kinds of work on different waves: fused_conv_roles_kernel (one tile block
// per workgroup) and fused_conv_stream_kernel (a workgroup walks over many).  See fused_conv.hip for the method and
// the dispatch.
#include "product_core.h"

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
// PW = 8 (channels-last, 4-byte buffer loads, K % 4 = 0): eight product waves, twelve waves in all, 64 filters per workgroup.
// On deep layers the workgroup's pace is set by the transform waves and by what the compute unit's vector-memory path
// takes in, while the product waves of the eight-wave form idle half of the time: with two product waves per SIMD one
// transform (and one set of patch loads) serves twice the filters.  Product wave pw owns filter block pw % 4 and half
// pw / 4 of the entries.  Three waves per SIMD leave a wave 168 registers, so in both modes the product waves keep 18
// joined channel sums (scaled mode: instead of the 36 resident limb accumulators), with a loop per half so that each
// half is allocated registers on its own, and the transform waves form their patch offsets per load.  The two 32-filter
// halves stage their outputs in one operand buffer each and store at the same time.
#ifdef WG_TIMESTAMPS
// Development aid (never compiled into the library): per-wave sums of the time spent in each part of the channel-block loop.
__device__ unsigned long long* g_roles_stamps = nullptr;
#define WG_CLOCK() __builtin_amdgcn_s_memtime()
#define WG_SPENT(i, since) do { const unsigned long long now_ = WG_CLOCK(); spent[i] += now_ - (since); (since) = now_; } while (0)
#else
#define WG_SPENT(i, since) do { } while (0)
#endif

template <int LAYOUT, bool VEC4, int MODE, bool SUMS, bool Q8, int PW = 4>
__global__ __launch_bounds__(64 * (4 + PW)) void fused_conv_roles_kernel(const int8_t* __restrict__ x, const uint8_t* __restrict__ blob,
                                                                         size_t table_off, size_t planes_off, int32_t* __restrict__ y,
                                                                         Problem p, Int8Epilogue q8) {
    static_assert(PW == 4 || (PW == 8 && VEC4 && SUMS && LAYOUT == WG_NHWC), "eight product waves: channels-last, buffer loads, channel sums");
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    const int lane = threadIdx.x & 63, wave8 = threadIdx.x >> 6;
    const bool transforms = wave8 < 4;
    const int tid = threadIdx.x & 255, wave = wave8 & 3;   // within the role (PW = 8: within the four waves that store together)
    int bx = blockIdx.x, by = blockIdx.y;
    {
        const int total = gridDim.x * gridDim.y;
        if (gridDim.y >= 2 && (total & 7) == 0) {   // XCD-major order, as in fused_conv_body
            const int launch = blockIdx.y * gridDim.x + blockIdx.x;
            const int w = (launch & 7) * (total >> 3) + (launch >> 3);
            by = w / (int)gridDim.x;
            bx = w - by * (int)gridDim.x;
        }
    }
    const int tile0 = bx * kFusedTiles, k0 = by * (kFusedFilters * (PW / 4));
    if (!blob_matches(reinterpret_cast<const BlobHeader*>(blob), p.K, p.C, MODE)) return;
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
        const int a_tile = tid >> 4, a_cq = tid & 15;
        const int a_t = tile0 + a_tile;
        const int a_tx = __shfl(my_tx, a_tile), a_ty = __shfl(my_ty, a_tile), a_n = __shfl(my_n, a_tile);
        OperandSplitter<MODE == WG_SCALED ? kSplitByteLimbs : kSplitTwoLimb, LdsPlaneSink> out;
        int8_t* const slot = lds + lds_slot(a_cq >> 2, a_tile) * 16 + (a_cq & 3) * 4;
        uint32_t patch[6][6];
        // 4-byte pixel loads: the 36 offsets of the patch (relative to x: they fit 32 bits) are
        // formed once; a channel block is then a uniform offset on top of these.  Scaled mode,
        // where these waves set the pace, loads through the buffer descriptor (no select per
        // pixel); lossless mode, where the product waves do, measured 3 % faster with plain
        // loads from clamped addresses.
        constexpr bool kBuffer = VEC4 && (MODE == WG_SCALED || PW == 8);
        uint32_t pixel[VEC4 && PW == 4 ? 36 : 1];
        uint32_t row_off[PW == 8 ? 6 : 1], col_off[PW == 8 ? 6 : 1];   // PW = 8: offsets are formed per load (registers are scarce)
        const __amdgpu_buffer_rsrc_t xbuf = activation_buffer(x, p);
        auto request = [&](int cb) {
            if constexpr (PW == 8) {
                // channel groups beyond C (last block of a C that is not a multiple of 64: a uniform branch) get zeros
                const bool have = (cb + 1) * kCBlock <= p.C || cb * kCBlock + 4 * a_cq < p.C;
#pragma unroll
                for (int i = 0; i < 36; ++i) {
                    const uint32_t at = __builtin_elementwise_add_sat(row_off[i / 6], col_off[i % 6]);
                    patch[i / 6][i % 6] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(xbuf, have ? at : kOutsideOffset, cb * kCBlock, 0);
                }
            } else if constexpr (kBuffer) {
                request_patch(xbuf, p, pixel, cb, 4 * a_cq, patch);
            } else if constexpr (VEC4) {
                const int c0 = cb * kCBlock + 4 * a_cq;
                const int8_t* base = x + (c0 < p.C ? c0 : 0);
#pragma unroll
                for (int i = 0; i < 36; ++i) patch[i / 6][i % 6] = *reinterpret_cast<const uint32_t*>(base + pixel[i]);
            } else {
                load_patch<LAYOUT, false>(x, p, a_n, a_ty, a_tx, cb * kCBlock + 4 * a_cq, patch);
            }
        };
        if constexpr (PW == 8) {
            const int h0 = 4 * a_ty - 1, w0 = 4 * a_tx - 1;
            const uint32_t image = (uint32_t)a_n * (uint32_t)p.H * (uint32_t)p.W * (uint32_t)p.C + (uint32_t)(4 * a_cq);
#pragma unroll
            for (int a = 0; a < 6; ++a) {
                row_off[a] = (unsigned)(h0 + a) < (unsigned)p.H ? image + (uint32_t)(h0 + a) * (uint32_t)p.W * (uint32_t)p.C : kOutsideOffset;
                col_off[a] = (unsigned)(w0 + a) < (unsigned)p.W ? (uint32_t)(w0 + a) * (uint32_t)p.C : kOutsideOffset;
            }
        } else if constexpr (kBuffer) {
            patch_offsets(p, a_n, a_ty, a_tx, 4 * a_cq, pixel);
        } else if constexpr (VEC4) {
            const int h0 = 4 * a_ty - 1, w0 = 4 * a_tx - 1;
            const uint32_t image = (uint32_t)a_n * (uint32_t)p.H * (uint32_t)p.W * (uint32_t)p.C;
#pragma unroll
            for (int a = 0; a < 6; ++a)
#pragma unroll
                for (int b = 0; b < 6; ++b)
                    pixel[6 * a + b] = image + ((uint32_t)min(max(h0 + a, 0), p.H - 1) * (uint32_t)p.W +
                                                (uint32_t)min(max(w0 + b, 0), p.W - 1)) * (uint32_t)p.C;
        }
        if (a_t < p.T) request(0);
        WG_SPENT(3, mark);
        for (int cb = 0; cb < p.CB; ++cb) {
            if (cb > 0) {   // barrier cb
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
            }
            WG_SPENT(0, mark);   // LDS writes landed + barrier
            out.sink.base = slot + (cb & 1) * kLdsBytes;
            if (a_t < p.T) {
#ifdef WG_TIMESTAMPS
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                WG_SPENT(1, mark);   // wait for the patch
#endif
                if constexpr (kBuffer) bias_buffer_patch(patch);
                else bias_patch(p, a_ty, a_tx, cb * kCBlock + 4 * a_cq, patch);
                transform_patch(patch, out);
                WG_SPENT(2, mark);   // transform
                if (cb + 1 < p.CB) request(cb + 1);
                WG_SPENT(3, mark);   // requests
            }
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
    // waves of filter blocks 2 group, 2 group + 1 store together (`wave` counts within that group, as store_block expects)
    const int pw = wave8 - 4;
    const int kblock4 = PW == 8 ? (pw & 3) : (wave & 1), half = PW == 8 ? (pw >> 2) : (wave >> 1);
    const int kblock = kblock4 & 1, group = kblock4 >> 1;
    const int k = k0 + kblock4 * 16 + (lane & 15);
    LaneContext cx;
    cx.table_k = reinterpret_cast<const ScaleEntry*>(blob + table_off) + (size_t)k * kEntries;
    cx.parked = nullptr;
    constexpr bool PARKED = SUMS && MODE == WG_SCALED;
    int8_t* const scale_area = lds + 2 * kLdsBytes + pw * kParkedScaleBytes;   // behind the two plane buffers: 1 KB per product wave
    constexpr int NP = MODE == WG_LOSSLESS ? 138 : 46;
    const int8_t* b_lane = reinterpret_cast<const int8_t*>(blob + planes_off) +
                           filter_plane_offset(0, 0, k, (lane >> 4) * 16, p.Kp, NP);
    const size_t b_block_stride = (size_t)(p.Kp >> 4) * NP * kFilterFragBytes;
    v4i Y[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) Y[i] = (v4i){0, 0, 0, 0};
    // SUMS: the product waves do no output transform per block.  Scaled: all 36 limb-product
    // accumulators stay resident (PW = 4), or 18 joined channel sums (PW = 8: 168 registers per wave); lossless: 18
    // joined channel sums (54 accumulators would not fit).
    constexpr bool RESIDENT = SUMS && MODE == WG_SCALED && PW == 4;
    constexpr int kLeanRing = PW == 8 ? (MODE == WG_SCALED ? 10 : 6) : 8;
    std::conditional_t<RESIDENT, ResidentScaled<0>, LeanProducts<MODE, 0, SUMS, kLeanRing>> phase0;
    std::conditional_t<RESIDENT, ResidentScaled<1>, LeanProducts<MODE, 1, SUMS, kLeanRing>> phase1;
    constexpr int kSumRegs = RESIDENT ? 36 : (SUMS ? kChannelSums : 1);
    v4i sums[kSumRegs];
    if constexpr (SUMS) {
#pragma unroll
        for (int i = 0; i < kSumRegs; ++i) sums[i] = (v4i){0, 0, 0, 0};
    }
    if constexpr (PW == 8) {
        // one loop per half (the same barriers in both), so that each is allocated registers on its own
        auto blocks = [&](auto& phase, auto H) {
            // the first block's filter prefetch goes out between the request for the reverse-scaling factors and their parking
            ParkedScales<H> scales;
            if constexpr (PARKED) scales.ask(cx, lane);
            cx.b_glob = b_lane;
            phase.prefetch(cx);
            if constexpr (PARKED) scales.park(cx, scale_area, lane);
            for (int cb = 0; cb < p.CB; ++cb) {
                if (cb > 0) {
                    cx.b_glob = b_lane + cb * b_block_stride;
                    phase.prefetch(cx);
                }
                WG_SPENT(3, mark);   // ring prefetch issue
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();   // barrier cb + 1
                WG_SPENT(0, mark);   // barrier
                cx.a_lds = lds + (cb & 1) * kLdsBytes + lds_slot(lane >> 4, lane & 15) * 16;
                phase.run(cx, sums, Y);
                WG_SPENT(2, mark);   // products
            }
        };
        if (half == 0) blocks(phase0, std::integral_constant<int, 0>{}); else blocks(phase1, std::integral_constant<int, 1>{});
    } else {
        cx.b_glob = b_lane;
        if (half == 0) {
            ParkedScales<0> scales;
            if constexpr (PARKED) scales.ask(cx, lane);
            phase0.prefetch(cx);
            if constexpr (PARKED) scales.park(cx, scale_area, lane);
        } else {
            ParkedScales<1> scales;
            if constexpr (PARKED) scales.ask(cx, lane);
            phase1.prefetch(cx);
            if constexpr (PARKED) scales.park(cx, scale_area, lane);
        }
        for (int cb = 0; cb < p.CB; ++cb) {
            if (cb > 0) {
                cx.b_glob = b_lane + cb * b_block_stride;
                if (half == 0) phase0.prefetch(cx); else phase1.prefetch(cx);
            }
            WG_SPENT(3, mark);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();   // barrier cb + 1
            WG_SPENT(0, mark);
            cx.a_lds = lds + (cb & 1) * kLdsBytes + lds_slot(lane >> 4, lane & 15) * 16;
            if constexpr (RESIDENT) {
                if (half == 0) phase0.run(cx, sums); else phase1.run(cx, sums);
            } else {
                if (half == 0) phase0.run(cx, sums, Y); else phase1.run(cx, sums, Y);
            }
            WG_SPENT(2, mark);
        }
    }
#ifdef WG_TIMESTAMPS
    report();
#endif
    if constexpr (RESIDENT) {
        if (half == 0) ResidentScaled<0>::finish(cx, sums, Y);
        else           ResidentScaled<1>::finish(cx, sums, Y);
    } else if constexpr (SUMS && MODE == WG_SCALED) {
        if (half == 0) ScaledSums<0>::template finish<0, true>(cx, sums, Y);
        else           ScaledSums<1>::template finish<0, true>(cx, sums, Y);
    } else if constexpr (SUMS) {
        if (half == 0) LeanProducts<MODE, 0, true>::finish_lossless(sums, Y);
        else           LeanProducts<MODE, 1, true>::finish_lossless(sums, Y);
    }
    const int my_row = 4 * my_ty, my_col = 4 * my_tx;
    int my_origin = -1;
    if (tile0 + (lane & 15) < p.T)
        my_origin = LAYOUT == WG_NHWC ? ((my_n * p.H + my_row) * p.W + my_col) * p.K
                                      : (my_n * p.K * p.H + my_row) * p.W + my_col;
    if constexpr (PW == 8) {
        // the two 32-filter halves of the workgroup stage in one operand buffer each and store side by side (the host
        // gives this form only channels-last outputs with K % 4 = 0, the layout store_block's two parts exist for)
        const int gtid = (2 * half + kblock) * 64 + lane;
        const StoreContext sc = {lds + group * kLdsBytes, gtid, lane, 2 * half + kblock, half, kblock, my_n, my_row, my_col, my_origin,
                                 MODE == WG_SCALED ? 8 : 0, y};
        __syncthreads();   // the operand planes are dead
        store_block<LAYOUT, Q8, 1>(sc, p, q8, Y, k0 + group * kFusedFilters);
        __syncthreads();
        store_block<LAYOUT, Q8, 2>(sc, p, q8, Y, k0 + group * kFusedFilters);
#ifdef WG_TIMESTAMPS
        if (g_roles_stamps != nullptr && lane == 0)
            g_roles_stamps[((size_t)(blockIdx.y * gridDim.x + blockIdx.x) * 12 + wave8) * 8 + 5] = WG_CLOCK() - entered;
#endif
    } else {
        const StoreContext sc = {lds, tid, lane, wave, half, kblock, my_n, my_row, my_col, my_origin,
                                 MODE == WG_SCALED ? 8 : 0, y};
        __syncthreads();   // the operand planes are dead
        store_block<LAYOUT, Q8>(sc, p, q8, Y, k0);
#ifdef WG_TIMESTAMPS
        if (g_roles_stamps != nullptr && lane == 0)
            g_roles_stamps[((size_t)(blockIdx.y * gridDim.x + blockIdx.x) * 12 + wave8) * 8 + 5] = WG_CLOCK() - entered;
#endif
    }
}

template <int LAYOUT, bool VEC4, int MODE, bool SUMS, bool Q8, int PW = 4>
hipError_t launch_roles(const int8_t* x, const uint8_t* blob, const BlobLayout& bl, int32_t* y, const Problem& p,
                        const Int8Epilogue& q8, hipStream_t s) {
    constexpr int lds_bytes = 2 * kLdsBytes + PW * kParkedScaleBytes;   // two plane buffers, the parked reverse-scaling factors
    static_assert(lds_bytes <= 160 * 1024, "fits the LDS of a compute unit");
    static LdsLimitOnce lds_limit;   // per template instance
    if (hipError_t e = lds_limit.set(reinterpret_cast<const void*>(&fused_conv_roles_kernel<LAYOUT, VEC4, MODE, SUMS, Q8, PW>), lds_bytes)) return e;
    dim3 grid(ceil_div(p.T, kFusedTiles), p.Kp / (kFusedFilters * (PW / 4)));   // Kp is a multiple of 64
    fused_conv_roles_kernel<LAYOUT, VEC4, MODE, SUMS, Q8, PW><<<grid, 64 * (4 + PW), lds_bytes, s>>>(x, blob, bl.table_off, bl.planes_off, y, p, q8);
    return hipGetLastError();
}

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
template <int MODE, bool Q8, bool WIDE = false>
__global__ __launch_bounds__(512) void fused_conv_stream_kernel(const int8_t* __restrict__ x, const uint8_t* __restrict__ blob,
                                                                size_t table_off, size_t planes_off, int32_t* __restrict__ y,
                                                                Problem p, Int8Epilogue q8, int tile_blocks) {
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    const int lane = threadIdx.x & 63, wave8 = threadIdx.x >> 6;
    const bool transforms = wave8 < 4;
    const int tid = threadIdx.x & 255, wave = wave8 & 3;   // within the role
    const int k0 = blockIdx.y * kFusedFilters * (WIDE ? 2 : 1);
    if (!blob_matches(reinterpret_cast<const BlobHeader*>(blob), p.K, p.C, MODE)) return;
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
        const int a_tile = tid >> 4, a_cq = tid & 15;
        OperandSplitter<MODE == WG_SCALED ? kSplitByteLimbs : kSplitTwoLimb, LdsPlaneSink> out;
        int8_t* const slot = lds + lds_slot(a_cq >> 2, a_tile) * 16 + (a_cq & 3) * 4;
        uint32_t patch[6][6], pixel[36];
        int a_t = 0, a_ty = 0, a_tx = 0;
        // identity of the thread's tile in tile block tb, and the 36 pixel offsets of its patch
        auto enter_tile_block = [&](int tb) {
            a_t = tb * kFusedTiles + a_tile;
            int a_n = 0;
            a_ty = 0; a_tx = 0;
            if (a_t < p.T) decode_tile(p, a_t, a_n, a_ty, a_tx);
            patch_offsets(p, a_n, a_ty, a_tx, 4 * a_cq, pixel);
        };
        const __amdgpu_buffer_rsrc_t xbuf = activation_buffer(x, p);
        auto request = [&](int cb) { request_patch(xbuf, p, pixel, cb, 4 * a_cq, patch); };
        // adds the two halves staged in `buffer` for tile block tb and writes them out
        auto flush = [&](int tb, int buffer) {
            int n = 0, ty = 0, tx = 0;
            const int t = tb * kFusedTiles + (lane & 15);
            if (t < p.T) decode_tile(p, t, n, ty, tx);
            const int row = 4 * ty, col = 4 * tx;
            const int origin = t < p.T ? ((n * p.H + row) * p.W + col) * p.K : -1;
            v4i none[16];
            if constexpr (WIDE) {
                constexpr int kCopyBytes = 16 * 16 * 36 * 4;   // one staged copy of 32 filters (store_block's layout)
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const StoreContext sc = {lds + buffer * kLdsBytes + g * kCopyBytes, tid, lane, wave, 0, 0, n, row, col, origin, rnd, y};
                    store_block<WG_NHWC, Q8, 3>(sc, p, q8, none, k0 + g * kFusedFilters);
                }
            } else {
                const StoreContext sc = {lds + buffer * kLdsBytes, tid, lane, wave, 0, 0, n, row, col, origin, rnd, y};
                store_block<WG_NHWC, Q8, 2>(sc, p, q8, none, k0);
            }
        };
        TransformWavesBarrier among_us = {reinterpret_cast<uint32_t*>(lds + 2 * kLdsBytes), 0u};
        if (tid == 0) *among_us.counter = 0u;   // lands before the first s_barrier, long before the first use
        int cb = 0, jb = 0;   // unit u = (tile block number jb of this workgroup, channel block cb)
        if (units > 0) {
            enter_tile_block(blockIdx.x);
            request(0);
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
            if (u < units) {
                out.sink.base = slot + (u & 1) * kLdsBytes;
                if (a_t < p.T) {
#ifdef WG_TIMESTAMPS
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    WG_SPENT(2, mark);   // wait for the patch
#endif
                    bias_buffer_patch(patch);
                    transform_patch(patch, out);
                }
            }
            WG_SPENT(3, mark);   // transform
            const bool last0 = u < units && cb == p.CB - 1;
            if (u < units) {   // next unit's patch, asked for before the waits below so that they cover its latency
                if (++cb == p.CB) { cb = 0; ++jb; }
                if (u + 1 < units) {
                    if (cb == 0) enter_tile_block((int)blockIdx.x + jb * (int)gridDim.x);
                    if (a_t < p.T) request(cb);
                }
            }
            WG_SPENT(5, mark);   // requests
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
    const int8_t* b_lane = reinterpret_cast<const int8_t*>(blob + planes_off) +
                           filter_plane_offset(0, 0, k, (lane >> 4) * 16, p.Kp, NP);
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
            cx.b_glob = b_lane;
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
                cx.b_glob = b_lane + cb * b_block_stride;
                all.prefetch(cx);
            }
            if (last) {
                WG_SPENT(2, mark);   // prefetch issue
                __syncthreads();   // D_u: every product wave has finished reading this unit's planes
                WG_SPENT(3, mark);   // barrier D
                const StoreContext sc = {lds + (u & 1) * kLdsBytes, tid, lane, wave, half, kblock, 0, 0, 0, -1, rnd, y};
                store_block<WG_NHWC, Q8, 1>(sc, p, q8, Y, k0);
                __syncthreads();   // S_u: staged
                WG_SPENT(4, mark);   // staging and barrier S
            }
        }
#ifdef WG_TIMESTAMPS
        report();
#endif
        return;
    }
    // 18 joined channel sums per wave in both modes (36 resident accumulators plus the outputs
    // would not fit the 256 registers here)
    // scaled mode has the registers for a second set of activation fragments (lossless mode would spill)
    LeanProducts<MODE, 0, true, 8, MODE == WG_SCALED> phase0;
    LeanProducts<MODE, 1, true, 8, MODE == WG_SCALED> phase1;
    constexpr int kSumRegs = kChannelSums;
    v4i sums[kSumRegs];
    v4i Y[16];
    int cb = 0;
    if (units > 0) {
        // the first unit's filter prefetch goes out between the request for the reverse-scaling factors and their parking
        cx.b_glob = b_lane;
        if (half == 0) {
            ParkedScales<0> scales;
            if constexpr (MODE == WG_SCALED) scales.ask(cx, lane);
            phase0.prefetch(cx);
            if constexpr (MODE == WG_SCALED) scales.park(cx, scale_area, lane);
        } else {
            ParkedScales<1> scales;
            if constexpr (MODE == WG_SCALED) scales.ask(cx, lane);
            phase1.prefetch(cx);
            if constexpr (MODE == WG_SCALED) scales.park(cx, scale_area, lane);
        }
    }
    for (int u = 0; u < units; ++u) {
        if (cb == 0) {
#pragma unroll
            for (int i = 0; i < kSumRegs; ++i) sums[i] = (v4i){0, 0, 0, 0};
        }
        WG_SPENT(5, mark);   // clearing the sums
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();   // U_{u+1}
        WG_SPENT(0, mark);   // barrier U
        cx.a_lds = lds + (u & 1) * kLdsBytes + lds_slot(lane >> 4, lane & 15) * 16;
        if (half == 0) phase0.run(cx, sums, Y); else phase1.run(cx, sums, Y);
        WG_SPENT(1, mark);   // products
        const bool last = cb == p.CB - 1;
        cb = last ? 0 : cb + 1;
        if (u + 1 < units) {   // the next unit's first filter fragments travel while this one is finished and staged
            cx.b_glob = b_lane + cb * b_block_stride;
            if (half == 0) phase0.prefetch(cx); else phase1.prefetch(cx);
        }
        if (last) {
#pragma unroll
            for (int i = 0; i < 16; ++i) Y[i] = (v4i){0, 0, 0, 0};
            if constexpr (MODE == WG_SCALED) {
                if (half == 0) ScaledSums<0>::template finish<0, true>(cx, sums, Y);
                else           ScaledSums<1>::template finish<0, true>(cx, sums, Y);
            } else {
                if (half == 0) LeanProducts<MODE, 0, true>::finish_lossless(sums, Y);
                else           LeanProducts<MODE, 1, true>::finish_lossless(sums, Y);
            }
            WG_SPENT(2, mark);   // finish
            __syncthreads();   // D_u: every product wave has finished reading this unit's planes
            WG_SPENT(3, mark);   // barrier D
            const StoreContext sc = {lds + (u & 1) * kLdsBytes, tid, lane, wave, half, kblock, 0, 0, 0, -1, rnd, y};
            store_block<WG_NHWC, Q8, 1>(sc, p, q8, Y, k0);
            __syncthreads();   // S_u: staged
            WG_SPENT(4, mark);   // staging and barrier S
        }
    }
#ifdef WG_TIMESTAMPS
    report();
#endif
}

// Workgroups per filter block of the streaming kernel: about one workgroup per compute unit in
// total (a test hook can set a smaller number, so that small problems stream, too).
std::atomic<int> g_stream_workgroups{0};
// Test hook for the streaming kernel's 64-filter form: 0 the library's choice, 1 wherever a layer streams, 2 never.
std::atomic<int> g_stream_variant{0};
int stream_workgroups(int tile_blocks, int filter_blocks) {
    const int forced = g_stream_workgroups.load(std::memory_order_relaxed);
    if (forced > 0) return std::max(1, std::min(tile_blocks, forced));
    // as many as the compute units allow, then as few as still finish in the same number of rounds
    const int wanted = std::max(1, compute_units() / filter_blocks);
    const int rounds = ceil_div(tile_blocks, wanted);
    return std::max(1, ceil_div(tile_blocks, rounds));
}

template <int MODE, bool Q8, bool WIDE = false>
hipError_t launch_stream(const int8_t* x, const uint8_t* blob, const BlobLayout& bl, int32_t* y, const Problem& p,
                         const Int8Epilogue& q8, hipStream_t s) {
    // two plane buffers, the transform waves' barrier counter, the parked reverse-scaling factors
    constexpr int lds_bytes = 2 * kLdsBytes + 64 + 4 * (WIDE ? ParkedScales<kAllRows>::kBytes : kParkedScaleBytes);
    static_assert(lds_bytes <= 160 * 1024, "fits the LDS of a compute unit");
    static LdsLimitOnce lds_limit;   // per template instance
    if (hipError_t e = lds_limit.set(reinterpret_cast<const void*>(&fused_conv_stream_kernel<MODE, Q8, WIDE>), lds_bytes)) return e;
    const int tile_blocks = ceil_div(p.T, kFusedTiles), filter_blocks = p.Kp / (kFusedFilters * (WIDE ? 2 : 1));   // Kp is a multiple of 64
    const int gx = stream_workgroups(tile_blocks, filter_blocks);
    fused_conv_stream_kernel<MODE, Q8, WIDE><<<dim3(gx, filter_blocks), 512, lds_bytes, s>>>(x, blob, bl.table_off, bl.planes_off, y, p,
                                                                                           q8, tile_blocks);
    return hipGetLastError();
}

std::atomic<int> g_scaled_variant{0};

template <bool Q8>
hipError_t launch_roles_mode(const int8_t* x, const uint8_t* b, const BlobLayout& bl, int32_t* y, const Problem& p,
                             int mode, const Int8Epilogue& q8, hipStream_t s, bool wide = false) {
    if (mode == WG_LOSSLESS && wide) return launch_roles<WG_NHWC, true, WG_LOSSLESS, true, Q8, 8>(x, b, bl, y, p, q8, s);
    if (mode == WG_LOSSLESS) return launch_roles<WG_NHWC, true, WG_LOSSLESS, true, Q8>(x, b, bl, y, p, q8, s);
    if (wide) return launch_roles<WG_NHWC, true, WG_SCALED, true, Q8, 8>(x, b, bl, y, p, q8, s);
    return launch_roles<WG_NHWC, true, WG_SCALED, true, Q8>(x, b, bl, y, p, q8, s);
}

}  // namespace

#ifdef WG_TIMESTAMPS
extern "C" int winograd_debug_set_roles_stamps(void* dev_ptr) {
    return hipMemcpyToSymbol(HIP_SYMBOL(g_roles_stamps), &dev_ptr, sizeof dev_ptr) == hipSuccess ? 0 : -5;
}
#endif

void set_scaled_variant(int v) { g_scaled_variant.store(v, std::memory_order_relaxed); }
void set_stream_variant(int v) { g_stream_variant.store(v, std::memory_order_relaxed); }

void set_stream_workgroups(int n) { g_stream_workgroups.store(n > 0 ? n : 0, std::memory_order_relaxed); }

}  // namespace wg
