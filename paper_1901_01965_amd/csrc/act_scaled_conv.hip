// The complex F(4x4,3x3) path with the activations of every tile scaled as well (act_scale.h), in two kernels: the factors
// of all tiles first, then a role-specialised convolution with them.  One kernel that does both (fused_conv.hip) transforms
// every tile twice per filter block, 2 K / 32 times in all, and the transform is what the kernels of this path are bound by:
// 256 -> 256 channels at 14x14, N = 64: 54 us.  Here a tile is transformed once for its factors and K / 64 times for its
// products, and the products run beside the next channel block's transform.
#include "act_scale.h"
#include "roles_conv.h"
#include "write_through.h"

namespace wg {
namespace {

// ---- factors ---------------------------------------------------------------------------------------------
// One or two waves take longer to bring the factor table than to look it up: 54 -> 48 channels at 51x51, N = 2 19.5 us and 16.4, 90 -> 200
// at 40x40, N = 8 28.3 and 24.4; four, 256 -> 256 at 14x14, N = 64: 26.4 with it in LDS, 26.8 without.
__host__ __device__ inline bool table_in_lds(const Problem& p) { return p.CB > 2; }
// grid: ceil(T / 4), 64 CB threads: wave = 64-channel block, lane = (tile, four channels).  Bound by latency: a patch load, a
// transform, a reduction.  The factor table comes to LDS beside the patch (looked up in memory it was a second trip after the
// reduction), and the reduction over a tile's sixteen lanes stays in the vector ALU.
__global__ __launch_bounds__(1024) void act_factors_kernel(const int8_t* __restrict__ x, WG_GEOMETRY_PARAMS, const uint8_t* __restrict__ blob,
                                                           uint32_t* __restrict__ factors, int32_t* __restrict__ act_table, Problem p) {
    WG_TAKE_GEOMETRY(p, 2);
    __shared__ int maxima[4 * kEntries];
    extern __shared__ uint32_t table[];   // kActMax + 1, or none
    const int tid = threadIdx.x, lane = tid & 63, cb = tid >> 6;
    const BlobHeaderWords header = read_blob_header(blob);
    const int tile = PatchLoader::tile_of(0, lane), t = blockIdx.x * 4 + tile, cq = PatchLoader::quad_of(lane);
    int n = 0, ty = 0, tx = 0;
    if (t < p.T) decode_tile(p, t, n, ty, tx);
    PatchLoader loader;
    loader.enter(p, n, ty, tx, lane);
    loader.drop_absent_channels(p, cb, lane);
    loader.request(activation_buffer(x, p), cb);
    if (table_in_lds(p))
        for (int i = tid; i <= kActMax; i += blockDim.x) table[i] = kActScale.v[i];
    for (int i = tid; i < 4 * kEntries; i += blockDim.x) maxima[i] = 0;
    __syncthreads();
    s16x2 mx[kEntries];
#pragma unroll
    for (int e = 0; e < kEntries; ++e) mx[e] = (s16x2){0, 0};
    transform_patch<StoredInt8>(loader.patch, MaxKeeper{mx});
    // over the sixteen threads of a tile, two entries per register; then one LDS maximum per tile, entry and wave
#pragma unroll
    for (int j = 0; j < kEntries / 2; ++j) {
        s16x2 m = {max(mx[2 * j].x, mx[2 * j].y), max(mx[2 * j + 1].x, mx[2 * j + 1].y)};
        auto with_row_rotated = [&](auto by) {   // by 8, 4, 2, 1 lanes within the sixteen
            m = __builtin_elementwise_max(m, as_s16x2((uint32_t)__builtin_amdgcn_update_dpp(0, (int)as_u32(m), 0x120 + by, 0xf, 0xf, false)));
        };
        with_row_rotated(std::integral_constant<int, 8>{});
        with_row_rotated(std::integral_constant<int, 4>{});
        with_row_rotated(std::integral_constant<int, 2>{});
        with_row_rotated(std::integral_constant<int, 1>{});
        if (cq == j) {
            atomicMax(&maxima[tile * kEntries + 2 * j], (int)m.x);
            atomicMax(&maxima[tile * kEntries + 2 * j + 1], (int)m.y);
        }
    }
    __syncthreads();
    if (!blob_matches(header, p.K, p.Cf, WG_SCALED)) return;
    for (int i = tid; i < 4 * kEntries; i += blockDim.x) {
        const size_t at = (size_t)blockIdx.x * 4 * kEntries + i;   // [tile][entry]
        if (at >= (size_t)p.T * kEntries) break;
        const int largest = min(maxima[i], kActMax);
        const uint32_t entry = table_in_lds(p) ? table[largest] : kActScale.v[largest];
        factors[at] = entry;
        if (act_table != nullptr) *reinterpret_cast<v4i*>(act_table + 4 * at) = act_table_row(entry);
    }
}

// ---- products ---------------------------------------------------------------------------------------------
// A wave's half of the entries; every sum is a matrix-core accumulator for the whole kernel.  A complex entry multiplies with
// Wr and Wi only: Re = Dr Wr - Di Wi needs an accumulator of its own for Di Wi.
template <int HALF, int RING>
struct ActProducts {
    using Phase = ProductPhase<kScaledTwoPlanes, HALF>;
    static constexpr int NE = Phase::NE, NB = Phase::NB;
    static constexpr int acc_start(int slot) {   // real: D W; complex: Dr Wr, Im, Di Wi
        int n = 0;
        for (int s = 0; s < slot; ++s) n += is_real(half_slot(HALF, s).entry) ? 1 : 3;
        return n;
    }
    static constexpr int kAcc = acc_start(NE);
    v4i ring[RING], acc[kAcc];
    __device__ inline void clear() {
#pragma unroll
        for (int i = 0; i < kAcc; ++i) acc[i] = (v4i){0, 0, 0, 0};
    }
    __device__ inline void prefetch(const LaneContext& cx) {
        static_for<(NB < RING ? NB : RING)>([&](auto I) { ring[I] = Phase::template load_b<I>(cx); });
    }
    __device__ inline void run(const LaneContext& cx) {
        static_for<NE>([&](auto S) {
            constexpr int entry = half_slot(HALF, S).entry, b = b_start<kScaledTwoPlanes>(HALF, S), v = acc_start(S);
            constexpr int plane = is_real(entry) ? entry : kRealEntries + 2 * (entry - kRealEntries);
            const v4i re = *reinterpret_cast<const v4i*>(cx.a_lds + plane * kPlaneBytes);
            auto mac = [&](int to, v4i d, int filter) {
                acc[v + to] = __builtin_amdgcn_mfma_i32_16x16x64_i8(d, ring[(b + filter) % RING], acc[v + to], 0, 0, 0);
            };
            mac(0, re, 0);
            if constexpr (!is_real(entry)) {
                const v4i im = *reinterpret_cast<const v4i*>(cx.a_lds + (plane + 1) * kPlaneBytes);
                mac(1, re, 1);
                mac(2, im, 1);
                mac(1, im, 0);
            }
            static_for<num_b<kScaledTwoPlanes>(entry)>([&](auto I) {
                if constexpr (b + I + RING < NB) ring[(b + I) % RING] = Phase::template load_b<b + I + RING>(cx);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    // The filter's reverse scaling, then the tile's (register q of a lane belongs to tile 4 (lane / 16) + q), and the output
    // transform.
    // NARROW: no channel sum exceeds 23 bits (see launch_act_scaled_roles), so the filter's scaling is a 24-bit multiply-add and a
    // shift.  The tile's factors come as rounding << 16 | r << 8 | q: the funnel shift looks at the low five bits only.
    template <bool NARROW>
    __device__ inline void finish(const LaneContext& cx, const uint32_t* rq_tab, int lane, v4i (&Y)[16]) const {
        v4i er[6], ei[6];
        static_for<NE>([&](auto S) {
            constexpr Slot sl = half_slot(HALF, S);
            constexpr int v = acc_start(S);
            v4i re = acc[v], im = {0, 0, 0, 0};
            if constexpr (!is_real(sl.entry)) {
                re -= acc[v + 2];
                im = acc[v + 1];
            }
            const ReverseScale by_filter = parked_scale<S>(cx);
            auto filter_side = [&](int m) { return NARROW ? (__mul24(m, by_filter.r) + by_filter.rnd) >> by_filter.q : by_filter(m); };
            const v4i rq = *reinterpret_cast<const v4i*>(rq_tab + sl.entry * 16 + 4 * (lane >> 4));
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const ReverseScale tile_side((rq[q] >> 8) & 255, rq[q], (int)((uint32_t)rq[q] >> 16));
                re[q] = tile_side(filter_side(re[q]));
                if constexpr (!is_real(sl.entry)) im[q] = tile_side(filter_side(im[q]));
            }
            place_entry<HALF, S>(re, im, er, ei, Y);
        });
    }
};

constexpr int kActPlaneBuffer = kActPlanes * kPlaneBytes;   // 36 KB per channel block, double-buffered
// The transform's factors lie behind the planes, where (PW = 8) the second half of the outputs is staged later; what the
// finishing lanes read lies behind what is staged.
constexpr int kActFactorsOff = kLdsBytes;
template <int PW> constexpr int act_rq_off() { return PW == 8 ? 2 * kLdsBytes : kLdsBytes + kActNpBytes; }
template <int PW> constexpr int act_lds_bytes() { return act_rq_off<PW>() + kActRqBytes + PW * kParkedScaleBytes; }
static_assert(2 * kActPlaneBuffer <= kLdsBytes && act_lds_bytes<8>() <= 160 * 1024, "LDS of one compute unit");

// grid (ceil(T/16), ceil(K / (8 PW))), 64 (4 + PW) threads: the roles of fused_conv_roles_kernel (roles_kernel.h): waves 0-3 transform one
// channel block ahead, the others multiply; product wave pw owns filter block pw % (PW / 2) and half pw / (PW / 2) of the entries.
template <int LAYOUT, int OUT, int PW, bool NARROW>
__global__ __launch_bounds__(64 * (4 + PW)) void act_scaled_roles_kernel(const int8_t* __restrict__ x, WG_GEOMETRY_PARAMS,
                                                                         WG_ORDER_PARAMS, const uint8_t* __restrict__ blob,
                                                                         size_t table_off, size_t planes_off, int32_t* __restrict__ y,
                                                                         const uint32_t* __restrict__ factors, Problem p) {
    WG_TAKE_GEOMETRY(p, 2);
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int bx, by;
    WG_TAKE_ORDER.place(bx, by);
    const int tile0 = bx * kFusedTiles, k0 = by * 8 * PW;
    const BlobHeaderWords header = read_blob_header(blob);   // compared by either role, see fused_conv_roles_kernel
    auto matches = [&] { return blob_matches(header, p.K, p.Cf, WG_SCALED); };
    uint32_t* const np_tab = reinterpret_cast<uint32_t*>(lds + kActFactorsOff);
    uint32_t* const rq_tab = reinterpret_cast<uint32_t*>(lds + act_rq_off<PW>());
    // the tiles' factors; tiles beyond the last one keep n = 1
    auto expand_factors = [&] {
        for (int i = threadIdx.x; i < 16 * kEntries; i += 64 * (4 + PW)) {
            const int tile = i / kEntries, e = i - tile * kEntries;
            const uint32_t entry = tile0 + tile < p.T ? factors[(size_t)tile0 * kEntries + i] : 0x00010000u;
            np_tab[i] = act_factors(entry);
            const uint32_t r = (entry >> 16) & 255u, q = entry >> 24;
            rq_tab[e * 16 + tile] = ((1u << q) >> 1) << 16 | r << 8 | q;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
    };

    if (wave < 4) {
        const int a_tile = PatchLoader::tile_of(wave, lane), a_cq = PatchLoader::quad_of(lane), a_t = tile0 + a_tile;
        int n = 0, ty = 0, tx = 0;
        if (a_t < p.T) decode_tile(p, a_t, n, ty, tx);
        const __amdgpu_buffer_rsrc_t xbuf = activation_buffer(x, p);
        PatchLoader loader;
        loader.enter(p, n, ty, tx, lane);
        loader.drop_absent_channels(p, 0, lane);
        loader.request(xbuf, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (!matches()) return;
        ScaledPlanes out;
        int8_t* const slot = lds + lds_slot(a_cq >> 2, a_tile) * 16 + (a_cq & 3) * 4;
        out.np = np_tab + a_tile * kEntries;
        expand_factors();
        for (int cb = 0; cb < p.CB; ++cb) {
            if (cb > 0) {   // barrier cb
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
            }
            out.sink.base = slot + (cb & 1) * kActPlaneBuffer;
            if (cb + 1 < p.CB) {
                loader.drop_absent_channels(p, cb + 1, lane);
                transform_patch<StoredInt8>(loader.patch, out, SignedInt8{}, NextColumns{loader, xbuf, cb + 1});
            } else {
                transform_patch<StoredInt8>(loader.patch, out);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();   // barrier CB: the last block's planes are published
        __syncthreads();                // the two barriers of the product waves' store
        __syncthreads();
        return;
    }

    if (!matches()) return;
    const int pw = wave - 4, kblock_all = pw % (PW / 2), half = pw / (PW / 2);
    const int kblock = kblock_all & 1, group = kblock_all >> 1;
    const int k = k0 + kblock_all * 16 + (lane & 15);
    LaneContext cx;
    cx.table_k = reinterpret_cast<const ScaleEntry*>(blob + table_off) + (size_t)k * kEntries;
    int8_t* const scale_area = lds + act_rq_off<PW>() + kActRqBytes + pw * kParkedScaleBytes;
    constexpr int NP = 46;
    const int8_t* const b_wave = filter_fragments(blob + planes_off, k - (lane & 15), p.Kp, NP);
    cx.b_lane = fragment_lane(lane);
    const size_t b_block_stride = (size_t)(p.Kp >> 4) * NP * kFilterFragBytes;
    v4i Y[16];
    // one loop per half (the same barriers in both), so that each is allocated registers on its own
    auto blocks = [&](auto H) {
        ActProducts<H, 8> products;
        ParkedScales<H> scales;
        scales.ask(cx, lane);
        cx.b_glob = b_wave;
        products.prefetch(cx);
        scales.park(cx, scale_area, lane);
        products.clear();
        expand_factors();
        for (int cb = 0; cb < p.CB; ++cb) {
            if (cb > 0) {
                cx.b_glob = b_wave + cb * b_block_stride;
                products.prefetch(cx);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();   // barrier cb + 1
            cx.a_lds = lds + (cb & 1) * kActPlaneBuffer + lds_slot(lane >> 4, lane & 15) * 16;
            products.run(cx);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) Y[i] = (v4i){0, 0, 0, 0};
        products.template finish<NARROW>(cx, rq_tab, lane, Y);
    };
    if (half == 0) blocks(std::integral_constant<int, 0>{}); else blocks(std::integral_constant<int, 1>{});
    StoreContext sc;
    sc.lds = lds + group * kLdsBytes;   // the 32-filter halves of the workgroup stage and store side by side
    sc.tid = (2 * half + kblock) * 64 + lane;
    sc.lane = lane; sc.rnd = 8; sc.y = y;
    locate_tile<LAYOUT>(sc, p, tile0);
    __syncthreads();   // the operand planes are dead
    stage_outputs(sc.lds, lane, half, kblock, Y);
    __syncthreads();
    store_staged<LAYOUT, OUT, true>(sc, p, Int8Epilogue{}, k0 + group * kFusedFilters);
}

}  // namespace

hipError_t launch_act_factors(const RolesCall& c, uint32_t* factors, int32_t* act_table, hipStream_t s) {
    act_factors_kernel<<<ceil_div(c.p.T, 4), 64 * c.p.CB, table_in_lds(c.p) ? (kActMax + 1) * sizeof(uint32_t) : 0, s>>>(c.x, WG_GEOMETRY(c.p), c.blob, factors, act_table, c.p);
    return hipGetLastError();
}

hipError_t launch_act_scaled_roles(const RolesCall& c, const uint32_t* factors, hipStream_t s) {
    // 64 filters per workgroup unless 32 fill the compute units in one round, or in so few rounds that a half-empty 64-filter block
    // costs more: a round of 32 takes about four fifths of one of 64 (both kernels together, us, 64 / 32 filters: three rounds against
    // four, 480 -> 80 at 59x79, N = 14, 108.8 / 126.3; six against eight, 79 -> 80 at 27x34, N = 169, 106.2 / 114.8; two each, 59 -> 32
    // at 47x47, N = 57, 49.2 / 43.2; 350 drawn layers 0.01 % behind the better one on average, with the line at 1.34 0.08).
    auto launch = [&](auto L, auto OUT, auto W, auto NARROW) -> hipError_t {
        constexpr int PW = W;
        static LdsLimitOnce lds_limit;   // per instance
        if (hipError_t e = lds_limit.set(reinterpret_cast<const void*>(&act_scaled_roles_kernel<L, OUT, PW, NARROW>), act_lds_bytes<PW>())) return e;
        const dim3 grid(ceil_div(c.p.T, kFusedTiles), ceil_div(c.p.K, 8 * PW));
        const GridOrder order(grid, workgroup_order(c.p, WG_SCALED, 8 * PW));
        act_scaled_roles_kernel<L, OUT, PW, NARROW><<<grid, 64 * (4 + PW), act_lds_bytes<PW>(), s>>>(
            c.x, WG_GEOMETRY(c.p), WG_ORDER(order), c.blob, c.bl.table_off, c.bl.planes_off, c.y, factors, c.p);
        return hipGetLastError();
    };
    using std::integral_constant;
    const bool through = f4_through(c.p, c.y, c.layout);
    auto go = [&](auto L, auto W, auto NARROW) {
        return through ? launch(L, integral_constant<int, kOutThrough>{}, W, NARROW) : launch(L, integral_constant<int, kOutInt32>{}, W, NARROW);
    };
    const int tile_blocks = ceil_div(c.p.T, kFusedTiles), cus = compute_units();
    auto rounds = [&](int filters) { return ((long long)tile_blocks * ceil_div(c.p.K, filters) + cus - 1) / cus; };
    const bool wide = rounds(32) > 1 && 4 * rounds(32) >= 5 * rounds(64);
    // a channel sum is at most 2 x 127 x 127 C (Re = Dr Wr - Di Wi), r at most 255
    const bool narrow = 2ll * 127 * 127 * c.p.Cf < 1 << 23;
    static_assert(((1ll << 23) - 1) * 255 + 64 < 1ll << 31, "a narrow sum times r, rounded, fits int32");
    auto form = [&](auto L, auto W) { return narrow ? go(L, W, std::true_type{}) : go(L, W, std::false_type{}); };
    if (c.layout == WG_NHWC)
        return wide ? form(integral_constant<int, WG_NHWC>{}, integral_constant<int, 8>{}) : form(integral_constant<int, WG_NHWC>{}, integral_constant<int, 4>{});
    return wide ? form(integral_constant<int, WG_NCHW>{}, integral_constant<int, 8>{}) : form(integral_constant<int, WG_NCHW>{}, integral_constant<int, 4>{});
}

}  // namespace wg
