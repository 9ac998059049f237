// Small device-side pieces shared by the single-kernel convolution variants.
#pragma once
#include <type_traits>
#include <utility>

#include "input_transform_core.h"

namespace wg {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kTileBlock = 16;                      // tiles per workgroup (one side of the 16x16x64 matrix-core product)
constexpr int kPlaneBytes = kTileBlock * kCBlock;   // one operand plane of a tile block in LDS

// LDS operand plane: the 16-byte piece holding 16 consecutive channels (group c16) of a tile
// sits in slot c16*16 + ((tile + 4*(c16/2)) & 15); lane l of a wave reads slot(l/16, l%16).  The reads, of which there
// are several per write, meet no bank conflicts this way (a rotation by 4*c16 favoured the 4-byte writes instead:
// 28x28x128 N=32 scaled 14.5 -> 14.2 us, 56x56x64 N=256 scaled 84.9 -> 83.5).
__device__ inline int lds_slot(int c16, int tile) { return c16 * 16 + ((tile + 4 * (c16 >> 1)) & 15); }

struct LdsPlaneSink {
    int8_t* base;
    __device__ inline void put(int plane, uint32_t bytes) const {
        *reinterpret_cast<uint32_t*>(base + plane * kPlaneBytes) = bytes;
    }
};

// Workgroups are dealt to the eight XCDs (each with its own L2) in turn.  kByTiles: an XCD runs all filter blocks of consecutive tile
// blocks, which share their patches, the patches' overlaps and the cache lines of channels-last outputs that two filter blocks
// write.  kByFilters: consecutive tile blocks of as few filter blocks as possible, so that a filter block's operand planes enter
// one or two L2s instead of all eight.  (What it takes is worked out on the host: a division by gridDim.x, which is itself a load,
// stood before a workgroup's first request and cost a 19 us kernel half a microsecond.)
enum WorkgroupOrder { kLaunchOrder, kByTiles, kByFilters };
struct GridOrder {
    int across;            // gridDim.x
    uint32_t each, rest;   // workgroups per XCD, rounded down, and what is left; each = 0: launch order
    uint32_t deep;         // gridDim.y, 0: by filters
    FastDiv by_inner;      // by what lies together: filter blocks, or tile blocks
    __device__ inline GridOrder(uint32_t o_across, uint32_t o_each, uint32_t o_mul, uint32_t o_small)
        : across((int)o_across), each(o_each), rest(o_small & 7), deep(o_small >> 8), by_inner{o_mul, (o_small >> 3) & 31} {}
    inline GridOrder(dim3 grid, WorkgroupOrder order)
        : across((int)grid.x), each(order == kLaunchOrder || grid.y == 1 ? 0 : grid.x * grid.y >> 3), rest(grid.x * grid.y & 7),
          deep(order == kByTiles ? grid.y : 0), by_inner(make_fast_div(order == kByTiles ? grid.y : grid.x)) {}
    __device__ inline void place(int& bx, int& by) const {
        int tile_block = blockIdx.x, filter_block = blockIdx.y;
        if (each != 0) {
            const uint32_t launch = blockIdx.y * (uint32_t)across + blockIdx.x, xcd = launch & 7;
            const uint32_t at = xcd * each + min(xcd, rest) + (launch >> 3);
            const uint32_t outer = fast_div(at, by_inner), inner = at - outer * (deep ? deep : (uint32_t)across);
            tile_block = (int)(deep ? outer : inner);
            // An XCD deals its workgroups to four shader engines in turn: a multiple of four filter blocks is turned by one from tile
            // block to tile block, or one engine would get every last, perhaps half-empty one (16 -> 201 at 105x105, N = 4, scaled,
            // int8 out, 49.2 -> 44.7 us; 84 layers of four filter blocks 1 %).
            const uint32_t turned = inner + ((deep & 3) == 0 ? outer & 3 : 0);
            filter_block = (int)(deep ? (turned >= deep ? turned - deep : turned) : outer);
        }
        bx = tile_block;
        by = filter_block;
    }
};
// By tiles, except where the operand planes are more than 3 MB (an L2 has 4) and than twice the activations, or than these where
// the filters come out even, eight or sixteen full blocks (`filters` in each): an XCD's share is the same everywhere then.  us,
// launch order / by filters / by tiles: 32 -> 145 filters at 92x92, N = 39, both sides scaled, 225 / 247 / 192; 48 -> 128 at 56x84, N = 59,
// scaled, channel-major, 88.4 / 72.6 / 70.2; 234 -> 65 at 57x9, N = 26, scaled, 20.8 / 20.9 / 18.0; 29 -> 432 at 49x12, N = 177, scaled,
// 72.6 / 86.0 / 75.8; 176 -> 448 at 9x8, N = 28, lossless, int8 out, 14.8 / 13.0 / 14.6; 240 -> 443 at 9x9, N = 16, lossless, 18.6 / 16.7 /
// 18.3.  1300 drawn layers of two and more filter blocks: 0.3 % behind the best order on average and 9 at worst (launch order
// alone 2.9 and 26, by filters 3.0 and 28, by tiles 0.35 and 12, launch order or, from five filter blocks on, by filters 2.6 and 26).
// 512 filters and planes of 1 .. 1.5, 1.5 .. 2, 2 .. 3 times the activations: by filters 0.965, 1.00 and 0.96 of the time by tiles.
inline WorkgroupOrder workgroup_order(const Problem& p, int mode, int filters) {
    const long long pixels = (long long)p.N * p.H * p.W, planes = (long long)p.K * num_filter_planes(mode);
    const bool even = p.K % (8 * filters) == 0;
    return planes * p.CB * kCBlock > 3000000 && planes > (even ? 1 : 2) * pixels ? kByFilters : kByTiles;
}
// as leading arguments (see WG_GEOMETRY_PARAMS, after which they fill what is loaded ahead)
#define WG_ORDER_PARAMS uint32_t o_across, uint32_t o_each, uint32_t o_mul, uint32_t o_small
#define WG_ORDER(o) (uint32_t)(o).across, (o).each, (o).by_inner.mul, (o).rest | (o).by_inner.shift << 3 | (o).deep << 8
#define WG_TAKE_ORDER GridOrder(o_across, o_each, o_mul, o_small)

// compile-time loop: f(std::integral_constant<int, 0>{}), ..., f(<N-1>)
template <class F, int... Is>
__device__ inline void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ inline void static_for(F&& f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// The optional int8 epilogue: v = (y + round) >> shift clamped to [lo, 127].
__device__ inline int requantise(int y, const Int8Epilogue& q) {
    return min(max((y + q.round) >> q.shift, q.lo), 127);
}
__device__ inline v4i requantise(v4i y, const Int8Epilogue& q) {
    y = (y + q.round) >> q.shift;
    const v4i lo = {q.lo, q.lo, q.lo, q.lo}, hi = {127, 127, 127, 127};
    return __builtin_elementwise_min(__builtin_elementwise_max(y, lo), hi);
}
__device__ inline uint32_t pack_bytes(v4i v) {
    return __builtin_amdgcn_perm((uint32_t)v[1], (uint32_t)v[0], 0x0c0c0400u) | __builtin_amdgcn_perm((uint32_t)v[3], (uint32_t)v[2], 0x04000c0cu);
}
// An output, or a sum for the next kernel, written through the L2 (device scope).  Left in the L2s, what a kernel wrote is written back when it
// ends (128 -> 128 at 28x28, N = 32: all of its 100,352 lines, written through none), and its end waits for that; written through, it is under way as
// soon as it is stored.  us, plain / through, outputs in rotation: that layer, scaled, 13.3 / 12.2 (with the requantisation that reads it 16.8 / 16.0),
// F(2x2) 15.5 / 14.6; 64 -> 64 at 56x56, N = 32, scaled 17.2 / 15.3, N = 8, direct 5.4 / 4.9; both scaled 256 -> 256 at 14x14, N = 64 26.4 / 23.9; partial
// sums of 512 -> 512 at 14x14, N = 1, scaled, both kernels 15.2 / 13.5.  (Non-temporal stores: as fast by themselves, but what reads the outputs
// next is slower by as much or more.)  Which outputs: write_through.h.  int8 outputs, a fourth of the bytes in parts of lines, gain in the limb-pair
// kernel (64 -> 64 at 56x56, N = 8 7.9 / 7.6) and first layers (3 -> 64 at 224x224, N = 16 39.7 / 37.4), and are level or behind elsewhere (0.98 - 1.03); so
// are the requantisation's (1.00 - 1.03) and channels-last copies (1.02 - 1.10).
// The compiler's own stores, not assembly: it keeps what overwrites a 16-byte store's data two wait states behind it (gfx950), which it does not
// do for a store that it cannot see.
template <class T>
__device__ inline void write_out(T* at, T v) {
    static_assert(sizeof(T) == 16 || sizeof(T) == 4, "dwords");
    if constexpr (sizeof(T) == 16) {
        typedef uint32_t v4u __attribute__((ext_vector_type(4)));
        __builtin_amdgcn_global_store_b128((v4u __attribute__((address_space(1)))*)at, __builtin_bit_cast(v4u, v), "agent");
    } else {
        __hip_atomic_store((T __attribute__((address_space(1)))*)at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}
template <bool THROUGH, class T>
__device__ inline void write_as(T* at, T v) {
    if constexpr (THROUGH) write_out(at, v); else *at = v;
}
// What a kernel writes: int32, requantised int8, int32 written through the L2, or, limb-pair kernel, its channels' part of the sums (kOutSums).  Which
// of the first and the third is chosen on the host, so that a kernel has one of them (with both, and a branch, small layers took 1 % longer).
constexpr int kOutInt32 = 0, kOutInt8 = 1, kOutThrough = 2, kOutSums = 3;

// Patch loads of the role-specialised kernels go through a buffer descriptor over the activation
// tensor: a load whose offset lies beyond the tensor returns zero, so a pixel outside the image
// (pad 1, ragged tiles) is an offset that can never be in range instead of a select per pixel and
// channel block.  Offsets of rows and columns outside the image are kOutsideOffset; they are
// combined with a saturating addition, so that any sum with an outside part stays at or above
// 2^31, more than the tensor can hold (the host checks N*C*H*W < 2^31).
constexpr uint32_t kOutsideOffset = 0x80000000u;
constexpr int kRawBufferWord3 = 0x00020000;   // untyped 32-bit data, as for every raw buffer on this target
__device__ inline __amdgpu_buffer_rsrc_t activation_buffer(const int8_t* x, const Problem& p) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(x), 0, p.N * p.H * p.W * p.C, kRawBufferWord3);
}

// A 1 KB filter fragment, 16 bytes per lane: `base` is the same for the whole wave, `at` a constant, `lane16` = 16 x lane.  As a
// buffer load it takes its address from scalar registers and one vector register; with 64-bit addresses every fourth fragment
// cost two vector instructions and a pair of registers.
__device__ inline v4i buffer_fragment(__amdgpu_buffer_rsrc_t from, uint32_t lane16, int at) {
    return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(from, lane16, at, 0));
}
__device__ inline v4i load_fragment(const int8_t* base, uint32_t lane16, int at) {
    return buffer_fragment(__builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(base), 0, 0x7fffffff, kRawBufferWord3), lane16, at);
}
// Most instructions of the product loops and of the transform have eight bytes: whether they begin at multiples of eight or four
// behind them decides 2 - 3 % of a kernel's time, and any change further up shifts it.  So the place is fixed, for each kind of
// kernel where it measured best.  The streaming kernel at a multiple of eight / four behind, us: products, 64 -> 64 at 56x56, N = 256,
// lossless, 87.3 / 87.6, scaled 76.3 / 77.7 (left alone 89.4 and 77.3), with eight product waves 256 -> 256 at 56x56, N = 16, scaled, 57.7 /
// 57.0 (57.3), lossless 76.5 / 76.3 (79.2); transform, 64 -> 64, lossless, 85.0 / 82.2 (83.4), with inputs in rotation 96.3 / 93.7,
// scaled 72.4 / 74.6 (74.9).
template <bool FOUR_BEHIND>
__device__ inline void place_loop(std::integral_constant<bool, FOUR_BEHIND>) {
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (FOUR_BEHIND) asm volatile(".p2align 3\n\ts_nop 0");
    else asm volatile(".p2align 3");
    __builtin_amdgcn_sched_barrier(0);
}
// The lane's number, formed anew where it is asked for: a register that is needed once per channel block is worth more than two
// instructions there.
__device__ inline int lane_again() {
    int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(lane));
    return lane;
}

// How the four transform waves of the role-specialised kernels bring the 6x6 patches of their 16 tiles, one channel block at
// a time: wave w has tiles 4w .. 4w + 3, lane = (tile, four channels).  Every lane loads its four channels of every pixel,
// sixteen neighbouring lanes 64 bytes in a row.  (Sixteen channels of every fourth pixel per lane, nine instructions instead of
// 36, and an exchange of dwords between lanes by lane swaps or through LDS were 1-2 % and 5-15 % slower: the exchange lengthens
// the transform waves' chain.  Eight channels of every second pixel and one swap of lane rows per two pixels, as many instructions as
// here: 4 - 17 % slower.  With half of these loads left out the kernels take 3 - 9 % less: that is all a cheaper form could give.)
// Pixels are numbered down the columns, i = 6 b + a.
struct PatchLoader {
    uint32_t patch[36];   // the patch, or what is in flight of it
    uint32_t at[36];      // each pixel's offset, channel block 0; a channel block is a uniform offset on top
    __device__ inline static int tile_of(int wave, int lane) { return 4 * wave + (lane >> 4); }
    __device__ inline static int quad_of(int lane) { return lane & 15; }   // of four channels

    // tile (n, ty, tx) of this lane; one that does not exist may be any: nobody stores its outputs
    __device__ inline void enter(const Problem& p, int n, int ty, int tx, int lane) {
        const int h0 = 4 * ty - 1, w0 = 4 * tx - 1;
        const uint32_t row = (uint32_t)p.W * (uint32_t)p.C, image = (uint32_t)n * (uint32_t)p.H * row + (uint32_t)(4 * quad_of(lane));
        uint32_t row_off[6], col_off[6];
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            row_off[a] = (unsigned)(h0 + a) < (unsigned)p.H ? image + (uint32_t)(h0 + a) * row : kOutsideOffset;
            col_off[a] = (unsigned)(w0 + a) < (unsigned)p.W ? (uint32_t)(w0 + a) * (uint32_t)p.C : kOutsideOffset;
        }
#pragma unroll
        for (int i = 0; i < 36; ++i) at[i] = __builtin_elementwise_add_sat(row_off[i % 6], col_off[i / 6]);
    }
    // To be called before block cb is asked for.  Only the last channel block of a C that is not a multiple of 64 has channels
    // beyond C (a uniform branch): there such a lane asks for the outside offset, so that it gets zeros and never touches
    // memory next to the tensor.  The table changes: enter() comes before another tile's or block's request.
    __device__ inline void drop_absent_channels(const Problem& p, int cb, int lane) {
        if ((cb + 1) * kCBlock > p.C) {
            const bool have = cb * kCBlock + 4 * quad_of(lane) < p.C;
#pragma unroll
            for (int i = 0; i < 36; ++i) at[i] = have ? at[i] : kOutsideOffset;
        }
    }
    __device__ inline void request_column(__amdgpu_buffer_rsrc_t xbuf, int cb, int b) {
#pragma unroll
        for (int i = 6 * b; i < 6 * b + 6; ++i) patch[i] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(xbuf, at[i], cb * kCBlock, 0);
    }
    __device__ inline void request(__amdgpu_buffer_rsrc_t xbuf, int cb) {
#pragma unroll
        for (int b = 0; b < 6; ++b) request_column(xbuf, cb, b);
    }
};
// transform_patch's done_with: column b of the block after the one being transformed is asked for as its registers become
// free.  A compute unit's memory path is full of filter fragments (a load instruction waits some 100 clocks to enter it), so
// a patch's loads in a row held the transform waves up longer than their arithmetic takes; spread over the column pass they
// enter beside it.  The barriers keep the compiler from collecting them in one place again.
struct NextColumns {
    PatchLoader& loader;
    __amdgpu_buffer_rsrc_t xbuf;
    int cb;
    __device__ inline void operator()(int b) const {
        __builtin_amdgcn_sched_barrier(0);
        loader.request_column(xbuf, cb, b);
        __builtin_amdgcn_sched_barrier(0);
    }
};

// What remains to be done to a loaded patch before transform_patch<Bytes>.  Pixels outside the image arrived as
// zero bytes: for signed int8 that is x = 0 like any other byte; for uint8 they have to become the zero point, which
// one three-input OR per pixel does (row and column terms that are zero inside the image).  (Channels beyond C meet zero filters, whatever they hold.)
template <class ENC>
struct PatchBias;
template <>
struct PatchBias<SignedInt8> {
    __device__ inline void enter(const Problem&, int, int, const SignedInt8) {}
    using Bytes = StoredInt8;
    __device__ inline void apply(uint32_t (&)[36]) const {}
};
template <>
struct PatchBias<ZeroPointU8> {
    using Bytes = BiasedBytes;
    uint32_t outside;      // bit a: patch row a lies outside the image, bit 6 + b: column b (one register while it waits)
    uint32_t zero_bytes;
    __device__ inline void enter(const Problem& p, int ty, int tx, const ZeroPointU8 enc) {
        outside = 0;
        zero_bytes = enc.zero_bytes;
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            outside |= (unsigned)(4 * ty - 1 + a) < (unsigned)p.H ? 0u : 1u << a;
            outside |= (unsigned)(4 * tx - 1 + a) < (unsigned)p.W ? 0u : 64u << a;
        }
    }
    __device__ inline void apply(uint32_t (&patch)[36]) const {
        uint32_t row[6], col[6], o = outside;
        asm volatile("" : "+v"(o));   // the terms are formed here, not ahead of the channel-block loop (36 registers)
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            row[a] = (uint32_t)((int)(o << (31 - a)) >> 31) & zero_bytes;
            col[a] = (uint32_t)((int)(o << (25 - a)) >> 31) & zero_bytes;
        }
#pragma unroll
        for (int i = 0; i < 36; ++i) patch[i] |= row[i % 6] | col[i / 6];
    }
};

// Row rule of A^T on (m0, m1, m2, m3, conj(m3), m5) with m0,m1,m2,m5 real:
//   z0 = m0+m1+m2+2Re m3, z1 = m1-m2-2Im m3, z2 = m1+m2-2Re m3, z3 = m1-m2+2Im m3+m5
template <class V>
__device__ inline void at_rule(V m0, V m1, V m2, V m3r, V m3i, V m5, V z[4]) {
    const V s = m1 + m2, d = m1 - m2;
    z[0] = m0 + s + 2 * m3r;
    z[1] = d - 2 * m3i;
    z[2] = s - 2 * m3r;
    z[3] = d + 2 * m3i + m5;
}

// A finished row of M is reduced by the row rule and enters the 16 outputs with the
// column-rule coefficients of A^T.  Real rows 0,1,2,5 (ROW = 0..3; entries m0,m1,m2,m5 real
// at positions 0..3, complex m3 at position 4): row 0 -> y0; rows 1, 2 -> (+,+,+,+), (+,-,+,-);
// row 5 -> y3.  The complex row 3 (ROW = 4; e0,e1,e2,e5 at positions 0..3, e3 = M[3][3] and
// e4 = M[3][4] at 4, 5; row 4 of M is its conjugate): y0 += 2Re z, y1 -= 2Im z, y2 -= 2Re z,
// y3 += 2Im z.
// Rows come in the order 0, 1, 2 and row 5 before row 3.  FRESH: no outputs yet (rows 0..2: from any of them; rows 5 and 3:
// from each other), so that nothing is cleared first and nothing added to zero.
template <int ROW, bool FRESH, class V>
__device__ inline void finish_row(const V (&er)[6], const V (&ei)[6], V (&Y)[16]) {
    if constexpr (ROW < 4) {
        V z[4];
        at_rule(er[0], er[1], er[2], er[4], ei[4], er[3], z);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (ROW == 0) Y[j] = FRESH ? z[j] : Y[j] + z[j];
            if constexpr (FRESH) {
                if constexpr (ROW == 1) Y[8 + j] = z[j];
                if constexpr (ROW == 2) {
                    const V d = Y[8 + j] - z[j];
                    Y[8 + j] += z[j];
                    Y[j] += Y[8 + j];
                    Y[4 + j] = d;
                    Y[12 + j] = d;
                }
            } else {
                if constexpr (ROW == 1) { Y[j] += z[j]; Y[4 + j] += z[j]; Y[8 + j] += z[j]; Y[12 + j] += z[j]; }
                if constexpr (ROW == 2) { Y[j] += z[j]; Y[4 + j] -= z[j]; Y[8 + j] += z[j]; Y[12 + j] -= z[j]; }
            }
            if constexpr (ROW == 3) Y[12 + j] = FRESH ? z[j] : Y[12 + j] + z[j];
        }
    } else {
        const V sr = er[4] + er[5], si = ei[4] + ei[5], dr = er[4] - er[5], di = ei[4] - ei[5];
        const V ar = er[1] + er[2], ai = ei[1] + ei[2], br = er[1] - er[2], bi = ei[1] - ei[2];
        V zr[4], zi[4];
        zr[0] = er[0] + ar + sr;   zi[0] = ei[0] + ai + si;
        zr[1] = br - di;           zi[1] = bi + dr;            // (e1-e2) + i (e3-e4)
        zr[2] = ar - sr;           zi[2] = ai - si;
        zr[3] = br + di + er[3];   zi[3] = bi - dr + ei[3];    // (e1-e2) - i (e3-e4) + e5
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const V r = 2 * zr[j], i = 2 * zi[j];
            Y[j] = FRESH ? r : Y[j] + r;
            Y[4 + j] = FRESH ? -i : Y[4 + j] - i;
            Y[8 + j] = FRESH ? -r : Y[8 + j] - r;
            Y[12 + j] += i;
        }
    }
}

}  // namespace wg
