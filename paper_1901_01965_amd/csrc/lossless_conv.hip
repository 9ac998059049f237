// The whole hot path in one kernel, lossless mode, for channels-last activations whose channel
// count is a multiple of four, and for channel-major ones.
//
// A 12-bit Winograd-domain filter value W = 256 Wh + Wl (byte limbs) enters the matrix cores as TWO
// ROWS of the first operand: a fragment is 8 filters x (Wh, Wl) x 64 channels.  The second operand
// is one limb plane of the transformed activations of 16 tiles (B^T d B, Section 3.3-3.4, D = 256 Dh +
// Dl).  One v_mfma_i32_16x16x64_i8 then leaves, in each lane, the products Wh*Dx and Wl*Dx of two
// filters with one tile: all limbs of a product meet in one lane, so
//   W * D = 2^16 WhDh + 2^8 (WlDh + WhDl) + WlDl
// is three shift-and-add instructions per value and no data crosses lanes for it.
//
// Workgroup: 16 tiles x 32 filters, 512 threads = 8 waves, two per SIMD: a single wave issues a
// vector instruction every five to six clocks, two waves on a SIMD keep their own pace, so eight
// waves nearly double the vector rate of the transform and of the joins.
//   Transform phase: thread = (tile, four channels, half of the rows of B^T d B): waves w and w + 4 share
//   four tiles; one forms rows 0, 1, 2 of the transformed tile, the other row 5 and the complex row 3
//   (the column pass splits the same way, so only the unpacking is done twice).  Every thread writes
//   36 four-byte pieces of operand planes: LDS takes one write instruction per four clocks whatever
//   its width, so narrower writes from more threads would cost more than they save.  Raw patches travel
//   global -> LDS in 16-byte pieces through the buffer descriptor of the activation tensor, so pixels
//   outside the image (pad 1, ragged tiles) and tiles beyond the last one arrive as zeros.
//   Product phase: wave = (filter group of 8) x (half of the 26 free entries of Section 3.4: the 16
//   real ones cost two matrix-core instructions each, the 10 complex ones eight, 56 per half).  Each
//   finished row of M is reduced by the output transform A^T M A at once, so a wave ends with partial
//   outputs of 2 filters x 1 tile per lane.
//   Store: both halves are staged in LDS filter-fastest (in an area of their own, so no wave waits for
//   the others before staging), added, shifted and stored as whole 128-byte lines (16 bytes per lane) -
//   partial-line stores from the lanes' own two filters measured twice as slow.
// Several channel blocks: the output transform is linear, so every block's rows of M are reduced
// into the same 16 outputs.
// Small grids (in_quarters): 16 filters per workgroup, a wave = filter group of 8 x a quarter of the entries, 28 matrix-core
// instructions on average instead of 56.  Such layers of several channel blocks run here, too (lossless_pair_takes).
#include <atomic>

#include "kernel_common.h"
#include "pair_products.h"
#include "roles_conv.h"
#include "write_through.h"

namespace wg {
namespace {

using namespace pairs;

#ifdef WG_TIMESTAMPS
// Development aid (never compiled into the library): per-wave cycle counts at the phase boundaries.
__device__ unsigned long long* g_stamps = nullptr;
#define WG_STAMP(i)                                                                                        \
    do {                                                                                                   \
        if (g_stamps != nullptr && (threadIdx.x & 63) == 0)                                                \
            g_stamps[((blockIdx.y * gridDim.x + blockIdx.x) * 8 + (threadIdx.x >> 6)) * 8 + (i)] = __builtin_amdgcn_s_memtime(); \
    } while (0)
#else
#define WG_STAMP(i)
#endif

constexpr int kWaves = 8;
constexpr int kBlockFilters = 4 * kPairFilters;         // 32 filters per workgroup
constexpr int kActPlanes = 72;                          // byte-limb planes: real p: 2p, 2p+1; complex j: 32+4j + {Re h, Re l, Im h, Im l}
constexpr int kPlanesBytes = kActPlanes * kPlaneBytes;  // 72 KB
constexpr int kRawPixel = 4 * kCBlock;                  // raw patches of four tiles (waves w and w + 4): [pixel 0..35][tile][64 channels]
constexpr int kRawQuad = 36 * kRawPixel + 16;           // 9 KB: nine 1 KB transfers; the quads' dwords of a pixel fall into different banks
// output staging (after the products): stage[half][output o][tile][32 filters], tile rows 36 dwords apart and
// outputs 16*36 + 32 dwords apart, so that the 16-byte reads of a 16-lane group (two outputs x eight filter
// quads) fall into different banks
// PARTS = 4 (16 filters per workgroup, four quarters of the entries): rows 20 dwords apart, outputs 336: a 16-lane group reads four
// outputs x four filter quads, and the writers' rows begin at every fourth bank.
template <int PARTS>
struct Stage {
    static constexpr int kFilters = 8 * kPairFilters / PARTS;   // per workgroup
    static constexpr int kRow = PARTS == 2 ? 36 : 20, kOut = 16 * kRow + (PARTS == 2 ? 32 : 16), kPart = 16 * kOut;   // dwords
    static constexpr int kBytes = PARTS * kPart * 4;
};
// LDS: [operand planes 72 KB][raw patches 36 KB, later the first part of the staged outputs][rest of the staged outputs]:
// the outputs are staged outside the operand planes, so a wave can stage its outputs while others still multiply
template <int PARTS>
constexpr int pair_lds_bytes() {
    static_assert(Stage<PARTS>::kBytes >= 4 * kRawQuad, "the staged outputs start in the raw patches' area");
    static_assert(kPlanesBytes + Stage<PARTS>::kBytes <= 160 * 1024, "LDS of one compute unit");
    return kPlanesBytes + Stage<PARTS>::kBytes;
}
constexpr int kLoadDwords = 1, kLoadDirect = 2;         // 4-byte loads into registers / 16-byte pieces straight into LDS
constexpr int kLoadPlanes = 3;                          // channel-major activations: rows of a patch, turned on the way into LDS

// ---- the input transform, four channels per thread, half of the rows per thread ---------------------
// Half of the channels are handled in the biased form u = x + 128 (StoredInt8); a constant patch maps to zero at every
// entry of B^T d B except (1,1), where the bias leaves 16 * 128 = 2048.  What lies outside the image arrived as zero bytes, i.e. x = 0
// after the XOR as well.
// The 1-D rule of B^T on a 6-vector (Section 3.4, the expansion of d' = B^T d):
//   t0 = v0 - v4, t1 = v1+v2+v3+v4, t2 = -v1+v2-v3+v4, t3 = (v4-v2) + i (v3-v1), t5 = v5 - v1.
// GROUP 0 forms rows 0, 1, 2 of the transformed tile (entries (r, 0..5) for r = 0, 1, 2: four real and one
// complex each), GROUP 1 row 5 and the complex row 3; of the column pass each group needs only its own rows.
// `tick` is called at ten places spread over the work (with std::integral_constant<int, 0..9>): the caller issues one
// global load at each, so that its requests enter the memory pipeline at the pace the pipeline takes them.
template <int GROUP, class Out, class Tick>
__device__ inline void transform_rows(const uint32_t (&u)[6][6], const Out& out, Tick&& tick) {
    Quad v[6][6];
    static_for<6>([&](auto A) {
#pragma unroll
        for (int b = 0; b < 6; ++b) v[A][b] = StoredInt8::lanes(u[A][b]);
        tick(A);
    });
    const Quad bias11 = StoredInt8::bias11(SignedInt8{});
    auto row_rule = [](const Quad (&c)[6]) { return bt_rule(c[0], c[1], c[2], c[3], c[4], c[5]); };
    auto emit_real_row = [&](int ri, const Line<Quad>& l) {
        out.real_entry(4 * ri + 0, l.t0);
        out.real_entry(4 * ri + 1, l.t1);
        out.real_entry(4 * ri + 2, l.t2);
        out.real_entry(4 * ri + 3, l.t5);
        out.complex_entry(ri, l.t3r, l.t3i);
    };
    if constexpr (GROUP == 0) {
        Quad r0[6], r1[6], r2[6];   // rows 0, 1, 2 of d' = B^T d, by column
#pragma unroll
        for (int b = 0; b < 6; ++b) {
            const Quad s13 = v[1][b] + v[3][b], s24 = v[2][b] + v[4][b];
            r0[b] = v[0][b] - v[4][b];
            r1[b] = s24 + s13;
            r2[b] = s24 - s13;
        }
        tick(std::integral_constant<int, 6>{});
        emit_real_row(0, row_rule(r0));
        tick(std::integral_constant<int, 7>{});
        Line<Quad> l1 = row_rule(r1);
        l1.t1 = l1.t1 - bias11;
        emit_real_row(1, l1);
        tick(std::integral_constant<int, 8>{});
        emit_real_row(2, row_rule(r2));
        tick(std::integral_constant<int, 9>{});
    } else {
        Quad r5[6], ra_[6], rb_[6];   // row 5, and row 3 = ra + i rb
#pragma unroll
        for (int b = 0; b < 6; ++b) {
            r5[b] = v[5][b] - v[1][b];
            ra_[b] = v[4][b] - v[2][b];
            rb_[b] = v[3][b] - v[1][b];
        }
        tick(std::integral_constant<int, 6>{});
        emit_real_row(3, row_rule(r5));
        tick(std::integral_constant<int, 7>{});
        // the rule acts on the real and the imaginary part of row 3 separately; entries (3,3) and (3,4) mix them
        const Line<Quad> ra = row_rule(ra_), rb = row_rule(rb_);
        out.complex_entry(4, ra.t0, rb.t0);
        out.complex_entry(5, ra.t1, rb.t1);
        out.complex_entry(6, ra.t2, rb.t2);
        tick(std::integral_constant<int, 8>{});
        out.complex_entry(7, ra.t5, rb.t5);
        out.complex_entry(8, ra.t3r - rb.t3i, rb.t3r + ra.t3i);
        out.complex_entry(9, ra.t3r + rb.t3i, rb.t3r - ra.t3i);
        tick(std::integral_constant<int, 9>{});
    }
}

// Offset (relative to x) of patch pixel `pixel` = 6a + b of tile (n, ty, tx), channel c; what does not
// exist (pixel >= 36, rows and columns outside the image, no tile) gets an offset no buffer can hold.
__device__ inline uint32_t pixel_offset(const Problem& p, bool tile_exists, int n, int ty, int tx, int pixel, int c) {
    const int a = (pixel * 43) >> 8, b = pixel - 6 * a;   // pixel / 6 for pixel < 48
    const int h = 4 * ty - 1 + a, w = 4 * tx - 1 + b;
    const bool inside = tile_exists && pixel < 36 && (unsigned)h < (unsigned)p.H && (unsigned)w < (unsigned)p.W;
    return inside ? (uint32_t)(((n * p.H + h) * p.W + w) * p.C + c) : kOutsideOffset;
}

// 16 bytes per lane from the buffer straight into LDS: lane l's piece lands at lds_dst + 16 l (lds_dst uniform).
__device__ inline void buffer_to_lds_16(__amdgpu_buffer_rsrc_t buffer, int8_t* lds_dst, uint32_t voffset, int soffset) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(buffer, (__attribute__((address_space(3))) int8_t*)lds_dst, 16, voffset, soffset, 0, 0);
}

// The raw patches of 16 tiles from channel-major activations.  A lane takes one row of one tile's patch in four channels: six
// bytes of each, with one 8-byte load at any address, so that the lanes of sixteen tiles side by side read 68 bytes in a row;
// twelve v_perm turn them into six pixels of four channels, whose dwords go where the direct transfers put theirs.  A
// workgroup's 6 x 16 rows and channel quads are three per thread.  (Without it such a layer is copied to channels-last first, a
// launch of its own: 16 -> 16 channels at 16x16 9.9 -> 7.6 us, 100 -> 75 at 37x53, N = 4, 15.4 -> 12.6.)
struct __attribute__((packed)) PackedPair {   // an 8-byte load at any address
    uint64_t v;
};
struct PlanePatch {
    static constexpr int kRows = 3;   // per thread
    int8_t* to[kRows];      // this lane's place in the raw area
    int from[kRows];        // offset of its row's first pixel in its first channel; -1 at most before the tensor
    uint32_t low[kRows], high[kRows];   // pixels 0 .. 3 and 4, 5 of the row that lie inside the image
    uint64_t row[kRows][4];             // the row in four channels, in flight
    __device__ inline static int quad_of(int wave, int i, int lane) { return 4 * ((wave * kRows + i) / 6) + (lane >> 4); }   // of four channels
    __device__ inline void enter(const Problem& p, int8_t* lds, int tile0, int wave, int lane) {
        const int tile = lane & 15, t = tile0 + tile;
        int n = 0, ty = 0, tx = 0;   // a tile that does not exist may be any: nobody stores its outputs
        if (t < p.T) decode_tile(p, t, n, ty, tx);
        const int w0 = 4 * tx - 1;
        uint32_t inside[2] = {0, 0};
#pragma unroll
        for (int b = 0; b < 6; ++b) inside[b >> 2] |= (unsigned)(w0 + b) < (unsigned)p.W ? 0xffu << (8 * (b & 3)) : 0u;
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            const int a = (wave * kRows + i) % 6, cq = quad_of(wave, i, lane), h = 4 * ty - 1 + a;
            const bool have = (unsigned)h < (unsigned)p.H;
            from[i] = ((n * p.C + min(4 * cq, p.C - 1)) * p.H + min(max(h, 0), p.H - 1)) * p.W + w0;
            low[i] = have ? inside[0] : 0u;
            high[i] = have ? inside[1] : 0u;
            to[i] = lds + kPlanesBytes + (tile >> 2) * kRawQuad + (6 * a) * kRawPixel + (tile & 3) * kCBlock + 4 * cq;
        }
    }
    // Rows of channels beyond C repeat the last channel (they meet zero filters); the first and the last row of the tensor are
    // read up to seven bytes later or earlier and shifted into place.
    __device__ inline void request(const int8_t* __restrict__ x, const Problem& p, int cb, int wave, int lane) {
        const int plane = p.H * p.W, last = p.N * p.C * plane - 8;   // >= 0: see lossless_pair_conv_choice
        int at[kRows][4];
        bool moved = false;
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            const int c0 = min(4 * quad_of(wave, i, lane), p.C - 1), c = cb * kCBlock + 4 * quad_of(wave, i, lane);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                at[i][j] = from[i] + (min(c + j, p.C - 1) - c0) * plane;
                moved |= at[i][j] < 0 || at[i][j] > last;
            }
        }
        if (__ballot(moved) == 0) {
#pragma unroll
            for (int i = 0; i < kRows; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) row[i][j] = reinterpret_cast<const PackedPair*>(x + at[i][j])->v;
        } else {
#pragma unroll
            for (int i = 0; i < kRows; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int s = min(max(at[i][j], 0), last);
                    const uint64_t v = reinterpret_cast<const PackedPair*>(x + s)->v;
                    row[i][j] = at[i][j] < s ? v << 8 : v >> (8 * (at[i][j] - s));
                }
        }
    }
    __device__ inline void put() const {
        auto perm = [](uint32_t hi, uint32_t lo, uint32_t sel) { return __builtin_amdgcn_perm(hi, lo, sel); };
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            uint32_t l[4], h[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                l[j] = (uint32_t)row[i][j] & low[i];
                h[j] = (uint32_t)(row[i][j] >> 32) & high[i];
            }
            const uint32_t l01a = perm(l[1], l[0], 0x05010400u), l01b = perm(l[1], l[0], 0x07030602u);
            const uint32_t l23a = perm(l[3], l[2], 0x05010400u), l23b = perm(l[3], l[2], 0x07030602u);
            const uint32_t h01 = perm(h[1], h[0], 0x05010400u), h23 = perm(h[3], h[2], 0x05010400u);
            const uint32_t px[6] = {perm(l23a, l01a, 0x05040100u), perm(l23a, l01a, 0x07060302u), perm(l23b, l01b, 0x05040100u),
                                    perm(l23b, l01b, 0x07060302u), perm(h23, h01, 0x05040100u), perm(h23, h01, 0x07060302u)};
#pragma unroll
            for (int b = 0; b < 6; ++b) *reinterpret_cast<uint32_t*>(to[i] + b * kRawPixel) = px[b];
        }
    }
};

// How the eight waves of a workgroup bring the raw patches of their 16 tiles: wave = quad + 4 half, four tiles per quad.
// Direct transfers (LOAD kLoadDirect): transfer i (0..8) moves pixels 4i .. 4i+3 of the four tiles: lane = 16 (pixel % 4) +
// 4 (tile % 4) + piece of 16 channels, and the hardware puts lane l's 16 bytes at (uniform destination) + 16 l, so the raw
// area is [pixel][tile % 4][64 channels].  Waves 0-3 issue transfers 0..4, waves 4-7 transfers 5..8.
// Channel-major activations (kLoadPlanes, see PlanePatch): the same raw area.
// Otherwise every thread loads the 36 pixels of its tile and four channels itself.
template <int LOAD>
struct RawPatch {
    std::conditional_t<LOAD == kLoadPlanes, PlanePatch, int> planes;
    int8_t* area;                                    // of the quad
    uint32_t raw_off[LOAD == kLoadDirect ? 5 : 1];   // this lane's piece in each of the wave's transfers
    uint32_t pixel[LOAD == kLoadDwords ? 36 : 1];    // or this thread's 36 pixels
    int first_transfer, transfers, channel;          // channel: first one of this lane's pieces
    __device__ inline void init(const Problem& p, int8_t* lds, int tile0, int quad, int half, int lane) {
        area = lds + kPlanesBytes + quad * kRawQuad;
        if constexpr (LOAD == kLoadPlanes) {
            planes.enter(p, lds, tile0, quad + 4 * half, lane);
            return;
        }
        first_transfer = half == 0 ? 0 : 5;
        transfers = half == 0 ? 5 : 4;
        const int t = tile0 + 4 * quad + (LOAD == kLoadDirect ? (lane >> 2) & 3 : lane >> 4);
        int n = 0, ty = 0, tx = 0;
        if (t < p.T) decode_tile(p, t, n, ty, tx);
        if constexpr (LOAD == kLoadDirect) {
            channel = 16 * (lane & 3);
#pragma unroll
            for (int j = 0; j < 5; ++j)
                raw_off[j] = pixel_offset(p, t < p.T, n, ty, tx, 4 * (first_transfer + j) + (lane >> 4), channel);
        } else {
            channel = 4 * (lane & 15);
            const uint32_t row = (uint32_t)p.W * (uint32_t)p.C, image = (uint32_t)n * (uint32_t)p.H * row + (uint32_t)channel;
            uint32_t row_off[6], col_off[6];
#pragma unroll
            for (int a = 0; a < 6; ++a) {
                const int h = 4 * ty - 1 + a, w = 4 * tx - 1 + a;
                row_off[a] = t < p.T && (unsigned)h < (unsigned)p.H ? image + (uint32_t)h * row : kOutsideOffset;
                col_off[a] = (unsigned)w < (unsigned)p.W ? (uint32_t)w * (uint32_t)p.C : kOutsideOffset;
            }
#pragma unroll
            for (int i = 0; i < 36; ++i) pixel[i] = __builtin_elementwise_add_sat(row_off[i / 6], col_off[i % 6]);
        }
    }
    // Channel block cb.  In the last block of a C that is not a multiple of 64 (a uniform branch) lanes whose
    // channels lie beyond C ask for the outside offset and get zeros.
    __device__ inline void request(const int8_t* __restrict__ x, const Problem& p, int cb, int wave, int lane, uint32_t (&u)[6][6]) {
        if constexpr (LOAD == kLoadPlanes) {
            planes.request(x, p, cb, wave, lane);
            return;
        }
        const __amdgpu_buffer_rsrc_t xbuf = activation_buffer(x, p);
        const bool tail = (cb + 1) * kCBlock > p.C;
        const bool have = !tail || cb * kCBlock + channel < p.C;
        if constexpr (LOAD == kLoadDirect) {
#pragma unroll
            for (int j = 0; j < 5; ++j)
                if (j < transfers)
                    buffer_to_lds_16(xbuf, area + (first_transfer + j) * 1024, have ? raw_off[j] : kOutsideOffset, cb * kCBlock);
        } else {
#pragma unroll
            for (int i = 0; i < 36; ++i)
                u[i / 6][i % 6] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(xbuf, have ? pixel[i] : kOutsideOffset, cb * kCBlock, 0);
        }
    }
    // Waits for what was requested, but not for the YOUNGER loads that were issued after it; afterwards (`again`: this is not
    // the first block) everyone is done reading the previous block's planes as well.
    template <int YOUNGER = 0>
    __device__ inline void take(bool again, int lane, uint32_t (&u)[6][6]) const {
        if constexpr (LOAD == kLoadPlanes) planes.put();   // nobody reads the previous block's raw patches any more: its planes were published since
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(YOUNGER) : "memory");
        if (LOAD != kLoadDwords || again) {
            // the raw pieces of a wave's tiles were moved by other waves
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
        }
        if constexpr (LOAD != kLoadDwords) {
#pragma unroll
            for (int i = 0; i < 36; ++i) u[i / 6][i % 6] = *reinterpret_cast<const uint32_t*>(area + i * kRawPixel + 4 * lane);
        }
    }
};

// grid (ceil(T/16), ceil(K/32)), 512 threads; PARTS = 4: ceil(K/16), for grids that leave half of the compute units idle: products
// and store take half as long there, see in_quarters.  lossless_pair_sums_kernel (OUT kOutSums): see SplitGrid.
// OUT kOutSums: the workgroup takes `blocks` channel blocks, those of split bz, and leaves the sum of its outputs,
// before the rescale by 2^-4, at y as int32 [split][tile block][32 filters][tile][output 4i+j][filter] (the output transform is
// linear, so these add up to the whole; sums_finish_kernel adds, rescales and stores).

// Where a workgroup works.  Not split: the grid's own numbers, all channel blocks.  Split channels: a grid of ceil(T/16) x ceil(K/32) x
// splits.  Every tile block reads all filters, so in lossless mode the splits are dealt out first and the tile blocks last, which brings more of the
// workgroups that read the same fragments to one XCD, whatever their numbers: 512 -> 512 at 28x28, N = 1, 18.0 -> 15.0 us, 592 -> 240 at
// 33x33 18.4 -> 15.3; of the time of the other order, up to ten tile blocks, 0.96 with 32 filters per workgroup (76 layers, 0.80 - 1.04), 0.99 with 16
// (192).  With more of them side by side it is level or behind (152 layers, 1.01 and 1.00; 0.93 - 1.14), as in scaled mode, whose filters
// are half as large (640 -> 128 at 48x48 19.4 -> 20.9).
struct SplitPlace {
    int tile_blocks, tile_block, filter_block, split, first, end;   // channel blocks first .. end - 1
    bool through;                                                   // the sums are written through the L2
};
struct SplitGrid {
    dim3 grid;
    uint32_t across, packed;   // tile blocks; 4 x channel blocks per split, + 1: splits are dealt out first, + 2: SplitPlace::through
    inline SplitGrid(int tile_blocks, int filter_blocks, int splits, int blocks, bool splits_first, bool through)
        : grid(splits_first ? dim3(splits, filter_blocks, tile_blocks) : dim3(tile_blocks, filter_blocks, splits)),
          across((uint32_t)tile_blocks), packed((uint32_t)blocks << 2 | (uint32_t)through << 1 | splits_first) {}
};
// as leading arguments (see WG_GEOMETRY_PARAMS: the first patch's place depends on all of them)
#define WG_SPLIT_PARAMS uint32_t s_across, uint32_t s_packed
#define WG_SPLIT(g) (g).across, (g).packed
__device__ inline SplitPlace place_split(WG_SPLIT_PARAMS) {
    const bool splits_first = s_packed & 1;
    const int blocks = s_packed >> 2, split = splits_first ? blockIdx.x : blockIdx.z, tile_block = splits_first ? blockIdx.z : blockIdx.x;
    return SplitPlace{(int)s_across, tile_block, (int)blockIdx.y, split, split * blocks, (split + 1) * blocks, (s_packed & 2) != 0};
}

// (p and q8 by value: by reference the compiler formed every store's conditions anew, 45 comparisons instead of 19 behind the last
// barrier with int8 outputs: 64 -> 64 at 56x56, N = 8, 7.11 us instead of 6.99)
template <int LAYOUT, int LOAD, int OUT, int PARTS>
__device__ __forceinline__ void lossless_pair(const int8_t* __restrict__ x, const uint8_t* __restrict__ blob, size_t pairs_off,
                                              int32_t* __restrict__ y, const Problem p, const Int8Epilogue q8, const SplitPlace at) {
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    constexpr bool Q8 = OUT == kOutInt8, SPLIT = OUT == kOutSums, STREAMS = SPLIT || PARTS == 4;   // the next block's filters travel early
    const int bx = at.tile_block, by = at.filter_block, bz = at.split;
    const int cb_first = at.first, cb_end = SPLIT ? min(at.end, p.CB) : p.CB;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tile0 = bx * kTileBlock;
    const int k0 = by * Stage<PARTS>::kFilters;
    WG_STAMP(0);

    // ---- the raw patch of the first channel block: the longest wait of the kernel, requested first ----
    // Transform thread: tile 4 (wave % 4) + lane / 16, channels 4 (lane % 16) .. + 3, rows by wave / 4.
    const int quad = wave & 3, half = wave >> 2;
    // Product phase: filters 8 group .. + 7, share `part` of the entries (halves: the same split again).
    const int group = PARTS == 2 ? quad : wave & 1, part = PARTS == 2 ? half : wave >> 1;
    constexpr int kFirstShare = PARTS == 2 ? 0 : kFirstQuarter;
    auto by_share = [&](auto&& f) {   // f(share of the entries, rows this wave transforms)
        using std::integral_constant;
        if constexpr (PARTS == 2) return half == 0 ? f(integral_constant<int, 0>{}, integral_constant<int, 0>{}) : f(integral_constant<int, 1>{}, integral_constant<int, 1>{});
        else return part < 2 ? (part == 0 ? f(integral_constant<int, kFirstShare>{}, integral_constant<int, 0>{})
                                          : f(integral_constant<int, kFirstShare + 1>{}, integral_constant<int, 0>{}))
                             : (part == 2 ? f(integral_constant<int, kFirstShare + 2>{}, integral_constant<int, 1>{})
                                          : f(integral_constant<int, kFirstShare + 3>{}, integral_constant<int, 1>{}));
    };
    const int a_tile = 4 * quad + (lane >> 4), a_cq = lane & 15;
    RawPatch<LOAD> raw;
    raw.init(p, lds, tile0, quad, half, lane);
    uint32_t u[6][6];
    raw.request(x, p, cb_first, wave, lane, u);
    // the blob header: requested now, looked at after the transform, so its latency hides behind the patch's
    __builtin_amdgcn_sched_barrier(0);
    const BlobHeaderWords header = read_blob_header(blob);
    __builtin_amdgcn_sched_barrier(0);

    // ---- identities of the two phases ------------------------------------------------------------------
    OperandSplitter<kSplitByteLimbs, LdsPlaneSink> out;
    out.sink.base = lds + lds_slot(a_cq >> 2, a_tile) * 16 + (a_cq & 3) * 4;
    WaveContext cx;
    cx.act = lds + lds_slot(lane >> 4, lane & 15) * 16;
    const int8_t* const wave_flt = reinterpret_cast<const int8_t*>(blob + pairs_off) + filter_pair_offset(0, 0, k0 + kPairFilters * (STREAMS ? __builtin_amdgcn_readfirstlane(group) : group), 0, 0, p.Kp);
    const size_t flt_block = (size_t)(p.Kp >> 3) * kPairValues * kFilterFragBytes;
    cx.flt = wave_flt + lane * 16;

    v2i Y[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) Y[i] = (v2i){0, 0};

    WG_STAMP(1);
    // the first kRing filter fragments of a block are requested at ten places spread over a transform
    static_assert(kRing == 10, "transform_rows calls its tick ten times");
    // the operand planes are complete once every wave's LDS writes have landed (and every wave has read its
    // raw patch); global requests stay in flight across the barrier
    auto published = [&] {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        WG_STAMP(3);
        __builtin_amdgcn_s_barrier();
        WG_STAMP(4);
    };
    if constexpr (STREAMS) {
        // Several blocks of few tiles are bound by what fetches the filters (147 KB per block and workgroup, from memory in a network, where
        // a compute unit takes in 10 - 16 bytes per clock): the next block's fragments are requested as this one's are used, behind its
        // patch, and travel beside its transform (452 -> 160 at 20x20, N = 4, 20.2 -> 14.3 us with the order of the grid).  The first
        // block's, too, before its patch is waited for: 512 -> 512 at 14x14, N = 1, 8.6 -> 9.3 us, other workgroups' patches then queue behind them.
        // A loop per half (the same barriers in both), so that the ring keeps its registers from block to block: one loop for both
        // copied it at the end of a block, which waits for what is in flight.
        const uint32_t lane16 = 16u * (uint32_t)lane;
        auto block_fragments = [&](int cb) {   // those of a block that is not this workgroup's arrive as zeros, without a trip to memory
            return __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(wave_flt + cb * flt_block), 0, cb < cb_end ? 0x7fffffff : 0, kRawBufferWord3);
        };
        auto blocks_of = [&](auto SHARE, auto H) -> bool {
            using Half = Products<SHARE>;
            v4i ring[kRing];
            for (int cb = cb_first; cb < cb_end; ++cb) {
                const __amdgpu_buffer_rsrc_t now = block_fragments(cb), next = block_fragments(cb + 1);
                if (cb == cb_first) {
                    raw.template take<0>(false, lane, u);
                    WG_STAMP(2);
                    transform_rows<H>(u, out, [&](auto I) {
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (I < Half::NF) ring[I] = Half::template fragment<I>(now, lane16);
                        __builtin_amdgcn_sched_barrier(0);
                    });
                    if (!blob_matches(header, p.K, p.Cf, WG_LOSSLESS)) return false;   // uniform: nobody reaches the next barrier
                } else {
                    raw.template take<(kRing < Half::NF ? kRing : Half::NF)>(true, lane, u);
                    WG_STAMP(2);
                    transform_rows<H>(u, out, [](auto) {});
                }
                published();
                if (cb + 1 < cb_end) {
                    raw.request(x, p, cb + 1, wave, lane, u);   // travels while this block's products run
                    // `take` counts the fragments below as younger than the patch: none of them may be requested ahead of it.  (Here, in
                    // the request's own basic block: behind it, it kept the products' first LDS reads back as well, 16 -> 16 at 16x16 6.48 -> 6.54 us.)
                    asm volatile("" ::: "memory");
                }
                Half::run(cx, ring, Y, [&](auto F) {
                    if constexpr (F + kRing < Half::NF) ring[F % kRing] = Half::template fragment<F + kRing>(now, lane16);
                    else ring[F % kRing] = Half::template fragment<F % kRing>(next, lane16);
                });
                WG_STAMP(5);
            }
            return true;
        };
        if (!by_share(blocks_of)) return;
    } else {
        using First = Products<0>;
        using Second = Products<1>;
        v4i ring0[kRing], ring1[kRing];
        for (int cb = 0; cb < cb_end; ++cb) {
            // This wave's share of the raw patch (or its 36 pixels) has arrived.  The filter fragments are only requested
            // now, so that at the start of the kernel, when every workgroup of the grid asks at once, the patches do not
            // share the memory system with them; the transform gives the fragments time enough to arrive.
            raw.template take<0>(cb > 0, lane, u);
            WG_STAMP(2);
            if (half == 0) transform_rows<0>(u, out, [&](auto I) { First::template prefetch_one<I>(cx, ring0); });
            else           transform_rows<1>(u, out, [&](auto I) { Second::template prefetch_one<I>(cx, ring1); });
            if (cb == 0 && !blob_matches(header, p.K, p.Cf, WG_LOSSLESS)) return;   // uniform: nobody reaches the next barrier
            published();
            if (cb + 1 < cb_end) raw.request(x, p, cb + 1, wave, lane, u);   // travels while this block's products run
            if (half == 0) First::run(cx, ring0, Y, [&](auto F) { if constexpr (F + kRing < First::NF) ring0[F % kRing] = First::template fragment<F + kRing>(cx); });
            else           Second::run(cx, ring1, Y, [&](auto F) { if constexpr (F + kRing < Second::NF) ring1[F % kRing] = Second::template fragment<F + kRing>(cx); });
            cx.flt += flt_block;
            WG_STAMP(5);
        }
    }

    // ---- stage the shares' partial outputs, add them, store whole lines ------------------------------
    // the staging area lies behind the operand planes (it begins where the raw patches were, which nobody reads
    // after the last transform), so a wave stages its outputs as soon as it has them
    int* const stage = reinterpret_cast<int*>(lds + kPlanesBytes);
    using St = Stage<PARTS>;
    {
        // lane = tile (lane & 15) x filters 8 group + 2 (lane / 16), + 1
        int* dst = stage + part * St::kPart + (lane & 15) * St::kRow + 8 * group + 2 * (lane >> 4);
#pragma unroll
        for (int o = 0; o < 16; ++o) *reinterpret_cast<v2i*>(dst + o * St::kOut) = Y[o];
    }
    if constexpr (STREAMS) {   // loads that nobody takes are still in flight
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
    } else {
        __syncthreads();
    }
    WG_STAMP(6);
    auto sixteen = [&](int o, int tile, int k4) {   // 16 x the finished outputs of filters k0 + 4 k4 .. + 3 at output o of a tile
        const int at = o * St::kOut + tile * St::kRow + 4 * k4;
        v4i sum = *reinterpret_cast<const v4i*>(stage + at);
#pragma unroll
        for (int i = 1; i < PARTS; ++i) sum += *reinterpret_cast<const v4i*>(stage + i * St::kPart + at);
        return sum;
    };
    auto staged = [&](int o, int tile, int k4) { return sixteen(o, tile, k4) >> 4; };
    auto best_of_window = [&](int pi, int pj, int tile, int k4) {   // the 2x2 maximum, then requantised (all of it is monotonic)
        const v4i a = __builtin_elementwise_max(sixteen(4 * (2 * pi) + 2 * pj, tile, k4), sixteen(4 * (2 * pi) + 2 * pj + 1, tile, k4));
        const v4i b = __builtin_elementwise_max(sixteen(4 * (2 * pi + 1) + 2 * pj, tile, k4), sixteen(4 * (2 * pi + 1) + 2 * pj + 1, tile, k4));
        return requantise(__builtin_elementwise_max(a, b) >> 4, q8);
    };
    constexpr int kQuads = St::kFilters / 4;   // of four filters
    if constexpr (LAYOUT == WG_NCHW && OUT != kOutSums) {
        // a filter's outputs lie together: sixteen consecutive tiles of an image row are 64 consecutive pixels
        const int tile = (tid >> 2) & 15, t = tile0 + tile;
        int n = 0, ty = 0, tx = 0;
        if (t < p.T) decode_tile(p, t, n, ty, tx);
        const int H = Q8 && q8.pool ? p.H >> 1 : p.H, W = Q8 && q8.pool ? p.W >> 1 : p.W;
        const size_t plane = (size_t)H * W;
        auto first = [&](auto* base, int k4, int h, int w) { return base + ((size_t)n * p.K + k0 + 4 * k4) * plane + (size_t)h * W + w; };
        if constexpr (!Q8) {
            // thread: row i, column j of a tile, half of the workgroup's groups of four filters
            const int j = tid & 3, i = (tid >> 6) & 3, h = 4 * ty + i, w = 4 * tx + j;
            if (t >= p.T || h >= H || w >= W) return;
#pragma unroll
            for (int g = 0; g < kQuads / 2; ++g) {
                const int k4 = kQuads / 2 * (tid >> 8) + g;
                const v4i v = staged(4 * i + j, tile, k4);
                int32_t* const at = first(y, k4, h, w);
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (k0 + 4 * k4 + c < p.K) write_as<OUT == kOutThrough>(at + c * plane, (int32_t)v[c]);
            }
        } else if (q8.pool) {
            // thread: one pooled pixel of a tile, four filters
            const int pj = tid & 1, pi = (tid >> 1) & 1, k4 = tid >> 6, h = 2 * ty + pi, w = 2 * tx + pj;
            if (t >= p.T || h >= H || w >= W || k4 >= kQuads) return;
            const v4i best = best_of_window(pi, pj, tile, k4);
            int8_t* const at = first(q8.out, k4, h, w);
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (k0 + 4 * k4 + c < p.K) at[c * plane] = (int8_t)best[c];
        } else {
            // thread: row i of a tile (four pixels: one dword where rows stay aligned), four filters
            const int i = tid & 3, k4 = tid >> 6, h = 4 * ty + i, w = 4 * tx;
            if (t >= p.T || h >= H || k4 >= kQuads) return;
            const bool word_store = ((W & 3) | (int)(reinterpret_cast<uintptr_t>(q8.out) & 3)) == 0;
            v4i px[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) px[j] = requantise(staged(4 * i + j, tile, k4), q8);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (k0 + 4 * k4 + c >= p.K) continue;
                int8_t* const at = first(q8.out, k4, h, w) + c * plane;
                if (word_store) {
                    *reinterpret_cast<uint32_t*>(at) = pack_bytes((v4i){px[0][c], px[1][c], px[2][c], px[3][c]});
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (w + j < W) at[j] = (int8_t)px[j][c];
                }
            }
        }
        return;
    }
    // thread: filters k0 + 4 k4 .. + 3 of output column j of tile `tile`; round r: output row r, of four (two with 16 filters, row0 ..)
    constexpr int kRows = 2 * kQuads / 4;
    const int k4 = tid & (kQuads - 1), j = (tid / kQuads) & 3, tile = (tid / (4 * kQuads)) & 15, row0 = kRows == 4 ? 0 : 2 * (tid >> 8);
    const int t = tile0 + tile, kk = k0 + 4 * k4;
    int n = 0, ty = 0, tx = 0;
    if (t < p.T) decode_tile(p, t, n, ty, tx);
    const int row = 4 * ty, col = 4 * tx + j;
    const bool live = t < p.T && col < p.W && kk < p.K;
    if constexpr (OUT == kOutSums) {
        v4i* const to = reinterpret_cast<v4i*>(y + split_sums_offset(16, bz, bx, k0 / kBlockFilters, at.tile_blocks, p.Kp)) +
                        (16 * tile + j) * (kBlockFilters / 4) + k0 % kBlockFilters / 4 + k4;
        v4i v[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) v[r] = sixteen(4 * (row0 + r) + j, tile, k4);
        if (at.through) {
#pragma unroll
            for (int r = 0; r < kRows; ++r) write_out(to + 4 * (row0 + r) * (kBlockFilters / 4), v[r]);
        } else {
#pragma unroll
            for (int r = 0; r < kRows; ++r) to[4 * (row0 + r) * (kBlockFilters / 4)] = v[r];
        }
        return;
    }
    if constexpr (!Q8) {
        int32_t* const first = y + ((size_t)(n * p.H + row) * p.W + col) * p.K + kk;
        const bool vector_store = (p.K & 3) == 0 && (reinterpret_cast<uintptr_t>(y) & 15) == 0;
        v4i v[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) v[r] = staged(4 * (row0 + r) + j, tile, k4);
        // (not through the L2: level at best, 64 -> 64 at 28x28, N = 1, 5.57 us, through 5.71)
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            if (!live || row + row0 + r >= p.H) continue;
            int32_t* at = first + (size_t)(row0 + r) * p.W * p.K;
            if (vector_store) {
                *reinterpret_cast<v4i*>(at) = v[r];
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (kk + q < p.K) at[q] = v[r][q];
            }
        }
    } else {
        // requantisation and clamp, then (a 4x4 tile holds whole 2x2 windows) the pooling maximum
        const bool word_store = (p.K & 3) == 0 && (reinterpret_cast<uintptr_t>(q8.out) & 3) == 0;
        auto put_bytes = [&](int8_t* at, v4i q) {
            if (word_store) {   // (always through: whole words of no more than two rounds of workgroups, 4 MB)
                write_out(reinterpret_cast<uint32_t*>(at), pack_bytes(q));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (kk + e < p.K) at[e] = (int8_t)q[e];
            }
        };
        if (!q8.pool) {
            v4i v[kRows];
#pragma unroll
            for (int r = 0; r < kRows; ++r) v[r] = requantise(staged(4 * (row0 + r) + j, tile, k4), q8);
#pragma unroll
            for (int r = 0; r < kRows; ++r)
                if (live && row + row0 + r < p.H) put_bytes(q8.out + ((size_t)(n * p.H + row + row0 + r) * p.W + col) * p.K + kk, v[r]);
        } else if (j < 2) {
            // thread: pooled column j (0, 1) of its tile, both pooled rows (one)
            const int Ho = p.H >> 1, Wo = p.W >> 1, ocol = 2 * tx + j;
#pragma unroll
            for (int pi = row0 / 2; pi < row0 / 2 + kRows / 2; ++pi) {
                const v4i best = best_of_window(pi, j, tile, k4);
                if (t < p.T && kk < p.K && ocol < Wo && 2 * ty + pi < Ho)
                    put_bytes(q8.out + ((size_t)(n * Ho + 2 * ty + pi) * Wo + ocol) * p.K + kk, best);
            }
        }
    }
    WG_STAMP(7);
}

template <int LAYOUT, int LOAD, int OUT, int PARTS>
__global__ __launch_bounds__(512) void lossless_pair_kernel(const int8_t* __restrict__ x, WG_GEOMETRY_PARAMS, const uint8_t* __restrict__ blob,
                                                            size_t pairs_off, int32_t* __restrict__ y, Problem p, Int8Epilogue q8) {
    WG_TAKE_GEOMETRY(p, 2);
    // grid (tile blocks, filter blocks), quarters also (1, filter blocks, tile blocks): see lossless_pair_filters_first.  (A third number that is
    // not needed costs the halves 0.5 %, 64 -> 64 at 56x56, N = 8, 7.02 us instead of 6.99.)
    const int tile_block = PARTS == 4 ? (int)(blockIdx.x + blockIdx.z) : (int)blockIdx.x;
    lossless_pair<LAYOUT, LOAD, OUT, PARTS>(x, blob, pairs_off, y, p, q8, SplitPlace{0, tile_block, (int)blockIdx.y, 0, 0, 0, false});
}
template <int LOAD, int PARTS>
__global__ __launch_bounds__(512) void lossless_pair_sums_kernel(const int8_t* __restrict__ x, WG_GEOMETRY_PARAMS, WG_SPLIT_PARAMS,
                                                                 const uint8_t* __restrict__ blob, size_t pairs_off, int32_t* __restrict__ sums, Problem p) {
    WG_TAKE_GEOMETRY(p, 2);
    lossless_pair<WG_NHWC, LOAD, kOutSums, PARTS>(x, blob, pairs_off, sums, p, Int8Epilogue{nullptr, 0, 0, 0, 0},
                                           place_split(s_across, s_packed));
}

// ---- scaled mode, split channels ---------------------------------------------------------------------
// The same eight-wave structure for layers with few tiles in scaled mode (Section 4.2), whose channel blocks are dealt to
// several workgroups: the filters are single int8 values, so a fragment is 16 filters, and the channel sums have to be
// complete before they are scaled back, so the workgroup leaves them as they are.  Wave = filter group of 16 (wave & 1) and a
// quarter of the entries (wave >> 1), 28 matrix-core instructions per channel block each:
//   quarters 0, 1: six real entries and two complex ones, quarters 2, 3: two and three.
// A complex entry multiplies with Wr and Wi only (Di Wi in accumulators of its own); every limb product keeps its
// accumulator across the channel blocks, so a block costs no vector work but the transform.  All eight to ten fragments of
// a wave and block are in flight before its transform ends.
constexpr int quarter_slots(int q) { return q < 2 ? 8 : 5; }
constexpr int quarter_entry(int q, int s) {
    if (q < 2) return s < 6 ? 6 * q + s : kRealEntries + 2 * q + s - 6;
    return s < 2 ? 12 + 2 * (q - 2) + s : kRealEntries + 4 + 3 * (q - 2) + s - 2;
}
constexpr int quarter_frag(int q, int s) {   // fragments before slot s
    int n = 0;
    for (int i = 0; i < s; ++i) n += entry_fragments(quarter_entry(q, i));
    return n;
}
constexpr int quarter_acc(int q, int s) {    // accumulators before slot s: (h, l), or Dr Wr, Im, Di Wi as (h, l) each
    int n = 0;
    for (int i = 0; i < s; ++i) n += real_entry(quarter_entry(q, i)) ? 2 : 6;
    return n;
}
template <int Q>
struct QuarterProducts {
    static constexpr int NS = quarter_slots(Q), NF = quarter_frag(Q, NS), NA = quarter_acc(Q, NS);
    static_assert(NF <= 10, "a wave's fragments are requested at the ten ticks of the transform");
    v4i w[NF], acc[NA];
    __device__ inline void clear() {
#pragma unroll
        for (int i = 0; i < NA; ++i) acc[i] = (v4i){0, 0, 0, 0};
    }
    template <int I>
    __device__ inline void prefetch_one(const int8_t* flt) {
        if constexpr (I < NF) {
            __builtin_amdgcn_sched_barrier(0);
            constexpr auto plane = [] {   // blob plane of fragment I: real entry p: p; complex entry j: 16 + 3j (Wr), + 1 (Wi)
                int s = 0;
                while (quarter_frag(Q, s + 1) <= I) ++s;
                const int e = quarter_entry(Q, s);
                return real_entry(e) ? e : kRealEntries + 3 * (e - kRealEntries) + (I - quarter_frag(Q, s));
            }();
            w[I] = *reinterpret_cast<const v4i*>(flt + plane * kFilterFragBytes);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __device__ inline void run(const int8_t* act) {
        v4i d[2][4];
        auto load = [&](auto S) {
            constexpr int e = quarter_entry(Q, S);
            static_for<2 * entry_fragments(e)>(
                [&](auto I) { d[S & 1][I] = *reinterpret_cast<const v4i*>(act + (entry_plane(e) + I) * kPlaneBytes); });
        };
        load(std::integral_constant<int, 0>{});
        static_for<NS>([&](auto S) {
            constexpr int e = quarter_entry(Q, S), f = quarter_frag(Q, S), a = quarter_acc(Q, S);
            if constexpr (S + 1 < NS) load(std::integral_constant<int, S + 1>{});
            auto mac = [&](int to, int filter, int from) {
                acc[a + to] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[f + filter], d[S & 1][from], acc[a + to], 0, 0, 0);
            };
            mac(0, 0, 0);
            mac(1, 0, 1);
            if constexpr (!real_entry(e)) {   // d = (Dr h, Dr l, Di h, Di l)
                mac(2, 0, 2);
                mac(3, 0, 3);
                mac(4, 1, 2);
                mac(5, 1, 3);
                mac(2, 1, 0);
                mac(3, 1, 1);
            }
        });
    }
    // lane = tile (lane & 15) x four filters: one 16-byte store per sum
    template <bool THROUGH>
    __device__ inline void store(v4i* to, int plane) const {
        static_for<NS>([&](auto S) {
            constexpr int e = quarter_entry(Q, S), a = quarter_acc(Q, S);
            if constexpr (real_entry(e)) {
                write_as<THROUGH>(to + e * plane, (acc[a] << kByteLimbShift) + acc[a + 1]);
            } else {
                constexpr int at = kRealEntries + 2 * (e - kRealEntries);
                write_as<THROUGH>(to + at * plane, ((acc[a] - acc[a + 4]) << kByteLimbShift) + (acc[a + 1] - acc[a + 5]));
                write_as<THROUGH>(to + (at + 1) * plane, (acc[a + 2] << kByteLimbShift) + acc[a + 3]);
            }
        });
    }
};

// grid: see SplitGrid, 512 threads; sums: int32 [split][tile block][32 filters][36][tile][filter].
template <int LOAD>
__global__ __launch_bounds__(512) void scaled_sums_kernel(const int8_t* __restrict__ x, WG_GEOMETRY_PARAMS, WG_SPLIT_PARAMS, const uint8_t* __restrict__ blob, size_t planes_off,
                                                          int32_t* __restrict__ sums, Problem p) {
    WG_TAKE_GEOMETRY(p, 2);
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const SplitPlace at = place_split(s_across, s_packed);
    const int tile0 = at.tile_block * kTileBlock, k0 = at.filter_block * kBlockFilters;
    const int cb_first = at.first, cb_end = min(at.end, p.CB);
    const int quad = wave & 3, half = wave >> 2;   // of the transform
    const int a_tile = 4 * quad + (lane >> 4), a_cq = lane & 15;
    RawPatch<LOAD> raw;
    raw.init(p, lds, tile0, quad, half, lane);
    uint32_t u[6][6];
    raw.request(x, p, cb_first, wave, lane, u);
    __builtin_amdgcn_sched_barrier(0);
    const BlobHeaderWords header = read_blob_header(blob);
    __builtin_amdgcn_sched_barrier(0);
    OperandSplitter<kSplitByteLimbs, LdsPlaneSink> out;
    out.sink.base = lds + lds_slot(a_cq >> 2, a_tile) * 16 + (a_cq & 3) * 4;
    const int8_t* const act = lds + lds_slot(lane >> 4, lane & 15) * 16;
    constexpr int NP = 46;
    const int kgroup = k0 + 16 * (wave & 1);
    const size_t flt_block = (size_t)(p.Kp >> 4) * NP * kFilterFragBytes;
    const int8_t* flt = reinterpret_cast<const int8_t*>(blob + planes_off) + filter_plane_offset(0, 0, kgroup + (lane & 15), (lane >> 4) * 16, p.Kp, NP) +
                        cb_first * flt_block;
    // one loop per quarter (the same barriers in all four), so that each is allocated registers on its own
    auto blocks_of = [&](auto Q) {
        QuarterProducts<Q> products;
        products.clear();
        for (int cb = cb_first; cb < cb_end; ++cb) {
            raw.template take<0>(cb > cb_first, lane, u);
            auto tick = [&](auto I) { products.template prefetch_one<I>(flt); };
            transform_rows<(Q < 2 ? 0 : 1)>(u, out, tick);
            if (cb == cb_first && !blob_matches(header, p.K, p.Cf, WG_SCALED)) return;   // uniform: nobody reaches the next barrier
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            if (cb + 1 < cb_end) raw.request(x, p, cb + 1, wave, lane, u);
            products.run(act);
            flt += flt_block;
        }
        constexpr int plane = kTileBlock * kBlockFilters / 4;   // in units of four sums
        v4i* const to = reinterpret_cast<v4i*>(sums + split_sums_offset(kAccPlanes, at.split, at.tile_block, at.filter_block, at.tile_blocks, p.Kp)) +
                           (lane & 15) * (kBlockFilters / 4) + 4 * (wave & 1) + (lane >> 4);
        if (at.through) products.template store<true>(to, plane); else products.template store<false>(to, plane);
    };
    switch (wave >> 1) {
        case 0: blocks_of(std::integral_constant<int, 0>{}); break;
        case 1: blocks_of(std::integral_constant<int, 1>{}); break;
        case 2: blocks_of(std::integral_constant<int, 2>{}); break;
        default: blocks_of(std::integral_constant<int, 3>{}); break;
    }
}

// (of the padding to 64 filters, a block of 32 that do not exist has nothing to do: no sums of theirs are looked at)
template <int LAYOUT, int LOAD, int OUT, int PARTS>
hipError_t launch(const int8_t* x, const uint8_t* blob, const BlobLayout& bl, int32_t* y, const Problem& p, const Int8Epilogue& q8, hipStream_t s) {
    static LdsLimitOnce lds_limit;   // per template instance
    if (hipError_t e = lds_limit.set(reinterpret_cast<const void*>(&lossless_pair_kernel<LAYOUT, LOAD, OUT, PARTS>), pair_lds_bytes<PARTS>())) return e;
    dim3 grid(ceil_div(p.T, kTileBlock), ceil_div(p.K, Stage<PARTS>::kFilters));
    if (PARTS == 4 && lossless_pair_filters_first(p)) grid = dim3(1, grid.y, grid.x);
    lossless_pair_kernel<LAYOUT, LOAD, OUT, PARTS><<<grid, 64 * kWaves, pair_lds_bytes<PARTS>(), s>>>(x, WG_GEOMETRY(p), blob, bl.pairs_off, y, p, q8);
    return hipGetLastError();
}
// Quarters of the entries and 16 filters per workgroup where their grid is still one round of the compute units: products and
// store take half as long, while the patches are loaded and transformed twice as often, on compute units that had nothing to do
// (us, halves / quarters: 16 -> 16 at 16x16, channel-major, 7.5 / 6.5; 100 -> 75 at 37x53, N = 4, channel-major, 12.3 / 10.75).  Several
// channel blocks, against the role-specialised kernel or a split that ran them before, 510 layers: 0.65 - 1.03 of the time, 0.87 on average.
bool in_quarters(const Problem& p, int splits) {
    return (long long)ceil_div(p.T, kTileBlock) * ceil_div(p.K, Stage<4>::kFilters) * splits <= compute_units();
}
// The splits' sums, which the next kernel reads from every XCD, are written through the L2 (write_out) where they are not few: 512 -> 512 at 14x14,
// N = 1 (4 and 9 MB), both kernels, scaled 15.2 us, through 13.5, lossless level; 128 -> 64 at 14x14, N = 2 (0.3 MB) 9.1, 9.4.
inline bool sums_through(const Problem& p, int mode, int splits) { return split_partial_bytes(p, mode, splits) >= sizeof(int32_t) * kThroughFewest; }
inline SplitGrid split_grid(const Problem& p, int blocks, int splits, int mode, int filters = kBlockFilters) {
    const int tile_blocks = ceil_div(p.T, kTileBlock);
    return SplitGrid(tile_blocks, ceil_div(p.K, filters), splits, blocks, mode == WG_LOSSLESS && tile_blocks <= 10, sums_through(p, mode, splits));
}

// How the patches of a tensor are read (see kLoadDwords ..).
int load_of(const int8_t* x, const Problem& p, int layout) {
    if (layout != WG_NHWC) return kLoadPlanes;
    return p.C % 16 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0 ? kLoadDirect : kLoadDwords;
}

std::atomic<int> g_lossless_variant{0};

}  // namespace

#ifdef WG_TIMESTAMPS
extern "C" int winograd_debug_set_stamps(void* dev_ptr) {
    return hipMemcpyToSymbol(HIP_SYMBOL(g_stamps), &dev_ptr, sizeof dev_ptr) == hipSuccess ? 0 : -5;
}
#endif

void set_lossless_variant(int v) { g_lossless_variant.store(v, std::memory_order_relaxed); }
int lossless_variant() { return g_lossless_variant.load(std::memory_order_relaxed); }

bool plane_patches_hold(const Problem& p) { return (long long)p.N * p.C * p.H * p.W >= 8; }   // whole 8-byte loads exist

// Workgroups go to the XCDs in turn.  With the tile blocks dealt out first and a multiple of eight of them, every XCD reads all filters of
// its few tiles' blocks; dealt out first, a multiple of eight filter blocks leaves each XCD an eighth of the filters.  (Quarters, several channel
// blocks, us, tile blocks / filter blocks first: 256 -> 512 at 9x55, N = 3, 16.2 / 12.7, 320 -> 512 at 10x17, N = 8, 18.7 / 15.3, 256 -> 256 at
// 53x12, N = 6, 13.9 / 13.1; 224 layers of 16 filter blocks and more 0.77 - 0.99, level with one channel block, with eight filter blocks 0.92 - 1.1,
// with other numbers of them up to 1.05.)
bool lossless_pair_filters_first(const Problem& p) {
    const int filter_blocks = ceil_div(p.K, Stage<4>::kFilters);
    return p.CB > 1 && filter_blocks >= 16 && filter_blocks % 8 == 0;
}

bool lossless_pair_takes(const Problem& p, bool pieces) { return in_quarters(p, 1) && (pieces || (p.CB <= 6 && p.CB * p.Kp <= 2048)); }

int lossless_pair_conv_choice(const int8_t* x, const Problem& p, int layout) {
    const int v = lossless_variant();
    const bool applies = layout == WG_NHWC ? p.C % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 4 == 0 : plane_patches_hold(p);
    if (v == 2 || !applies) return 0;
    return v == 1 ? 2 : 1;
}

hipError_t launch_lossless_pair_conv(const int8_t* x, const void* blob, int32_t* y, const Problem& p, int layout,
                                     const Int8Epilogue& q8, hipStream_t s) {
    const BlobLayout bl = blob_layout(p.Kp, p.Cf, WG_LOSSLESS);
    const uint8_t* b = static_cast<const uint8_t*>(blob);
    auto form = [&](auto LAYOUT, auto LOAD, auto PARTS) {
        if (q8.out != nullptr) return launch<LAYOUT, LOAD, kOutInt8, PARTS>(x, b, bl, y, p, q8, s);
        if constexpr (LAYOUT == WG_NCHW)
            if (pair_planes_through(p, y)) return launch<LAYOUT, LOAD, kOutThrough, PARTS>(x, b, bl, y, p, q8, s);
        return launch<LAYOUT, LOAD, kOutInt32, PARTS>(x, b, bl, y, p, q8, s);
    };
    auto go = [&](auto LAYOUT, auto LOAD) {
        return in_quarters(p, 1) ? form(LAYOUT, LOAD, std::integral_constant<int, 4>{}) : form(LAYOUT, LOAD, std::integral_constant<int, 2>{});
    };
    using std::integral_constant;
    constexpr integral_constant<int, WG_NHWC> nhwc{};
    switch (load_of(x, p, layout)) {
        case kLoadPlanes: return go(integral_constant<int, WG_NCHW>{}, integral_constant<int, kLoadPlanes>{});
        case kLoadDirect: return go(nhwc, integral_constant<int, kLoadDirect>{});
        default: return go(nhwc, integral_constant<int, kLoadDwords>{});
    }
}

hipError_t launch_lossless_pair_sums(const int8_t* x, const void* blob, int32_t* sums, const Problem& p, int layout, int blocks, int splits,
                                     hipStream_t s) {
    const BlobLayout bl = blob_layout(p.Kp, p.Cf, WG_LOSSLESS);
    auto form = [&](auto LOAD, auto PARTS) -> hipError_t {
        static LdsLimitOnce lds_limit;   // per instance
        if (hipError_t e = lds_limit.set(reinterpret_cast<const void*>(&lossless_pair_sums_kernel<LOAD, PARTS>), pair_lds_bytes<PARTS>())) return e;
        const SplitGrid grid = split_grid(p, blocks, splits, WG_LOSSLESS, Stage<PARTS>::kFilters);
        lossless_pair_sums_kernel<LOAD, PARTS><<<grid.grid, 64 * kWaves, pair_lds_bytes<PARTS>(), s>>>(
            x, WG_GEOMETRY(p), WG_SPLIT(grid), static_cast<const uint8_t*>(blob), bl.pairs_off, sums, p);
        return hipGetLastError();
    };
    auto go = [&](auto LOAD) {
        return in_quarters(p, splits) ? form(LOAD, std::integral_constant<int, 4>{}) : form(LOAD, std::integral_constant<int, 2>{});
    };
    using std::integral_constant;
    switch (load_of(x, p, layout)) {
        case kLoadPlanes: return go(integral_constant<int, kLoadPlanes>{});
        case kLoadDirect: return go(integral_constant<int, kLoadDirect>{});
        default: return go(integral_constant<int, kLoadDwords>{});
    }
}

hipError_t launch_scaled_sums(const int8_t* x, const void* blob, int32_t* sums, const Problem& p, int layout, int blocks, int splits, hipStream_t s) {
    const BlobLayout bl = blob_layout(p.Kp, p.Cf, WG_SCALED);
    const SplitGrid grid = split_grid(p, blocks, splits, WG_SCALED);
    auto go = [&](auto LOAD) -> hipError_t {
        static LdsLimitOnce lds_limit;   // per LOAD
        constexpr int lds_bytes = kPlanesBytes + 4 * kRawQuad;
        if (hipError_t e = lds_limit.set(reinterpret_cast<const void*>(&scaled_sums_kernel<LOAD>), lds_bytes)) return e;
        scaled_sums_kernel<LOAD><<<grid.grid, 64 * kWaves, lds_bytes, s>>>(x, WG_GEOMETRY(p), WG_SPLIT(grid), static_cast<const uint8_t*>(blob),
                                                                              bl.planes_off, sums, p);
        return hipGetLastError();
    };
    using std::integral_constant;
    switch (load_of(x, p, layout)) {
        case kLoadPlanes: return go(integral_constant<int, kLoadPlanes>{});
        case kLoadDirect: return go(integral_constant<int, kLoadDirect>{});
        default: return go(integral_constant<int, kLoadDwords>{});
    }
}

}  // namespace wg
