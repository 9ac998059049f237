// Second half of a convolution whose channel blocks were dealt to several workgroups (lossless_conv.hip): adds the splits
// and finishes.  Scaled mode: Winograd-domain channel sums, scaled back (Section 4.2) and transformed (Section 3.3) here;
// lossless mode: 16 x outputs.  Only layers with few tiles come here (without the split they would fill less than half the
// chip), so the kernels are bound by the latency of their reads, not by their amount: all of a thread's reads of a split are
// in flight together.
// One image, int8 out, filters out of the L2s, one kernel against both of these together: 512 -> 512 at 14x14 lossless 21.9 / 11.5 us (16
// workgroups of eight channel blocks, 128 of one), scaled 18.6 / 15.0; at 28x28 lossless 22.5 / 15.6.
#include "kernel_common.h"
#include "output_transform_core.h"
#include "roles_conv.h"

namespace wg {
namespace {

// Filters of one tile per workgroup: as many as lie together in memory (lossless mode, 64 / 32, both kernels: 512 -> 75 at 14x14, N = 4,
// channel-major, 10.5 / 10.2 us, 512 -> 512 at 14x14, N = 1, 11.07 / 10.98).
constexpr int kItems = 32;

// Sum of the splits of N vectors that lie `step` vectors apart (and a split `split` vectors from the next), up to eight splits in flight.
template <int N>
__device__ inline void add_splits(const v4i* from, size_t split, int step, int splits, v4i (&sum)[N]) {
    auto add = [&](auto FLIGHT) {
        constexpr int n = decltype(FLIGHT)::value;
        for (int s = 0; s < splits; s += n) {
            v4i part[N][n];
#pragma unroll
            for (int j = 0; j < n; ++j)
#pragma unroll
                for (int i = 0; i < N; ++i) part[i][j] = from[(size_t)min(s + j, splits - 1) * split + i * step];
#pragma unroll
            for (int j = 0; j < n; ++j)
#pragma unroll
                for (int i = 0; i < N; ++i) sum[i] += s + j < splits ? part[i][j] : (v4i){0, 0, 0, 0};
        }
    };
#pragma unroll
    for (int i = 0; i < N; ++i) sum[i] = (v4i){0, 0, 0, 0};
    if (splits <= 2)      add(std::integral_constant<int, 2>{});
    else if (splits <= 4) add(std::integral_constant<int, 4>{});
    else                  add(std::integral_constant<int, 8>{});
}

// Scaled mode.  grid: (padded tiles, ceil(K / 32)), 128 threads: 32 filters of one tile.  First 96 threads take four filters of three
// sums each, in 16-byte reads, while the other 32 bring the filters' factors (r, q) to LDS in whole lines; then a thread has one row of
// outputs (one pooled output) of one filter.
// (The kernel alone, 512 -> 512 at 14x14, N = 1, eight splits, pooled or not: 9.1 - 12.4 us with a lane per filter, four-byte reads, factors read 8
// bytes of every 16 by lanes 416 apart, and one wave in four finishing; 5.0 now.  Both kernels, 512 -> 16 at 7x14: 12.5 -> 10.4.)
constexpr int kReaders = 96;
constexpr int kFactorRow = kEntries + 1;   // of a filter in LDS: an odd number of 8-byte pairs
template <int LAYOUT, bool Q8>
__global__ __launch_bounds__(128) void split_finish_kernel(const int32_t* __restrict__ partial, WG_GEOMETRY_PARAMS, int Kp, int splits,
                                                           const uint8_t* __restrict__ blob,
                                                           size_t table_off, int32_t* __restrict__ y, Problem p, Int8Epilogue q8) {
    WG_TAKE_GEOMETRY(p, 2);
    p.Kp = Kp;
    __shared__ __attribute__((aligned(16))) int sums[kAccPlanes][kItems];
    __shared__ int2 factors[kItems * kFactorRow];
    const int tid = threadIdx.x, t = blockIdx.x, k0 = blockIdx.y * kItems;
    if (t >= p.T) return;   // (uniform)
    const int tile_blocks = (p.T + 15) / 16;
    const BlobHeaderWords header = read_blob_header(blob);
    constexpr int kOwn = kAccPlanes / (kReaders / 8);   // sums per reading thread
    static_assert(kOwn * (kReaders / 8) == kAccPlanes, "every sum has a reader");
    const int l = tid & 7, e0 = (tid >> 3) * kOwn;
    v4i m[kOwn];
    if (tid < kReaders) {
        const size_t split = split_sums_offset(kAccPlanes, 1, 0, 0, tile_blocks, p.Kp) / 4;
        const v4i* const from = reinterpret_cast<const v4i*>(partial + split_sums_offset(kAccPlanes, 0, t >> 4, k0 >> 5, tile_blocks, p.Kp) +
                                                             (t & 15) * 32 + e0 * (16 * 32)) + l;
        add_splits<kOwn>(from, split, 16 * 32 / 4, splits, m);
    } else {
        const ScaleEntry* const table = reinterpret_cast<const ScaleEntry*>(blob + table_off) + (size_t)k0 * kEntries;
        const int i0 = tid - kReaders;
#pragma unroll
        for (int i = 0; i < kEntries; ++i) {
            const int at = 32 * i + i0, k = at / kEntries;   // kEntries x 32 entries
            const v4i entry = *reinterpret_cast<const v4i*>(table + at);
            factors[k * kFactorRow + at - k * kEntries] = make_int2(entry[2], entry[3]);
        }
    }
    __syncthreads();
    if (tid < kReaders) {
#pragma unroll
        for (int i = 0; i < kOwn; ++i) {
            const int e = e0 + i, entry = e < kRealEntries ? e : kRealEntries + (e - kRealEntries) / 2;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int2 rq = factors[(4 * l + c) * kFactorRow + entry];
                m[i][c] = ReverseScale(rq.x, rq.y)(m[i][c]);   // Section 4.2
            }
            *reinterpret_cast<v4i*>(&sums[e][4 * l]) = m[i];
        }
    }
    __syncthreads();
    const int kk = tid & (kItems - 1), row = tid / kItems, k = k0 + kk;
    if (k >= p.K || !blob_matches(header, p.K, p.Cf, WG_SCALED)) return;
    int re[16], cr[10], ci[10];
#pragma unroll
    for (int e = 0; e < 16; ++e) re[e] = sums[e][kk];
#pragma unroll
    for (int j = 0; j < 10; ++j) {
        cr[j] = sums[16 + 2 * j][kk];
        ci[j] = sums[17 + 2 * j][kk];
    }
    int out[4][4];   // out[j][i]: output row i, column j
    output_tile(re, cr, ci, out);

    int n, ty, tx;
    decode_tile(p, t, n, ty, tx);
    constexpr int rnd = 8;
    auto at = [&](int h, int w, int H, int W) {
        return LAYOUT == WG_NHWC ? (((size_t)n * H + h) * W + w) * p.K + k : (((size_t)n * p.K + k) * H + h) * W + w;
    };
    auto mine = [&](int a, int b, int c, int d) { return row < 2 ? (row == 0 ? a : b) : (row == 2 ? c : d); };
    if (Q8 && q8.pool) {   // window (row / 2, row % 2)
        auto best = [&](int i, int j) { return max(max(out[2 * j][2 * i], out[2 * j + 1][2 * i]), max(out[2 * j][2 * i + 1], out[2 * j + 1][2 * i + 1])); };
        const int h = 2 * ty + (row >> 1), w = 2 * tx + (row & 1), v = mine(best(0, 0), best(0, 1), best(1, 0), best(1, 1));
        if (h < p.H >> 1 && w < p.W >> 1) q8.out[at(h, w, p.H >> 1, p.W >> 1)] = (int8_t)requantise((v + rnd) >> 4, q8);
        return;
    }
    const int h = 4 * ty + row;
    if (h >= p.H) return;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int w = 4 * tx + j, v = (mine(out[j][0], out[j][1], out[j][2], out[j][3]) + rnd) >> 4;
        if (w >= p.W) continue;
        if constexpr (Q8) q8.out[at(h, w, p.H, p.W)] = (int8_t)requantise(v, q8);
        else              y[at(h, w, p.H, p.W)] = v;
    }
}

// The same for launch_lossless_pair_sums, whose workgroups leave 16 x outputs: adds the splits, rescales and stores.
// Thread: four filters of one output of a tile, up to eight splits' reads in flight together; with pooling the four outputs of a
// window lie in lanes eight apart, which take their maximum across them.
// (The kernel alone, 512 -> 512 at 14x14, N = 1, eight splits, pooled: 5.2 us with a thread per window that read its four outputs, and four
// splits of each, one after another; 3.1 now.  One image through the VGG-16-shaped network, eight such layers, 170.1 -> 163.9.)
// grid: (padded tiles, ceil(K / 32)), 128 threads: 8 x four filters, 16 outputs.
template <int LAYOUT, bool Q8>
__global__ __launch_bounds__(128) void sums_finish_kernel(const int32_t* __restrict__ sums, WG_GEOMETRY_PARAMS, int Kp, int splits,
                                                          const uint8_t* __restrict__ blob, int32_t* __restrict__ y, Problem p, Int8Epilogue q8) {
    WG_TAKE_GEOMETRY(p, 2);
    p.Kp = Kp;
    const int t = blockIdx.x, kk = kItems * blockIdx.y + 4 * (threadIdx.x & 7), i = threadIdx.x >> 3;
    const bool pool = Q8 && q8.pool;
    if (t >= p.T) return;   // (uniform)
    const BlobHeaderWords header = read_blob_header(blob);
    const int o = pool ? (i & 8) + (i & 4) / 2 + (i & 2) * 2 + (i & 1) : i;   // pooling: window i / 4, output i % 4 of it
    const int tile_blocks = (p.T + 15) / 16;
    const size_t split = split_sums_offset(16, 1, 0, 0, tile_blocks, p.Kp) / 4;   // v4i per split
    const v4i* const from = reinterpret_cast<const v4i*>(sums + split_sums_offset(16, 0, t >> 4, kk >> 5, tile_blocks, p.Kp) +
                                                         (t & 15) * (16 * 32) + o * 32 + (kk & 31));
    v4i total[1];
    add_splits<1>(from, split, 0, splits, total);
    v4i v = total[0] >> 4;
    int n, ty, tx;
    decode_tile(p, t, n, ty, tx);
    int h = 4 * ty + (o >> 2), w = 4 * tx + (o & 3), H = p.H, W = p.W;
    if (pool) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            v[c] = max(v[c], __shfl_xor(v[c], 8));
            v[c] = max(v[c], __shfl_xor(v[c], 16));
        }
        h >>= 1; w >>= 1; H >>= 1; W >>= 1;
        if (threadIdx.x & 24) return;   // one of the four stores
    }
    if constexpr (Q8) v = requantise(v, q8);
    if (!blob_matches(header, p.K, p.Cf, WG_LOSSLESS) || h >= H || w >= W) return;
    const size_t pixel = ((size_t)n * H + h) * W + w, plane = (size_t)H * W;
    if (LAYOUT == WG_NHWC && (p.K & 3) == 0) {
        if (kk >= p.K) return;
        if constexpr (Q8) *reinterpret_cast<uint32_t*>(q8.out + pixel * p.K + kk) = pack_bytes(v);
        else              *reinterpret_cast<v4i*>(y + pixel * p.K + kk) = v;
        return;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if (kk + c >= p.K) break;
        const size_t at = LAYOUT == WG_NHWC ? pixel * p.K + kk + c : ((size_t)n * p.K + kk + c) * plane + (pixel - (size_t)n * plane);
        if constexpr (Q8) q8.out[at] = (int8_t)v[c];
        else              y[at] = v[c];
    }
}

}  // namespace

// A workgroup per tile, and none for the rest of the last block of 16: a multiple of 8 keeps a tile's workgroups on one XCD, whose
// L2 then joins the lines of their outputs (288 -> 368 at 38x38, N = 1, lossless, channel-major, 22.4 us; with a grid of the tiles alone 23.6).
static int padded_tiles(const Problem& p) { return 16 * ceil_div(p.T, 16); }

hipError_t launch_sums_finish(const RolesCall& c, const int32_t* sums, int splits, hipStream_t s) {
    const dim3 grid(padded_tiles(c.p), ceil_div(c.p.K, kItems));
    auto go = [&](auto kernel) {
        kernel<<<grid, 128, 0, s>>>(sums, WG_GEOMETRY(c.p), c.p.Kp, splits, c.blob, c.y, c.p, c.q8);
        return hipGetLastError();
    };
    if (c.layout == WG_NHWC) return c.q8.out ? go(&sums_finish_kernel<WG_NHWC, true>) : go(&sums_finish_kernel<WG_NHWC, false>);
    return c.q8.out ? go(&sums_finish_kernel<WG_NCHW, true>) : go(&sums_finish_kernel<WG_NCHW, false>);
}

hipError_t launch_split_finish(const RolesCall& c, const int32_t* partial, int splits, hipStream_t s) {
    const dim3 grid(padded_tiles(c.p), ceil_div(c.p.K, kItems));
    auto go = [&](auto kernel) {
        kernel<<<grid, 128, 0, s>>>(partial, WG_GEOMETRY(c.p), c.p.Kp, splits, c.blob, c.bl.table_off, c.y, c.p, c.q8);
        return hipGetLastError();
    };
    if (c.layout == WG_NHWC) return c.q8.out ? go(&split_finish_kernel<WG_NHWC, true>) : go(&split_finish_kernel<WG_NHWC, false>);
    return c.q8.out ? go(&split_finish_kernel<WG_NCHW, true>) : go(&split_finish_kernel<WG_NCHW, false>);
}

}  // namespace wg
