// F(2x2,3x3) convolution (f2x2_conv.hip has the method, the filter transform and the forms for other inputs) for
// channels-last activations with C % 4 = 0, as given or as a padded copy; any K, either output layout.
//
// What bounds it: latency.  A workgroup of 16 tiles x 64 filters waits for its patch, transforms, waits at a barrier,
// multiplies, and a layer of 128 channels has two such rounds; with the limb products in accumulators of their own (32 or 48
// of four registers) two workgroups fit a compute unit and 28x28, 128 -> 128, N = 32 (784 workgroups) took 22 us scaled and
// 31 lossless for 3 us worth of bytes.  Here the limbs are joined block by block: the low products accumulate in the channel
// sum itself, the others enter it by one shift-and-add per register, which leaves 16 sums per wave.  Lossless mode: 161
// registers, three workgroups per compute unit whose waits overlap, 16.5 us.  Scaled mode: the filter fragments come by buffer
// loads (load_fragment), whose addresses take no vector registers, so that it fits 128 and four workgroups share a compute unit:
// 15.7 -> 14.5 us, 56x56x256 N = 16 66.6 -> 63.2, 14x14x256 N = 64 23.0 -> 20.8 (with 64-bit addresses it spilled at 128 and four
// workgroups were 4-12 % slower).  Layers with few channel blocks keep 64-bit addresses and three workgroups (launch_f2_fast).  The
// reverse-scaling factors are parked in LDS at the start, the blob header is compared only before the store, and pixels outside the
// image arrive as zeros.
#include "kernel_common.h"
#include "write_through.h"

namespace wg {
namespace {

constexpr int kTiles = 16, kFilters = 64, kPlanes = 2 * kF2Entries;
constexpr int kPlanesBytes = kPlanes * kPlaneBytes;              // 32 KB; later the staged outputs
constexpr int kScalesBytes = kF2Entries * kFilters * 4;          // r | q << 8, [entry][filter]
constexpr int kLds = kPlanesBytes + kScalesBytes;
constexpr int kRow = 68;                                         // stage[output][tile][64 filters, padded]
static_assert(4 * 16 * kRow * 4 <= kPlanesBytes, "staging fits the operand planes' LDS");

// The 4x4 patch of tile (n, ty, tx), four channels per thread.  The descriptor starts one row and one pixel before the
// tensor, so that the patch's first pixel has a non-negative offset and the others follow at wave-uniform distances (the
// scalar offset of the load): a thread keeps one offset and one mask.  Pixels outside the image ask for an offset beyond any
// tensor and arrive as zeros.
struct Patch {
    uint32_t first, outside;   // outside: bit a: patch row a lies outside the image, bit 4 + b: column b
    __device__ inline static __amdgpu_buffer_rsrc_t buffer(const int8_t* x, const Problem& p) {
        const int before = (p.W + 1) * p.C;   // these sums and products fit: f2_fast_holds
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(x) - before, 0, p.N * p.H * p.W * p.C + before, kRawBufferWord3);
    }
    __device__ inline void enter(const Problem& p, int n, int ty, int tx, int c_lane) {
        first = ((uint32_t)(n * p.H + 2 * ty) * (uint32_t)p.W + (uint32_t)(2 * tx)) * (uint32_t)p.C + (uint32_t)c_lane;
        outside = 0;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            outside |= (unsigned)(2 * ty - 1 + a) < (unsigned)p.H ? 0u : 1u << a;
            outside |= (unsigned)(2 * tx - 1 + a) < (unsigned)p.W ? 0u : 16u << a;
        }
    }
    // all ones where row a / column b lies outside, from an opaque copy of the mask (the terms kept for the whole kernel
    // would be sixteen registers)
    __device__ inline void terms(uint32_t (&r)[4], uint32_t (&c)[4], uint32_t value) const {
        uint32_t o = outside;
        asm volatile("" : "+v"(o));
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            r[a] = (uint32_t)((int)(o << (31 - a)) >> 31) & value;
            c[a] = (uint32_t)((int)(o << (27 - a)) >> 31) & value;
        }
    }
    __device__ inline void request(__amdgpu_buffer_rsrc_t xbuf, const Problem& p, int cb, int c_lane, uint32_t (&u)[16]) const {
        const bool have = (cb + 1) * kCBlock <= p.C || cb * kCBlock + c_lane < p.C;
        const uint32_t base = have ? first : kOutsideOffset;
        uint32_t r[4], c[4];
        terms(r, c, kOutsideOffset);
#pragma unroll
        for (int i = 0; i < 16; ++i)
            u[i] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(xbuf, base | r[i / 4] | c[i % 4], ((i / 4) * p.W + i % 4) * p.C + cb * kCBlock, 0);
    }
    // signed int8: StoredInt8 takes the bytes as they are; uint8: pixels outside the image become the zero point
    __device__ inline void bias(uint32_t (&)[16], const SignedInt8) const {}
    __device__ inline void bias(uint32_t (&u)[16], const ZeroPointU8 enc) const {
        uint32_t r[4], c[4];
        terms(r, c, enc.zero_bytes);
#pragma unroll
        for (int i = 0; i < 16; ++i) u[i] |= r[i / 4] | c[i % 4];
    }
};

// B^T d B (rule t0 = v0 - v2, t1 = v1 + v2, t2 = v2 - v1, t3 = v1 - v3 down the columns, then along the rows) into operand
// planes 2e (high limb), 2e + 1 (low): byte limbs in scaled mode, v = 64 h + l in lossless mode (input_transform_core.h).
template <int MODE, class Bytes>
__device__ inline void transform(const uint32_t (&u)[16], const Quad bias11, int8_t* put) {
    Quad col[4][4];
    auto rule = [](Quad v0, Quad v1, Quad v2, Quad v3, Quad (&t)[4]) {
        t[0] = v0 - v2;
        t[1] = v1 + v2;
        t[2] = v2 - v1;
        t[3] = v1 - v3;
    };
#pragma unroll
    for (int b = 0; b < 4; ++b) rule(Bytes::lanes(u[b]), Bytes::lanes(u[4 + b]), Bytes::lanes(u[8 + b]), Bytes::lanes(u[12 + b]), col[b]);
    OperandSplitter<MODE == WG_SCALED ? kSplitByteLimbs : kSplitTwoLimb, LdsPlaneSink> out;
    out.sink.base = put;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        Quad t[4];
        rule(col[0][r], col[1][r], col[2][r], col[3][r], t);
        if (r == 1) t[1] = t[1] - bias11;
#pragma unroll
        for (int c = 0; c < 4; ++c) out.limbs(2 * (4 * r + c), t[c]);
    }
}

// NARROW: every channel sum fits 24 bits and its product with r <= 255 fits 32, so the reverse scaling is a 24-bit
// multiply-add and a shift (see launch_f2_fast).
template <bool NARROW>
__device__ inline int unscale(int m, uint32_t rq) {
    const int r = (int)(rq & 0xffu), q = (int)(rq >> 8);
    if constexpr (NARROW) return (__mul24(m, r) + ((1 << q) >> 1)) >> q;
    else return ReverseScale(r, q)(m);
}

// grid: (ceil(T / 16), Kp / 64), 256 threads.  Transform: thread = (tile, four channels).  Products: wave w owns filters
// 16 w .. 16 w + 15 of the 16 tiles for all 16 entries.  BUFFERS: the filter fragments come by buffer loads, and in scaled mode four
// workgroups share a compute unit.
template <int LAYOUT, int MODE, bool Q8, bool NARROW, bool BUFFERS, bool THROUGH, class ENC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MODE == WG_SCALED && BUFFERS ? 4 : 3))) void f2_fast_kernel(
    const int8_t* __restrict__ x, WG_GEOMETRY_PARAMS, WG_ORDER_PARAMS, const uint8_t* __restrict__ blob, size_t table_off,
    size_t planes_off, int32_t* __restrict__ y, Problem p, ENC enc, Int8Epilogue q8) {
    WG_TAKE_GEOMETRY(p, 1);
    using Bytes = std::conditional_t<std::is_same_v<ENC, SignedInt8>, StoredInt8, BiasedBytes>;
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int bx, by;
    WG_TAKE_ORDER.place(bx, by);
    const int tile0 = bx * kTiles, kbase = by * kFilters;
    const int a_tile = tid >> 4, cq = tid & 15;
    const __amdgpu_buffer_rsrc_t xbuf = Patch::buffer(x, p);
    Patch patch;
    {
        int n = 0, ty = 0, tx = 0;
        if (tile0 + a_tile < p.T) decode_tile(p, tile0 + a_tile, n, ty, tx);
        patch.enter(p, n, ty, tx, 4 * cq);
    }
    // Workgroups that run side by side on an XCD read the same filter fragments; each starts at a channel block of its own
    // (the integer sums do not depend on the order) so that they do not all ask for the same lines at the same time.
    int cb = bx % p.CB;
    uint32_t u[16];
    patch.request(xbuf, p, cb, 4 * cq, u);
    const BlobHeaderWords header = read_blob_header(blob);
    constexpr int NBP = MODE == WG_LOSSLESS ? 2 : 1;         // filter planes per entry
    constexpr int NP = NBP * kF2Entries;
    // a wave-uniform base and a lane offset: the fragments' addresses take no vector registers
    const int8_t* const b_wave = reinterpret_cast<const int8_t*>(blob + planes_off) +
                                 filter_plane_offset(0, 0, kbase + __builtin_amdgcn_readfirstlane(wave) * 16, 0, p.Kp, NP);
    const uint32_t b_lane = (uint32_t)lane * 16u;
    const size_t b_block_stride = (size_t)(p.Kp >> 4) * NP * kFilterFragBytes;
    uint32_t* const scales = reinterpret_cast<uint32_t*>(lds + kPlanesBytes);
    if constexpr (MODE == WG_SCALED) {   // this wave's factors, for itself: entry lane / 4 of filters lane % 4 + 4 i
        int2 rq[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            rq[i] = *reinterpret_cast<const int2*>(
                &reinterpret_cast<const ScaleEntry*>(blob + table_off)[(size_t)(kbase + wave * 16 + (lane & 3) + 4 * i) * kF2Entries + (lane >> 2)].r);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            scales[(lane >> 2) * kFilters + wave * 16 + (lane & 3) + 4 * i] = (uint32_t)rq[i].x | ((uint32_t)rq[i].y << 8);
    }
    int8_t* const put = lds + lds_slot(cq >> 2, a_tile) * 16 + (cq & 3) * 4;
    const int8_t* const a_lds = lds + lds_slot(lane >> 4, lane & 15) * 16;

    v4i sum[kF2Entries];
#pragma unroll
    for (int e = 0; e < kF2Entries; ++e) sum[e] = (v4i){0, 0, 0, 0};
    // Entries' filter fragments in flight (one less while an entry multiplies).  Where the fragments miss the L2 (fewer than eight
    // filter blocks, which every XCD then reads, and few workgroups to share them) a deep layer's time is their latency: lossless,
    // N = 1, 512 -> 256 at 28x28 32.4 us with two, 25.8 three, 23.3 four, 22.1 five, as many as three waves' registers hold
    // (161 of 168); 28x28x128 N = 32 18.9 / 17.7 / 18.3 / 18.3.
    constexpr int kRing = MODE == WG_LOSSLESS ? 5 : 4;
    for (int step = 0; step < p.CB; ++step) {
        const int8_t* const b_cb = b_wave + cb * b_block_stride;
        v4i bf[kRing][NBP];
        auto request_b = [&](auto E) {
#pragma unroll
            for (int i = 0; i < NBP; ++i) {
                constexpr int first = NBP * E * kFilterFragBytes;
                if constexpr (BUFFERS) bf[E % kRing][i] = load_fragment(b_cb, b_lane, first + i * kFilterFragBytes);
                else                   bf[E % kRing][i] = *reinterpret_cast<const v4i*>(b_cb + first + i * kFilterFragBytes + b_lane);
            }
        };
        if (step > 0) __syncthreads();   // the previous block's operand planes have been consumed
        patch.bias(u, enc);
        const Quad bias16 = Bytes::bias11(enc);   // of the 6x6 transform: 16 * bias; here it leaves 4 * bias
        transform<MODE, Bytes>(u, Quad{bias16.a >> (short)2, bias16.b >> (short)2}, put);
        __builtin_amdgcn_sched_barrier(0);   // the transform's registers are dead before the fragments take theirs
        static_for<kRing - 1>([&](auto E) { request_b(E); });
        cb = cb + 1 == p.CB ? 0 : cb + 1;
        if (step + 1 < p.CB) patch.request(xbuf, p, cb, 4 * cq, u);   // travels while this block multiplies
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();    // the operand planes are complete; what was requested stays in flight
        v4i af[2][2];
        auto request_a = [&](auto E) {
            af[E & 1][0] = *reinterpret_cast<const v4i*>(a_lds + (2 * E) * kPlaneBytes);
            af[E & 1][1] = *reinterpret_cast<const v4i*>(a_lds + (2 * E + 1) * kPlaneBytes);
        };
        __builtin_amdgcn_sched_barrier(0);
        request_a(std::integral_constant<int, 0>{});
        v4i high[2], mid[2];   // of the current and the previous entry
        static_for<kF2Entries + 1>([&](auto E) {
            constexpr int e = E;
            constexpr v4i zero = {0, 0, 0, 0};
            if constexpr (e < kF2Entries) {
                if constexpr (e + kRing - 1 < kF2Entries) request_b(std::integral_constant<int, e + kRing - 1>{});
                if constexpr (e + 1 < kF2Entries) request_a(std::integral_constant<int, e + 1>{});
                const v4i ah = af[e & 1][0], al = af[e & 1][1];
                if constexpr (MODE == WG_LOSSLESS) {
                    const v4i bh = bf[e % kRing][0], bl = bf[e % kRing][NBP - 1];
                    mid[e & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah, bl, zero, 0, 0, 0);
                    high[e & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah, bh, zero, 0, 0, 0);
                    sum[e] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al, bl, sum[e], 0, 0, 0);
                    mid[e & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al, bh, mid[e & 1], 0, 0, 0);
                } else {
                    high[e & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah, bf[e % kRing][0], zero, 0, 0, 0);
                    sum[e] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al, bf[e % kRing][0], sum[e], 0, 0, 0);
                }
            }
            if constexpr (e > 0) {
                constexpr int d = e - 1;
                if constexpr (MODE == WG_LOSSLESS) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        int t = (high[d & 1][q] << 6) + mid[d & 1][q];
                        asm("" : "+v"(t));   // keeps the two shift-and-add instructions apart
                        sum[d][q] += t << 6;
                    }
                } else {
                    sum[d] += high[d & 1] << kByteLimbShift;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    }

    // ---- undo the filter scaling; Y = A^T M A with A^T = [1 1 1 0; 0 1 -1 -1] and the rescale by 2^-2 -------------
    if constexpr (MODE == WG_SCALED) {
#pragma unroll
        for (int e = 0; e < kF2Entries; ++e) {
            const uint32_t rq = scales[e * kFilters + wave * 16 + (lane & 15)];
#pragma unroll
            for (int q = 0; q < 4; ++q) sum[e][q] = unscale<NARROW>(sum[e][q], rq);
        }
    }
    constexpr int rnd = MODE == WG_SCALED ? 2 : 0;
    v4i out[4];   // output pixel 2 i + j
    {
        v4i z[2][4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            z[0][c] = sum[c] + sum[4 + c] + sum[8 + c];
            z[1][c] = sum[4 + c] - sum[8 + c] - sum[12 + c];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            out[2 * i + 0] = (z[i][0] + z[i][1] + z[i][2] + rnd) >> 2;
            out[2 * i + 1] = (z[i][1] - z[i][2] - z[i][3] + rnd) >> 2;
        }
    }
    const bool pooled = Q8 && q8.pool != 0;   // a 2x2 output tile is one pooling window
    const int NO = pooled ? 1 : 4, Ho = pooled ? p.H >> 1 : p.H, Wo = pooled ? p.W >> 1 : p.W;
    if constexpr (Q8) {   // (requantisation is monotonic: it comes after the maximum)
        if (pooled) {
            out[0] = requantise(__builtin_elementwise_max(__builtin_elementwise_max(out[0], out[1]), __builtin_elementwise_max(out[2], out[3])), q8);
        } else {
#pragma unroll
            for (int o = 0; o < 4; ++o) out[o] = requantise(out[o], q8);
        }
    }

    // ---- staged filter-fastest, then stored in whole lines ----------------------------------------------------------
    __syncthreads();   // the operand planes are dead
    int* const stage = reinterpret_cast<int*>(lds);
#pragma unroll
    for (int o = 0; o < 4; ++o)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (o < NO) stage[(o * 16 + 4 * (lane >> 4) + q) * kRow + wave * 16 + (lane & 15)] = out[o][q];
    __syncthreads();
    if (!((header.w[0] == kF2BlobMagic) & (header.w[1] == kBlobVersion) & ((int)header.w[2] == p.K) & ((int)header.w[3] == p.Cf) &
          ((int)header.w[4] == MODE)))
        return;
    if constexpr (LAYOUT == WG_NHWC) {
        // thread: filters 4 k4 .. 4 k4 + 3 of tile `tile`, all four pixels; sixteen lanes cover the 256 bytes of a pixel
        const int k4 = tid & 15, tile = tid >> 4, kk = kbase + 4 * k4;
        int n = 0, ty = 0, tx = 0;
        if (tile0 + tile >= p.T || kk >= p.K) return;
        decode_tile(p, tile0 + tile, n, ty, tx);
        const bool quads = (p.K & 3) == 0;
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            if (o >= NO) break;
            const int h = pooled ? ty : 2 * ty + (o >> 1), w = pooled ? tx : 2 * tx + (o & 1);
            if (h >= Ho || w >= Wo) continue;
            const v4i v = *reinterpret_cast<const v4i*>(stage + (o * 16 + tile) * kRow + 4 * k4);
            const size_t at = (((size_t)n * Ho + h) * Wo + w) * p.K + kk;
            if (quads) {
                if constexpr (Q8) *reinterpret_cast<uint32_t*>(q8.out + at) = pack_bytes(v);
                else              write_as<THROUGH>(reinterpret_cast<v4i*>(y + at), v);
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (kk + c < p.K) {
                        if constexpr (Q8) q8.out[at + c] = (int8_t)v[c];
                        else              y[at + c] = v[c];
                    }
            }
        }
    } else {
        // thread: four filters of tile tid % 16: sixteen consecutive tiles of a row are 32 consecutive pixels
        const int tile = tid & 15, k4 = tid >> 4;
        int n = 0, ty = 0, tx = 0;
        if (tile0 + tile >= p.T) return;
        decode_tile(p, tile0 + tile, n, ty, tx);
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            if (o >= NO) break;
            const int h = pooled ? ty : 2 * ty + (o >> 1), w = pooled ? tx : 2 * tx + (o & 1);
            if (h >= Ho || w >= Wo) continue;
            const v4i v = *reinterpret_cast<const v4i*>(stage + (o * 16 + tile) * kRow + 4 * k4);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int kk = kbase + 4 * k4 + c;
                if (kk >= p.K) break;
                const size_t at = (((size_t)n * p.K + kk) * Ho + h) * Wo + w;
                if constexpr (Q8) q8.out[at] = (int8_t)v[c];
                else              y[at] = v[c];
            }
        }
    }
}

}  // namespace

// The whole offset of a load, from the start of its descriptor, is compared with the descriptor's 32-bit range, and the
// distance of a pixel from the patch's first one is a signed 32-bit scalar: the tensor together with the row and the pixel
// before it, and four rows and pixels, have to stay below 2^31.  Tensors of less than 2 GiB exceed that only where an image
// row is long against the whole (N = H = 1, or within a row of 2 GiB); such calls take the kernel in f2x2_conv.hip, whose
// addresses are 64-bit.
bool f2_fast_holds(const Problem& p) {
    const long long before = (long long)(p.W + 1ll) * p.C, limit = 0x7fffffffll;
    return (long long)p.N * p.H * p.W * p.C + before <= limit && 4 * before <= limit;
}

hipError_t launch_f2_fast(const int8_t* x, int is_unsigned, int zero_point, const void* blob, int32_t* y, const Problem& p, int layout,
                          int mode, const Int8Epilogue& q8, hipStream_t s) {
    const F2BlobLayout bl = f2_blob_layout(p.Kp, p.Cf, mode);
    // 64-bit addresses and three workgroups per compute unit where buffer loads cost more than they give, us with / without:
    // lossless, up to two channel blocks (56x56x64 N = 8 6.94 / 6.80, 28x28x128 N = 32 16.85 / 16.67; three blocks, 130 -> 176 at 58x30
    // N = 36, 66.2 / 66.5, eight, 512 -> 512 at 7x7 N = 8, 18.0 / 18.6); scaled, one block and no fourth workgroup for any compute unit
    // (56x56x64 N = 8 7.29 / 7.02, 64 -> 16 at 33x33 N = 22 6.72 / 6.55; with one, N = 16 11.0 / 11.7; two blocks level).
    const dim3 grid(ceil_div(p.T, kTiles), p.Kp / kFilters);
    const bool buffers = mode == WG_LOSSLESS ? p.CB > 2 : p.CB > 1 || (long long)grid.x * grid.y > 3LL * compute_units();
    auto launch = [&](auto L, auto M, auto Q, auto N, auto B, const auto& enc) -> hipError_t {
        using ENC = std::decay_t<decltype(enc)>;
        const GridOrder order(grid, grid.y >= 8 ? kByFilters : kLaunchOrder);   // (with fewer filter blocks the launch order is as fast)
        auto run = [&](auto THROUGH) {
            f2_fast_kernel<L, M, Q, N, B, THROUGH, ENC><<<grid, 256, kLds, s>>>(x, WG_GEOMETRY(p), WG_ORDER(order), static_cast<const uint8_t*>(blob),
                                                                                bl.table_off, bl.planes_off, y, p, enc, q8);
            return hipGetLastError();
        };
        if constexpr (!Q && L == WG_NHWC)
            if (f2_through(p, y)) return run(std::true_type{});   // (see write_out; a branch in the kernel cost small layers 2 - 5 %)
        return run(std::false_type{});
    };
    auto go = [&](auto L, auto M, auto Q, auto N, const auto& enc) {
        return buffers ? launch(L, M, Q, N, std::true_type{}, enc) : launch(L, M, Q, N, std::false_type{}, enc);
    };
    // a channel sum is at most C * 127 * (4 * 128, or 4 * 255 with a zero point)
    const long long most = (long long)p.Cf * 127 * 4 * (is_unsigned ? 255 : 128);
    const bool narrow = most < (1 << 23) && most * 255 + 64 < (1ll << 31);
    using std::integral_constant;
    auto form = [&](auto L, auto Q, const auto& enc) {
        if (mode == WG_LOSSLESS) return go(L, integral_constant<int, WG_LOSSLESS>{}, Q, std::false_type{}, enc);
        return narrow ? go(L, integral_constant<int, WG_SCALED>{}, Q, std::true_type{}, enc)
                      : go(L, integral_constant<int, WG_SCALED>{}, Q, std::false_type{}, enc);
    };
    constexpr integral_constant<int, WG_NHWC> nhwc{};
    constexpr integral_constant<int, WG_NCHW> nchw{};
    if (is_unsigned) {
        const ZeroPointU8 zero = make_zero_point(zero_point);   // int32 outputs only
        return layout == WG_NHWC ? form(nhwc, std::false_type{}, zero) : form(nchw, std::false_type{}, zero);
    }
    if (q8.out != nullptr) return layout == WG_NHWC ? form(nhwc, std::true_type{}, SignedInt8{}) : form(nchw, std::true_type{}, SignedInt8{});
    return layout == WG_NHWC ? form(nhwc, std::false_type{}, SignedInt8{}) : form(nchw, std::false_type{}, SignedInt8{});
}

}  // namespace wg
