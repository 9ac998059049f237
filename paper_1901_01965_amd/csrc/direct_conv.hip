// Direct evaluation of the 3x3 stride-1 pad-1 convolution, the method with 144
// multiplications per 4x4 output tile and channel pair that Section 3.4 compares
// against:  y[n,k,h,w] = sum_{c,a,b} x[n,c,h+a-1,w+b-1] g[k,c,a,b].
// Serves as the on-device cross-check and the direct baseline.  Where scratch memory (or the layout) allows, the
// matrix product over linear pixels in direct_gemm.hip runs; this file has what is left for calls without scratch memory
// and for rows too long for that kernel's LDS: channels-last tensors with
// K % 4 == 0 and a 16-byte aligned output on the matrix cores by patches (operands are staged with 16-byte loads when
// C % 16 == 0 and the pointers allow it, else byte by byte), everything else in the plain kernel; and the requantisation kernels.
#include "wg_internal.h"

namespace wg {
namespace {

// One thread per (pixel, filter), lanes along K.  Channels-last inputs whose C is a
// multiple of 4 use the packed 4 x int8 dot product.
template <int LAYOUT>
__global__ __launch_bounds__(256) void direct_conv_kernel(const int8_t* __restrict__ x,
                                                          const int8_t* __restrict__ g,
                                                          int32_t* __restrict__ y, Problem p) {
    const int k = blockIdx.y * 64 + (threadIdx.x & 63);
    const long long pix = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const long long npix = (long long)p.N * p.H * p.W;
    if (k >= p.K || pix >= npix) return;
    const int w = (int)(pix % p.W), h = (int)((pix / p.W) % p.H), n = (int)(pix / ((long long)p.W * p.H));
    int acc = 0;
    for (int a = 0; a < 3; ++a) {
        const int hh = h + a - 1;
        if (hh < 0 || hh >= p.H) continue;
        for (int b = 0; b < 3; ++b) {
            const int ww = w + b - 1;
            if (ww < 0 || ww >= p.W) continue;
            if (LAYOUT == WG_NHWC) {
                const int8_t* xp = x + (((size_t)n * p.H + hh) * p.W + ww) * p.C;
                const int8_t* gp = g + ((size_t)k * 9 + a * 3 + b) * p.C;
                int c = 0;
                if (p.C % 4 == 0)
                    for (; c < p.C; c += 4)
                        acc = __builtin_amdgcn_sdot4(*reinterpret_cast<const int*>(xp + c),
                                                     *reinterpret_cast<const int*>(gp + c), acc, false);
                for (; c < p.C; ++c) acc += (int)xp[c] * (int)gp[c];
            } else {
                const size_t plane = (size_t)p.H * p.W;
                const int8_t* xp = x + (size_t)n * p.C * plane + (size_t)hh * p.W + ww;
                const int8_t* gp = g + (size_t)k * p.C * 9 + a * 3 + b;
                for (int c = 0; c < p.C; ++c) acc += (int)xp[c * plane] * (int)gp[c * 9];
            }
        }
    }
    if (LAYOUT == WG_NHWC) y[(size_t)pix * p.K + k] = acc;
    else                   y[(((size_t)n * p.K + k) * p.H + h) * p.W + w] = acc;
}

// ---- channels-last fast path on the int8 matrix cores ---------------------------------------
// Implicit GEMM: for each of the nine taps, [64 filters x 64 channels] x [64 channels x 128
// pixels].  A workgroup owns an 8 x 16 patch of output pixels of one image and 64 filters; the
// 10 x 18 input halo and the nine filter taps of one 64-channel block are staged in LDS (rows of
// 64 bytes, the 16-byte pieces of a row XOR-swizzled by (row / 4) % 4 so that the fragment reads
// of 16 consecutive rows are conflict-free); zero padding and the ragged edges of H, W, C and K
// become zeros while staging.  Filters are the rows and pixels the columns of
// v_mfma_i32_32x32x32_i8, so that a lane ends up with four consecutive filters of one pixel: 16-byte
// stores.  Wave w multiplies patch rows 2w, 2w+1 (32 pixels) by all 64 filters.
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
constexpr int kPatchRows = 8, kPatchCols = 16, kHaloCols = kPatchCols + 2;
constexpr int kHaloPixels = (kPatchRows + 2) * kHaloCols;   // 180
constexpr int kDirectFilters = 64;

__device__ inline int row_swizzle(int row) { return (row >> 2) & 3; }

// 16 bytes of channels c..c+15 at `at` (channel 0 of a pixel or filter tap): one 16-byte load when
// the tensors allow it (VEC16), else byte by byte with channels beyond C read as zero.
template <bool VEC16>
__device__ inline v4i load_channels(const int8_t* at, int c, int C) {
    if constexpr (VEC16) {
        return *reinterpret_cast<const v4i*>(at + c);
    } else {
        v4i v = {0, 0, 0, 0};
#pragma unroll
        for (int b = 0; b < 16; ++b)
            if (c + b < C) v[b >> 2] |= (int)(uint8_t)at[c + b] << (8 * (b & 3));
        return v;
    }
}

template <bool VEC16>
__global__ __launch_bounds__(256) void direct_conv_mfma_kernel(const int8_t* __restrict__ x,
                                                               const int8_t* __restrict__ g,
                                                               int32_t* __restrict__ y, Problem p, int patches_h,
                                                               int patches_w) {
    __shared__ __attribute__((aligned(16))) int8_t halo[kHaloPixels * kCBlock];
    __shared__ __attribute__((aligned(16))) int8_t taps[9 * kDirectFilters * kCBlock];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int pw = blockIdx.x % patches_w, ph = (blockIdx.x / patches_w) % patches_h;
    const int n = blockIdx.x / (patches_w * patches_h);
    const int h0 = ph * kPatchRows, w0 = pw * kPatchCols, k0 = blockIdx.y * kDirectFilters;

    v16i acc[2];
    acc[0] = (v16i){0};
    acc[1] = (v16i){0};
    // this lane's pixel (a column of the product) and its 16-byte piece of a 32-channel step
    const int pr = 2 * wave + ((lane & 31) >> 4), pc = lane & 15, piece = lane >> 5;

    for (int cb = 0; cb < p.CB; ++cb) {
        if (cb > 0) __syncthreads();   // the previous block's fragments have been read
        constexpr v4i zero = {0, 0, 0, 0};
        v4i in[3], flt[9];
#pragma unroll
        for (int it = 0; it < 3; ++it) {
            const int item = tid + 256 * it, pix = item >> 2;
            const int h = h0 - 1 + pix / kHaloCols, w = w0 - 1 + pix % kHaloCols, c = cb * kCBlock + (item & 3) * 16;
            const bool ok = pix < kHaloPixels && (unsigned)h < (unsigned)p.H && (unsigned)w < (unsigned)p.W && c < p.C;
            in[it] = zero;
            if (ok) in[it] = load_channels<VEC16>(x + (((size_t)n * p.H + h) * p.W + w) * p.C, c, p.C);
        }
#pragma unroll
        for (int it = 0; it < 9; ++it) {
            const int item = tid + 256 * it, kt = item >> 2;   // kt = filter * 9 + tap: contiguous in memory
            const int kk = k0 + kt / 9, c = cb * kCBlock + (item & 3) * 16;
            flt[it] = zero;
            if (kk < p.K && c < p.C) flt[it] = load_channels<VEC16>(g + ((size_t)k0 * 9 + kt) * p.C, c, p.C);
        }
#pragma unroll
        for (int it = 0; it < 3; ++it) {
            const int item = tid + 256 * it, pix = item >> 2;
            if (pix < kHaloPixels)
                *reinterpret_cast<v4i*>(halo + pix * kCBlock + (((item & 3) ^ row_swizzle(pix)) * 16)) = in[it];
        }
#pragma unroll
        for (int it = 0; it < 9; ++it) {
            const int item = tid + 256 * it, kt = item >> 2;
            const int row = (kt % 9) * kDirectFilters + kt / 9;   // [tap][filter]
            *reinterpret_cast<v4i*>(taps + row * kCBlock + (((item & 3) ^ row_swizzle(row)) * 16)) = flt[it];
        }
        __syncthreads();
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            const int hp = (pr + tap / 3) * kHaloCols + pc + tap % 3;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const int at = 2 * ks + piece;
                const v4i b = *reinterpret_cast<const v4i*>(halo + hp * kCBlock + ((at ^ row_swizzle(hp)) * 16));
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) {
                    const int row = tap * kDirectFilters + mt * 32 + (lane & 31);
                    const v4i a = *reinterpret_cast<const v4i*>(taps + row * kCBlock + ((at ^ row_swizzle(row)) * 16));
                    acc[mt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, acc[mt], 0, 0, 0);
                }
            }
        }
    }
    // register i of a 32x32 product: row (filter) 8 (i / 4) + 4 (lane / 32) + i % 4, column (pixel) lane % 32
    const int h = h0 + pr, w = w0 + pc;
    if (h >= p.H || w >= p.W) return;
    int32_t* out = y + (((size_t)n * p.H + h) * p.W + w) * p.K;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int kk = k0 + mt * 32 + 8 * q + 4 * piece;
            if (kk < p.K)
                *reinterpret_cast<v4i*>(out + kk) = (v4i){acc[mt][4 * q], acc[mt][4 * q + 1], acc[mt][4 * q + 2], acc[mt][4 * q + 3]};
        }
}

// v = (y + 2^(shift-1)) >> shift without the sum (y is any int32): the arithmetic shift plus the last bit shifted out.
__device__ inline v4i requant_any(v4i y, int shift, int lo) {
    if (shift > 0) y = (y >> shift) + ((y >> (shift - 1)) & 1);
    const v4i low = {lo, lo, lo, lo}, high = {127, 127, 127, 127};
    return __builtin_elementwise_min(__builtin_elementwise_max(y, low), high);
}
__device__ inline uint32_t bytes_of(v4i v) {
    return (uint32_t)(v[0] & 0xff) | ((uint32_t)(v[1] & 0xff) << 8) | ((uint32_t)(v[2] & 0xff) << 16) | ((uint32_t)v[3] << 24);
}
// Without pooling every output is a function of the input at the same place, whatever the layout: four (a thread's 16-byte
// load and 4-byte store) at a time.  Bound by memory: 5 bytes per element.
__global__ __launch_bounds__(256) void requant_kernel(const int32_t* __restrict__ y, int8_t* __restrict__ out, size_t total, int shift, int lo) {
    const size_t i = 4 * ((size_t)blockIdx.x * 256 + threadIdx.x);
    if (i + 4 <= total) {
        *reinterpret_cast<uint32_t*>(out + i) = bytes_of(requant_any(*reinterpret_cast<const v4i*>(y + i), shift, lo));
    } else {
        for (size_t j = i; j < total; ++j) out[j] = (int8_t)requant_any((v4i){y[j], 0, 0, 0}, shift, lo)[0];
    }
}
// 2x2 stride-2 maximum, four outputs per thread: four channels of a pixel (channels-last, K % 4 = 0: `run` = K, four 16-byte
// loads) or four pixels of a row (channel-major, (W / 2) % 4 = 0: two rows of eight values).  256 -> 256 outputs at 56x56,
// N = 16: 17 us with one thread and four 4-byte loads per output, 8.8 us so (55 MB).
template <int LAYOUT>
__global__ __launch_bounds__(256) void requant_pool4_kernel(const int32_t* __restrict__ y, int8_t* __restrict__ out, uint32_t quads, int run,
                                                            int W, FastDiv div_run4, FastDiv div_wo, int shift, int lo) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;   // output quad
    if (i >= quads) return;
    v4i best;
    if constexpr (LAYOUT == WG_NHWC) {
        // output pixel q of the batch: row q / Wo (two input rows each), column q % Wo
        const uint32_t q = fast_div(i, div_run4), k4 = i - q * ((uint32_t)run >> 2), row = fast_div(q, div_wo), col = q - row * ((uint32_t)W >> 1);
        const int32_t* at = y + ((size_t)(2 * row) * W + 2 * col) * run + 4 * k4;
        v4i v[4];
        v[0] = *reinterpret_cast<const v4i*>(at);
        v[1] = *reinterpret_cast<const v4i*>(at + run);
        v[2] = *reinterpret_cast<const v4i*>(at + (size_t)W * run);
        v[3] = *reinterpret_cast<const v4i*>(at + (size_t)W * run + run);
        best = __builtin_elementwise_max(__builtin_elementwise_max(v[0], v[1]), __builtin_elementwise_max(v[2], v[3]));
    } else {
        const uint32_t row = fast_div(i, div_wo), c4 = i - row * ((uint32_t)W >> 3);   // div_wo: quads per output row
        const int32_t* at = y + (size_t)(2 * row) * W + 8 * c4;
        v4i v[4];
        v[0] = *reinterpret_cast<const v4i*>(at);
        v[1] = *reinterpret_cast<const v4i*>(at + 4);
        v[2] = *reinterpret_cast<const v4i*>(at + W);
        v[3] = *reinterpret_cast<const v4i*>(at + W + 4);
        const v4i a = __builtin_elementwise_max(v[0], v[2]), b = __builtin_elementwise_max(v[1], v[3]);
        best = (v4i){max(a[0], a[1]), max(a[2], a[3]), max(b[0], b[1]), max(b[2], b[3])};
    }
    // rounding and clamp do not change the order, so the maximum comes first
    *reinterpret_cast<uint32_t*>(out + 4 * (size_t)i) = bytes_of(requant_any(best, shift, lo));
}

// ... and one output element per thread, for the shapes the kernel above does not take.
template <int LAYOUT>
__global__ __launch_bounds__(256) void requant_relu_pool_kernel(const int32_t* __restrict__ y,
                                                                int8_t* __restrict__ out, int N, int K,
                                                                int H, int W, int shift, int lo, int pool) {
    const int Ho = pool ? H / 2 : H, Wo = pool ? W / 2 : W;
    const size_t total = (size_t)N * K * Ho * Wo;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    int n, k, h, w;
    if (LAYOUT == WG_NHWC) {
        k = (int)(i % K); w = (int)((i / K) % Wo); h = (int)((i / ((size_t)K * Wo)) % Ho);
        n = (int)(i / ((size_t)K * Wo * Ho));
    } else {
        w = (int)(i % Wo); h = (int)((i / Wo) % Ho); k = (int)((i / ((size_t)Wo * Ho)) % K);
        n = (int)(i / ((size_t)Wo * Ho * K));
    }
    const int span = pool ? 2 : 1;
    const int rnd = shift > 0 ? (1 << (shift - 1)) : 0;
    int best = -129;
    for (int a = 0; a < span; ++a)
        for (int b = 0; b < span; ++b) {
            const int hh = pool ? 2 * h + a : h, ww = pool ? 2 * w + b : w;
            const int32_t v0 = LAYOUT == WG_NHWC ? y[(((size_t)n * H + hh) * W + ww) * K + k]
                                                 : y[(((size_t)n * K + k) * H + hh) * W + ww];
            int v = (int)(((long long)v0 + rnd) >> shift);
            v = v < lo ? lo : (v > 127 ? 127 : v);
            best = v > best ? v : best;
        }
    out[i] = (int8_t)best;
}

}  // namespace

namespace {

bool aligned16(const void* q) { return reinterpret_cast<uintptr_t>(q) % 16 == 0; }

// What the linear-pixel kernel (direct_gemm.hip) needs: channels-last operands with 16-byte pieces, as given or as padded
// copies.  It takes every layer whose image rows fit its LDS and whose (padded) operands fit 32-bit offsets.
struct DirectPlan {
    bool applies, copy_x, copy_w;
    Problem padded;
    size_t x_bytes, bytes;   // scratch: the copies of x and w
};
DirectPlan plan_direct(const Problem& p, int layout, bool operands_aligned) {
    DirectPlan d;
    d.copy_x = d.copy_w = layout != WG_NHWC || p.C % 16 != 0 || !operands_aligned;
    d.padded = p;
    if (d.copy_x) d.padded.C = ceil_div(p.C, 16) * 16;
    const long long limit = 0x7fffffffll, C = d.padded.C;
    d.applies = (long long)p.N * p.H * p.W * C <= limit && (long long)p.K * 9 * C <= limit && direct_gemm_applies(d.padded);
    d.x_bytes = d.applies && d.copy_x ? round_up((size_t)p.N * p.H * p.W * C, 256) : 0;
    d.bytes = d.x_bytes + (d.applies && d.copy_w ? round_up((size_t)p.K * 9 * C, 256) : 0);
    return d;
}

}  // namespace

size_t direct_conv_scratch_wanted(const Problem& p, int layout) { return plan_direct(p, layout, true).bytes; }

hipError_t launch_direct_conv(const int8_t* x, const int8_t* w, int32_t* y, const Problem& p, int layout,
                              const Scratch& scratch, hipStream_t s) {
    const bool vectors = p.C % 16 == 0 && aligned16(x) && aligned16(w), by_patches = layout == WG_NHWC && p.K % 4 == 0 && aligned16(y);
    const DirectPlan d = plan_direct(p, layout, aligned16(x) && aligned16(w));
    // (Patches are behind wherever both run, also where few workgroups make a layer's time that of one: 1x14x14, 512 -> 512 16.4 us by
    // patches, 12.2 by linear pixels; 48x7x7, 512 -> 512 21.9 / 13.2; 36x14x14, 128 -> 128 7.4 / 5.7.)
    if (d.applies && d.bytes <= scratch.bytes) {
        if (d.copy_x) {
            int8_t* const xs = static_cast<int8_t*>(scratch.p);
            int8_t* const ws = xs + d.x_bytes;
            if (hipError_t e = launch_channels_last(x, xs, p, layout, d.padded.C, 0, s)) return e;
            // [K][C][3][3] (or [K][3][3][C]) as a batch of K images of nine pixels
            if (hipError_t e = launch_channels_last(w, ws, make_problem(p.K, p.C, 3, 3, 1), layout, d.padded.C, 0, s)) return e;
            x = xs;
            w = ws;
        }
        return launch_direct_gemm(x, w, y, d.padded, layout, s);
    }
    if (by_patches) {
        const int patches_h = ceil_div(p.H, kPatchRows), patches_w = ceil_div(p.W, kPatchCols);
        dim3 grid((unsigned)(p.N * patches_h * patches_w), ceil_div(p.K, kDirectFilters));
        if (vectors)
            direct_conv_mfma_kernel<true><<<grid, 256, 0, s>>>(x, w, y, p, patches_h, patches_w);
        else
            direct_conv_mfma_kernel<false><<<grid, 256, 0, s>>>(x, w, y, p, patches_h, patches_w);
        return hipGetLastError();
    }
    const long long npix = (long long)p.N * p.H * p.W;
    dim3 grid((unsigned)((npix + 3) / 4), ceil_div(p.K, 64));
    if (layout == WG_NHWC) direct_conv_kernel<WG_NHWC><<<grid, 256, 0, s>>>(x, w, y, p);
    else                   direct_conv_kernel<WG_NCHW><<<grid, 256, 0, s>>>(x, w, y, p);
    return hipGetLastError();
}

hipError_t launch_requant_relu_pool(const int32_t* y, int8_t* out, int N, int K, int H, int W, int layout,
                                    int shift, int relu, int pool, hipStream_t s) {
    const size_t total = (size_t)N * K * (pool ? H / 2 : H) * (pool ? W / 2 : W);
    const int lo = relu ? 0 : -128;
    const bool vectors = aligned16(y) && reinterpret_cast<uintptr_t>(out) % 4 == 0;
    if (!pool && vectors) {
        requant_kernel<<<(unsigned)((total + 1023) / 1024), 256, 0, s>>>(y, out, total, shift, lo);
        return hipGetLastError();
    }
    const unsigned quads = (unsigned)(total / 4), quad_blocks = (quads + 255) / 256;
    if (pool && vectors && layout == WG_NHWC && K % 4 == 0) {
        requant_pool4_kernel<WG_NHWC><<<quad_blocks, 256, 0, s>>>(y, out, quads, K, W, make_fast_div(K / 4), make_fast_div(W / 2), shift, lo);
        return hipGetLastError();
    }
    if (pool && vectors && layout == WG_NCHW && W % 8 == 0) {
        requant_pool4_kernel<WG_NCHW><<<quad_blocks, 256, 0, s>>>(y, out, quads, 0, W, make_fast_div(1), make_fast_div(W / 8), shift, lo);
        return hipGetLastError();
    }
    const unsigned blocks = (unsigned)((total + 255) / 256);
    if (layout == WG_NHWC) requant_relu_pool_kernel<WG_NHWC><<<blocks, 256, 0, s>>>(y, out, N, K, H, W, shift, lo, pool);
    else                   requant_relu_pool_kernel<WG_NCHW><<<blocks, 256, 0, s>>>(y, out, N, K, H, W, shift, lo, pool);
    return hipGetLastError();
}

}  // namespace wg
