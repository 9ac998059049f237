// Direct convolution on the int8 matrix cores as an implicit matrix product over linear pixels: y[pixel][k] = sum over nine
// taps and C channels.  Activations channels-last with C % 16 = 0 (as given, or as a padded copy), filters [K][9][C].
//
// What bounds it: with operands in LDS a wave reads (A + B) fragments of 1 KB for A x B matrix instructions of 32 clocks, and
// LDS delivers 128 B per clock to a compute unit.  A wave tile of 64 filters x 128 pixels asks for 6 KB per eight
// instructions, 96 B per clock for four SIMDs; the 32 x 64 tile per wave of the patch kernel (direct_conv.hip) asks for
// 192 B per clock, which is what held that kernel at 1260 TOPS on 256 -> 256 channels at 56x56, N = 16 (47 us).
//
// Workgroup: P consecutive pixels of the batch (in memory order, so only the last workgroup has idle columns, whatever the
// image size) x F filters.  LDS holds, per block of 64 channels, the pixel rows p0 - W - 1 .. p0 + P + W (a tap is a row
// offset of (a - 1) W + (b - 1)) and the taps of one filter row; both double-buffered and filled by 16-byte transfers from
// memory straight into LDS that run during the products.  A tap that falls outside the image reads a row of zeros: one
// select per fragment address.  A stage is one filter row of one channel block: 48 matrix instructions per wave, one barrier.
#include <algorithm>

#include "kernel_common.h"

namespace wg {
namespace {

typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kZeroRow = 64;   // bytes of zeros at the start of LDS

// 16-byte pieces of a 64-byte LDS row are XOR-swizzled so that the fragment reads of 16 consecutive rows fall into
// different banks; the swizzle is applied on the global side of the transfers.
__device__ inline int piece_at(int row, int slot) { return slot ^ ((row >> 2) & 3); }

__device__ inline void to_lds_16(__amdgpu_buffer_rsrc_t buffer, int8_t* lds_dst, uint32_t voffset) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(buffer, (__attribute__((address_space(3))) int8_t*)lds_dst, 16, voffset, 0, 0, 0);
}

// Pixel rows a workgroup keeps, rounded up to whole 1 KB transfers.
__host__ __device__ inline int halo_rows(int P, int W) { return (P + 2 * W + 2 + 15) / 16 * 16; }

// WF x WP waves; a wave multiplies 64 filters x 32 PG pixels.  F = 64 WF, P = 32 PG WP.
// grid: (ceil(pixels / P), ceil(K / F)), 64 WF WP threads.
template <int LAYOUT, int WF, int WP, int PG>
__global__ __launch_bounds__(64 * WF * WP) void direct_gemm_kernel(const int8_t* __restrict__ x, const int8_t* __restrict__ w,
                                                                   int N, int C, int H, int W, int K, int32_t* __restrict__ y, Problem p) {
    p.N = N; p.C = C; p.H = H; p.W = W; p.K = K;   // (in registers when a wave starts)
    constexpr int F = 64 * WF, P = 32 * PG * WP, T = 64 * WF * WP;
    constexpr int kTapBytes = 3 * F * kCBlock;
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wf = wave % WF, wp = wave / WF;
    const int pixels = p.N * p.H * p.W, p0 = blockIdx.x * P, k0 = blockIdx.y * F;
    const int rows = halo_rows(P, p.W), halo_bytes = rows * kCBlock;
    int8_t* const taps = lds + kZeroRow;                    // two buffers
    int8_t* const halo = taps + 2 * kTapBytes;              // two buffers
    const __amdgpu_buffer_rsrc_t xbuf = activation_buffer(x, p);
    const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(w), 0, p.K * 9 * p.C, kRawBufferWord3);
    if (tid < kZeroRow / 4) reinterpret_cast<int*>(lds)[tid] = 0;

    // pieces beyond C, pixels outside the batch and filters beyond K ask for an offset no buffer holds, and arrive as zeros
    auto request_halo = [&](int cb, int8_t* dst) {
        const int total = rows * 4;
        for (int base = wave * 64; base < total; base += T) {
            const int at = base + lane, row = at >> 2, c = cb * kCBlock + 16 * piece_at(row, at & 3);
            const int pixel = p0 - p.W - 1 + row;
            const bool have = at < total && (unsigned)pixel < (unsigned)pixels && c < p.C;
            to_lds_16(xbuf, dst + base * 16, have ? (uint32_t)pixel * (uint32_t)p.C + (uint32_t)c : kOutsideOffset);
        }
    };
    auto request_taps = [&](int cb, int a, int8_t* dst) {
        // LDS row = 3 taps x F filters: [tap b][filter]
#pragma unroll
        for (int i = 0; i < (3 * F * 4 + T - 1) / T; ++i) {
            const int base = i * T + wave * 64, at = base + lane, row = at >> 2, b = row / F, k = k0 + row % F;
            if (base >= 3 * F * 4) break;
            const int c = cb * kCBlock + 16 * piece_at(row, at & 3);
            const bool have = k < p.K && c < p.C;
            to_lds_16(wbuf, dst + base * 16, have ? ((uint32_t)k * 9 + 3 * a + b) * (uint32_t)p.C + (uint32_t)c : kOutsideOffset);
        }
    };

    // this lane's pixels (one per group): which of the nine taps lie inside the image
    int valid[PG];
#pragma unroll
    for (int g = 0; g < PG; ++g) {
        const int pixel = p0 + (wp * PG + g) * 32 + (lane & 31);
        const int h = (pixel / p.W) % p.H, wcol = pixel % p.W;
        int m = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b)
                m |= ((unsigned)(h + a - 1) < (unsigned)p.H && (unsigned)(wcol + b - 1) < (unsigned)p.W) << (3 * a + b);
        valid[g] = m;
    }
    v16i acc[2][PG];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int g = 0; g < PG; ++g) acc[f][g] = (v16i){0};

    request_halo(0, halo);
    request_taps(0, 0, taps);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    const int upper = lane >> 5;   // which 16 of a step's 32 channels
    const int stages = 3 * p.CB;
    int a = 0, cb = 0;
    for (int s = 0; s < stages; ++s) {
        const int next_a = a == 2 ? 0 : a + 1, next_cb = a == 2 ? cb + 1 : cb;
        if (s + 1 < stages) request_taps(next_cb, next_a, taps + ((s + 1) & 1) * kTapBytes);
        if (a == 0 && cb + 1 < p.CB) request_halo(cb + 1, halo + ((cb + 1) & 1) * halo_bytes);
        const int8_t* const tap_rows = taps + (s & 1) * kTapBytes;
        const int8_t* const pixel_rows = halo + (cb & 1) * halo_bytes;
        // six steps of 32 channels (tap b, half ks); a step's fragments are read while the step before multiplies
        v4i A[2][2], B[2][PG];
        auto read = [&](auto S) {
            constexpr int b = S / 2, ks = S % 2;
            const int piece = 2 * ks + upper;
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const int row = b * F + wf * 64 + f * 32 + (lane & 31);
                A[S & 1][f] = *reinterpret_cast<const v4i*>(tap_rows + row * kCBlock + 16 * piece_at(row, piece));
            }
#pragma unroll
            for (int g = 0; g < PG; ++g) {
                const int row = (wp * PG + g) * 32 + (lane & 31) + a * p.W + b;
                const int8_t* at = pixel_rows + row * kCBlock + 16 * piece_at(row, piece);
                B[S & 1][g] = *reinterpret_cast<const v4i*>((valid[g] >> (3 * a + b)) & 1 ? at : lds);
            }
        };
        read(std::integral_constant<int, 0>{});
        static_for<6>([&](auto S) {
            if constexpr (S + 1 < 6) read(std::integral_constant<int, S + 1>{});
#pragma unroll
            for (int g = 0; g < PG; ++g)
#pragma unroll
                for (int f = 0; f < 2; ++f) acc[f][g] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[S & 1][f], B[S & 1][g], acc[f][g], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        });
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        a = next_a;
        cb = next_cb;
    }

    // register i of a 32x32 product: row (filter) 8 (i / 4) + 4 (lane / 32) + i % 4, column (pixel) lane % 32
#pragma unroll
    for (int g = 0; g < PG; ++g) {
        const int pixel = p0 + (wp * PG + g) * 32 + (lane & 31);
        if (pixel >= pixels) continue;
        const int plane = p.H * p.W, n = pixel / plane;
        int32_t* const out = LAYOUT == WG_NHWC ? y + (size_t)pixel * p.K : y + (size_t)n * p.K * plane + (pixel - n * plane);
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int k = k0 + wf * 64 + f * 32 + 8 * q + 4 * upper;
                const v4i v = {acc[f][g][4 * q], acc[f][g][4 * q + 1], acc[f][g][4 * q + 2], acc[f][g][4 * q + 3]};
                if (LAYOUT == WG_NHWC && (p.K & 3) == 0) {
                    if (k < p.K) *reinterpret_cast<v4i*>(out + k) = v;
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (k + c < p.K) out[LAYOUT == WG_NHWC ? (size_t)(k + c) : (size_t)(k + c) * plane] = v[c];
                }
            }
    }
}

struct Form {
    int F, P, threads;
};
constexpr Form kForms[] = {{128, 512, 512}, {64, 512, 512}, {64, 256, 512}, {64, 128, 256}};
constexpr int kLdsMost = 160 * 1024;
int lds_bytes(const Form& f, const Problem& p) { return kZeroRow + 2 * 3 * f.F * kCBlock + 2 * halo_rows(f.P, p.W) * kCBlock; }

// The form with the least estimated time: rounds of the compute units times what a workgroup takes, its matrix instructions
// at the share of the peak that its wave tile reaches (128 x 512: 96 B of LDS reads per clock; the others 128 B and more).
int choose_form(const Problem& p) {
    const long long pixels = (long long)p.N * p.H * p.W;
    int best = -1;
    double best_cost = 0;
    for (int i = 0; i < 4; ++i) {
        const Form& f = kForms[i];
        if (lds_bytes(f, p) > kLdsMost) continue;
        const long long groups = (pixels + f.P - 1) / f.P * ceil_div(p.K, f.F);
        const int per_cu = std::max(1, kLdsMost / lds_bytes(f, p));
        constexpr double clocks_per_product[4] = {1.0, 1.3, 1.6, 1.6};   // relative
        const double cost = (double)((groups + compute_units() * per_cu - 1) / (compute_units() * per_cu)) * per_cu * f.F * f.P * clocks_per_product[i] + 4000.0;
        if (best < 0 || cost < best_cost) {
            best = i;
            best_cost = cost;
        }
    }
    return best;
}

template <int LAYOUT, int WF, int WP, int PG>
hipError_t launch(const int8_t* x, const int8_t* w, int32_t* y, const Problem& p, hipStream_t s) {
    constexpr Form f = {64 * WF, 32 * PG * WP, 64 * WF * WP};
    static LdsLimitOnce lds_limit;   // per template instance
    if (hipError_t e = lds_limit.set(reinterpret_cast<const void*>(&direct_gemm_kernel<LAYOUT, WF, WP, PG>), kLdsMost)) return e;
    const dim3 grid((unsigned)(((long long)p.N * p.H * p.W + f.P - 1) / f.P), ceil_div(p.K, f.F));
    direct_gemm_kernel<LAYOUT, WF, WP, PG><<<grid, f.threads, lds_bytes(f, p), s>>>(x, w, p.N, p.C, p.H, p.W, p.K, y, p);
    return hipGetLastError();
}
template <int LAYOUT>
hipError_t launch_form(int form, const int8_t* x, const int8_t* w, int32_t* y, const Problem& p, hipStream_t s) {
    switch (form) {
        case 0: return launch<LAYOUT, 2, 4, 4>(x, w, y, p, s);
        case 1: return launch<LAYOUT, 1, 8, 2>(x, w, y, p, s);
        case 2: return launch<LAYOUT, 1, 8, 1>(x, w, y, p, s);
        default: return launch<LAYOUT, 1, 4, 1>(x, w, y, p, s);
    }
}

}  // namespace

bool direct_gemm_applies(const Problem& p) { return choose_form(p) >= 0; }

hipError_t launch_direct_gemm(const int8_t* x, const int8_t* w, int32_t* y, const Problem& p, int layout, hipStream_t s) {
    const int form = choose_form(p);
    return layout == WG_NHWC ? launch_form<WG_NHWC>(form, x, w, y, p, s) : launch_form<WG_NCHW>(form, x, w, y, p, s);
}

}  // namespace wg
