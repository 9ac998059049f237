// Direct convolution on the int8 matrix cores as an implicit matrix product over linear pixels: y[pixel][k] = sum over nine
// taps and C channels.  Activations channels-last with C % 16 = 0 (as given, or as a padded copy), filters [K][9][C].
//
// What bounds it: with operands in LDS a wave reads (A + B) fragments of 1 KB for A x B matrix instructions of 32 clocks.  A
// wave tile of 64 filters x 128 pixels asks for 6 KB per eight of them, 96 B per clock for four SIMDs; the 32 x 64 tile per
// wave of the patch kernel (direct_conv.hip) asks for 192 B per clock.  Vector instructions delay matrix instructions of their
// SIMD, so the loop has few: read addresses are kept, not formed (see at_pixel), and transfers take one addition each
// (93 vector instructions for 144 products; formed anew, 620, and 256 -> 256 channels at 56x56, N = 16 took 39.8 us instead of 37.4,
// 512 -> 512 at 28x28 39.4 instead of 35.5).  The former takes 33.0 us (1790 TOPS) on activations of which half are zeros, 37.2 on
// uniform ones, of which set-up and first transfers some 2, stores of 51 MB at the end, all compute units at once, 10; 256 -> 256 at
// 56x56, N = 4 11.2.  (A 256 x 224 tile of 16 x 16 x 64 products, 224 workgroups instead of 196 there: level.)
//
// Workgroup: P consecutive pixels of the batch (in memory order, so only the last workgroup has idle columns, whatever the
// image size) x F filters.  LDS holds, per block of 64 channels, the pixel rows p0 - W - 1 .. p0 + P + W (a tap is a row
// offset of (a - 1) W + (b - 1)) and the taps of one filter row; both double-buffered and filled by 16-byte transfers from
// memory straight into LDS that run during the products.  A tap that falls outside the image reads a row of zeros.  A stage is
// one filter row of one channel block: 48 matrix instructions per wave, one barrier.
#include <algorithm>

#include "kernel_common.h"
#include "write_through.h"

namespace wg {
namespace {

typedef int v16i __attribute__((ext_vector_type(16)));

// 16-byte pieces of a 64-byte LDS row are XOR-swizzled so that the fragment reads of 16 consecutive rows fall into
// different banks; the swizzle is applied on the global side of the transfers.
__device__ inline int piece_at(int row, int slot) { return slot ^ ((row >> 2) & 3); }

__device__ inline void to_lds_16(__amdgpu_buffer_rsrc_t buffer, int8_t* lds_dst, uint32_t voffset) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(buffer, (__attribute__((address_space(3))) int8_t*)lds_dst, 16, voffset, 0, 0, 0);
}

// Fragments are read at addresses within LDS, kept as integers: as offsets from its start each read added that start first.
using LdsBytes = const __attribute__((address_space(3))) int8_t;
__device__ inline v4i fragment_at(int address) { return *reinterpret_cast<const __attribute__((address_space(3))) v4i*>(reinterpret_cast<LdsBytes*>((uintptr_t)(uint32_t)address)); }

constexpr int kStagedPixel = 64 * 4 + 16;   // bytes of a pixel's 64 sums in LDS, and what keeps the writes off each other's banks

// Pixel rows a workgroup keeps, rounded up to whole 1 KB transfers; a row of zeros follows them.
__host__ __device__ inline int halo_rows(int P, int W) { return (P + 2 * W + 2 + 15) / 16 * 16; }
__host__ __device__ inline int halo_bytes_of(int P, int W) { return (halo_rows(P, W) + 1) * kCBlock; }

// WF x WP waves; a wave multiplies 64 filters x 32 PG pixels.  F = 64 WF, P = 32 PG WP.  THROUGH: whole pixels are written through the L2 (write_out).
// grid: (ceil(pixels / P), ceil(K / F)), 64 WF WP threads.
template <int LAYOUT, int WF, int WP, int PG, bool THROUGH>
__global__ __launch_bounds__(64 * WF * WP) void direct_gemm_kernel(const int8_t* __restrict__ x, const int8_t* __restrict__ w,
                                                                   int N, int C, int H, int W, int K, int32_t* __restrict__ y, Problem p) {
    p.N = N; p.C = C; p.H = H; p.W = W; p.K = K;   // (in registers when a wave starts)
    constexpr int F = 64 * WF, P = 32 * PG * WP, T = 64 * WF * WP, TAPS = (3 * F * 4 + T - 1) / T;
    constexpr int kTapBytes = 3 * F * kCBlock;
    extern __shared__ __attribute__((aligned(16))) int8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wf = wave % WF, wp = wave / WF;
    const int pixels = p.N * p.H * p.W, p0 = blockIdx.x * P, k0 = blockIdx.y * F;
    const int rows = halo_rows(P, p.W), halo_bytes = halo_bytes_of(P, p.W);
    int8_t* const taps = lds;                    // two buffers
    int8_t* const halo = taps + 2 * kTapBytes;   // two buffers
    const __amdgpu_buffer_rsrc_t xbuf = activation_buffer(x, p);
    const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(w), 0, p.K * 9 * p.C, kRawBufferWord3);
    if (tid < 2 * kCBlock / 4) reinterpret_cast<int*>(halo + (tid >> 4) * halo_bytes + rows * kCBlock)[tid & 15] = 0;

    // A thread's transfers lie T / 4 rows apart, a multiple of 16: its piece of a row is the same in all.  Pixels outside the batch
    // and filters beyond K lie outside the buffers and arrive as zeros.  So do taps beyond C; what the pixels hold there does not matter.
    const int my_row = tid >> 2, my_c = 16 * piece_at(my_row, tid & 3);
    const uint32_t first_pixel = (uint32_t)(p0 - p.W - 1 + my_row) * (uint32_t)p.C + (uint32_t)my_c;
    uint32_t first_tap[TAPS];
#pragma unroll
    for (int i = 0; i < TAPS; ++i) {
        const int row = i * (T / 4) + my_row, b = row / F, k = k0 + row % F;   // LDS row = 3 taps x F filters: [tap b][filter]
        first_tap[i] = (uint32_t)(k * 9 + b) * (uint32_t)p.C + (uint32_t)my_c;
    }
    auto request_halo = [&](int cb, int8_t* dst) {
        uint32_t at = first_pixel + cb * kCBlock;
        for (int base = wave * 64; base < rows * 4; base += T) {
            to_lds_16(xbuf, dst + base * 16, at);
            at += T / 4 * p.C;
        }
    };
    auto request_taps = [&](int cb, int a, int8_t* dst) {
        const bool have = cb * kCBlock + my_c < p.C;
        const uint32_t from = 3 * a * p.C + cb * kCBlock;
#pragma unroll
        for (int i = 0; i < TAPS; ++i) {
            const int base = i * T + wave * 64;
            if (base < 3 * F * 4) to_lds_16(wbuf, dst + base * 16, have ? first_tap[i] + from : kOutsideOffset);
        }
    };

    // Where this lane reads its pixels' rows (one pixel per group) for each tap, in the halo buffer of this channel block: rows outside
    // the image are the row of zeros.  One addition and one exclusive or per tap, group and channel block keep them up to date
    // (the channel halves are taken in the order 0 1, 1 0, ...).
    int at_pixel[9][PG];
    const int lds_start = (int)(uint32_t)reinterpret_cast<uintptr_t>((LdsBytes*)lds);
    const int upper = lane >> 5;   // which 16 of a step's 32 channels
#pragma unroll
    for (int g = 0; g < PG; ++g) {
        const int in_block = (wp * PG + g) * 32 + (lane & 31), pixel = p0 + in_block;
        const int h = (pixel / p.W) % p.H, wcol = pixel % p.W;
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const bool inside = (unsigned)(h + a - 1) < (unsigned)p.H && (unsigned)(wcol + b - 1) < (unsigned)p.W;
                const int row = inside ? in_block + a * p.W + b : rows;
                at_pixel[3 * a + b][g] = lds_start + 2 * kTapBytes + row * kCBlock + 16 * piece_at(row, upper);
            }
    }
    const int tap_row = wf * 64 + (lane & 31);   // the others lie a multiple of 32 rows away
    const int at_tap = lds_start + tap_row * kCBlock + 16 * piece_at(tap_row, upper);
    v16i acc[2][PG];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int g = 0; g < PG; ++g) acc[f][g] = (v16i){0};

    // Six steps of 32 channels (tap b, half) a stage.  A step's fragments are read while the step before multiplies, a stage's first
    // ones too: the barrier that says that its rows are there comes before the last step of the stage before, when all
    // fragments of that stage are in registers.
    v4i A[2][2], B[2][PG];
    auto read = [&](auto TAP, auto STEP, int cb, int stage) {   // STEP: 2 b + how many halves of this tap are read already
        constexpr int tap = TAP, step = STEP;
        const int tap_rows = (stage & 1) * kTapBytes + (at_tap ^ 32 * ((cb ^ step) & 1));
#pragma unroll
        for (int f = 0; f < 2; ++f) A[step & 1][f] = fragment_at(tap_rows + ((step / 2) * F + f * 32) * kCBlock);
#pragma unroll
        for (int g = 0; g < PG; ++g) {
            int& at = at_pixel[tap][g];
            B[step & 1][g] = fragment_at(at);
            if constexpr (step & 1) at += cb & 1 ? -halo_bytes : halo_bytes;
            else at ^= 32;
        }
    };
    auto rows_are_there = [] {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
    };
    request_halo(0, halo);
    request_taps(0, 0, taps);
    rows_are_there();
    read(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, 0, 0);
    for (int cb = 0; cb < p.CB; ++cb) {
        const bool more = cb + 1 < p.CB;
        static_for<3>([&](auto ROW) {
            constexpr int a = ROW;
            const int s = 3 * cb + a;
            if (a < 2) request_taps(cb, a + 1, taps + ((s + 1) & 1) * kTapBytes);
            else if (more) request_taps(cb + 1, 0, taps + ((s + 1) & 1) * kTapBytes);
            if (a == 0 && more) request_halo(cb + 1, halo + ((cb + 1) & 1) * halo_bytes);
            static_for<6>([&](auto S) {
                constexpr int step = S;
                if constexpr (step + 1 < 6) {
                    read(std::integral_constant<int, 3 * a + (step + 1) / 2>{}, std::integral_constant<int, step + 1>{}, cb, s);
                } else if constexpr (a < 2) {
                    rows_are_there();
                    read(std::integral_constant<int, 3 * a + 3>{}, std::integral_constant<int, 0>{}, cb, s + 1);
                } else if (more) {
                    rows_are_there();
                    read(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, cb + 1, s + 1);
                }
#pragma unroll
                for (int g = 0; g < PG; ++g)
#pragma unroll
                    for (int f = 0; f < 2; ++f) acc[f][g] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[step & 1][f], B[step & 1][g], acc[f][g], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    }

    // Whole cache lines per store: 32 pixels x 64 filters at a time by way of LDS, 256 bytes of a pixel from 16 lanes, or from 64 where
    // K is no multiple of 4.  Stored from the registers, 32 bytes a pixel, the 51 MB of 256 -> 256 channels at 56x56, N = 16 took
    // 37.4 us in all instead of 36.0, 16 -> 320 at 19x19, N = 43 9.9 instead of 8.2; 151 -> 245 at 54x14,
    // N = 106 112 instead of 73; 60 mixed channels-last layers 1.08 times as fast.  Waves with fewer filters, 33 where K is no multiple
    // of 4: level, or slower by the trip (97 -> 23 at 18x18, N = 4 10.1 and 10.7).
    const int kw = k0 + wf * 64;
    const bool quads = (p.K & 3) == 0;
    const int staged_from = quads ? 64 : 33;
    if (LAYOUT == WG_NHWC && k0 + staged_from <= p.K) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();   // nobody reads the last stage's rows any more
        if (kw + staged_from <= p.K) {
            int8_t* const mine = lds + wave * (32 * kStagedPixel);
            int8_t* const put = mine + (lane & 31) * kStagedPixel + 16 * upper;
#pragma unroll
            for (int g = 0; g < PG; ++g) {
                const int first = p0 + (wp * PG + g) * 32;
#pragma unroll
                for (int f = 0; f < 2; ++f)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *reinterpret_cast<v4i*>(put + 128 * f + 32 * q) = (v4i){acc[f][g][4 * q], acc[f][g][4 * q + 1], acc[f][g][4 * q + 2], acc[f][g][4 * q + 3]};
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if (quads) {
                    const int8_t* const take = mine + (lane >> 4) * kStagedPixel + 16 * (lane & 15);
                    const int pixel = first + (lane >> 4);
                    int32_t* const out = y + (size_t)pixel * p.K + kw + 4 * (lane & 15);
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const v4i v = *reinterpret_cast<const v4i*>(take + 4 * i * kStagedPixel);
                        if (pixel + 4 * i < pixels) write_as<THROUGH>(reinterpret_cast<v4i*>(out + (size_t)(4 * i) * p.K), v);
                    }
                } else if (kw + lane < p.K) {
                    int32_t* const out = y + (size_t)first * p.K + kw + lane;
#pragma unroll 8
                    for (int i = 0; i < 32; ++i) {
                        const int32_t v = *reinterpret_cast<const int32_t*>(mine + i * kStagedPixel + 4 * lane);
                        if (first + i < pixels) out[(size_t)i * p.K] = v;
                    }
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
            return;
        }
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
                if (LAYOUT == WG_NHWC && quads) {
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
// (the sums of 32 pixels and 64 filters per wave take the place of the operands)
int lds_bytes(const Form& f, const Problem& p) {
    return std::max(2 * 3 * f.F * kCBlock + 2 * halo_bytes_of(f.P, p.W), f.threads / 64 * 32 * kStagedPixel);
}

// The form with the least estimated time: workgroups of the fullest compute unit times what one takes.  Per output that is, for each
// channel block, its products and the pixel rows that come beside its own, and once the set-up and the stores, which the other
// workgroups' products hide where two or more fit a compute unit.  The weights are fitted to 1720 layers of 16 .. 512 channels and
// rows of 7 .. 112 pixels, every form timed on each, and are 0.4 % from the best form on average.  (Products alone, at 1.0, 1.3, 1.4
// and 1.8: 2.5 %, with one channel block 4 %: 16 -> 304 at 23x23, N = 28 9.3 us, by 64 x 128 7.4; 16 -> 16 at 70x70, N = 129 27.9, by
// 64 x 256 22.1.)
int choose_form(const Problem& p) {
    const long long pixels = (long long)p.N * p.H * p.W;
    int best = -1;
    double best_cost = 0;
    for (int i = 0; i < 4; ++i) {
        const Form& f = kForms[i];
        if (lds_bytes(f, p) > kLdsMost) continue;
        const long long groups = (pixels + f.P - 1) / f.P * ceil_div(p.K, f.F);
        constexpr double products[4] = {1.0, 1.55, 1.7, 1.7};   // relative, as are the others
        const double beside = 1.95 * (halo_rows(f.P, p.W) - f.P) / f.P, once = 2 * lds_bytes(f, p) > kLdsMost ? 1.75 : 0.0;
        const double cost = (double)((groups + compute_units() - 1) / compute_units()) * f.F * f.P * ((products[i] + beside) * p.CB + once);
        if (best < 0 || cost < best_cost) {
            best = i;
            best_cost = cost;
        }
    }
    return best;
}

template <int LAYOUT, int WF, int WP, int PG, bool THROUGH>
hipError_t launch(const int8_t* x, const int8_t* w, int32_t* y, const Problem& p, hipStream_t s) {
    constexpr Form f = {64 * WF, 32 * PG * WP, 64 * WF * WP};
    static LdsLimitOnce lds_limit;   // per template instance
    if (hipError_t e = lds_limit.set(reinterpret_cast<const void*>(&direct_gemm_kernel<LAYOUT, WF, WP, PG, THROUGH>), kLdsMost)) return e;
    const dim3 grid((unsigned)(((long long)p.N * p.H * p.W + f.P - 1) / f.P), ceil_div(p.K, f.F));
    direct_gemm_kernel<LAYOUT, WF, WP, PG, THROUGH><<<grid, f.threads, lds_bytes(f, p), s>>>(x, w, p.N, p.C, p.H, p.W, p.K, y, p);
    return hipGetLastError();
}
template <int LAYOUT, bool THROUGH>
hipError_t launch_form(int form, const int8_t* x, const int8_t* w, int32_t* y, const Problem& p, hipStream_t s) {
    switch (form) {
        case 0: return launch<LAYOUT, 2, 4, 4, THROUGH>(x, w, y, p, s);
        case 1: return launch<LAYOUT, 1, 8, 2, THROUGH>(x, w, y, p, s);
        case 2: return launch<LAYOUT, 1, 8, 1, THROUGH>(x, w, y, p, s);
        default: return launch<LAYOUT, 1, 4, 1, THROUGH>(x, w, y, p, s);
    }
}

}  // namespace

// Two filter blocks that write a line together (K % 32 != 0, or outputs off a line) must not do so from the same XCD at the same time: workgroups go
// to the eight XCDs in turn, so they do where the pixel blocks are a multiple of eight (us, plain / through: 64 -> 84 at 32x32, N = 16, 5.2 / 8.5,
// N = 32 7.0 / 13.1; at 56x56, N = 13, 160 pixel blocks, 8.3 / 12.5, N = 12 and 14, 147 and 172, 8.6 / 7.8 and 9.1 / 8.4; 64 -> 80, N = 15 8.4 / 9.7).
static bool through(const Problem& p, const int32_t* y, const Form& f) {
    const bool whole_lines = p.K % 32 == 0 && reinterpret_cast<uintptr_t>(y) % 128 == 0;
    return rows_through(p, y, 64) && (whole_lines || p.K <= f.F || ((long long)p.N * p.H * p.W + f.P - 1) / f.P % 8 != 0);
}
bool direct_through(const Problem& p, const int32_t* y) {
    const int form = choose_form(p);
    return form >= 0 && through(p, y, kForms[form]);
}
bool direct_gemm_applies(const Problem& p) { return choose_form(p) >= 0; }

hipError_t launch_direct_gemm(const int8_t* x, const int8_t* w, int32_t* y, const Problem& p, int layout, hipStream_t s) {
    const int form = choose_form(p);
    if (layout != WG_NHWC) return launch_form<WG_NCHW, false>(form, x, w, y, p, s);
    return through(p, y, kForms[form]) ? launch_form<WG_NHWC, true>(form, x, w, y, p, s) : launch_form<WG_NHWC, false>(form, x, w, y, p, s);
}

}  // namespace wg
