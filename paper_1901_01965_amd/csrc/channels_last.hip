// Channels-last copy of activations, pixel stride padded to a multiple of four (sixteen) channels, for inputs that the
// 4-byte pixel loads of the convolution kernels cannot read: channel-major tensors, and channel counts that are not a
// multiple of four.  Reading those tensors inside the convolution takes one load per byte (144 per tile and four
// channels, 36 instead) and repeats it for every filter block: 100 -> 75 channels at 37x53, N = 4, channel-major, 47 us
// in one kernel.  The copy moves each byte once.
//
// Bound by memory: a thread reads four pixels of sixteen channels with 4-byte loads (any alignment), turns each 4x4 block
// of bytes with eight v_perm, and stores 16 bytes per pixel.
#include "wg_internal.h"

namespace wg {
namespace {

struct __attribute__((packed)) PackedWord {   // a 4-byte load at any address
    uint32_t v;
};
__device__ inline uint32_t load_word(const int8_t* at) { return reinterpret_cast<const PackedWord*>(at)->v; }
__device__ inline uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) { return __builtin_amdgcn_perm(hi, lo, sel); }

// Channel-major: x[n][c][pixel], pixel < HW.  Thread: pixels q0 .. q0 + 3 (the last thread of an image steps back so that
// all four exist, and rewrites what its neighbour writes) and channels 16 g .. 16 g + 15.  HW >= 4.
// grid: (ceil(quads / 64), ceil(Cp / 64), N), 256 threads: lane = pixel quad, wave = channel group.
__global__ __launch_bounds__(256) void channels_last_from_planes_kernel(const int8_t* __restrict__ x, int8_t* __restrict__ out, int C, int Cp,
                                                                        int HW, uint32_t fill) {
    const int quad = blockIdx.x * 64 + (threadIdx.x & 63), c0 = (blockIdx.y * 4 + (threadIdx.x >> 6)) * 16;
    const int quads = (HW + 3) >> 2;
    if (quad >= quads || c0 >= Cp) return;
    const int q0 = min(4 * quad, HW - 4);
    const int8_t* const src = x + (size_t)blockIdx.z * C * HW + q0;
    uint32_t in[16], px[4][4];   // [channel], [pixel][four channels]
#pragma unroll
    for (int c = 0; c < 16; ++c) in[c] = c0 + c < C ? load_word(src + (size_t)(c0 + c) * HW) : fill;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const uint32_t a = perm(in[4 * g + 1], in[4 * g], 0x05010400u), b = perm(in[4 * g + 1], in[4 * g], 0x07030602u);
        const uint32_t c = perm(in[4 * g + 3], in[4 * g + 2], 0x05010400u), d = perm(in[4 * g + 3], in[4 * g + 2], 0x07030602u);
        px[0][g] = perm(c, a, 0x05040100u);
        px[1][g] = perm(c, a, 0x07060302u);
        px[2][g] = perm(d, b, 0x05040100u);
        px[3][g] = perm(d, b, 0x07060302u);
    }
    int8_t* const dst = out + ((size_t)blockIdx.z * HW + q0) * Cp + c0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (Cp % 16 == 0) *reinterpret_cast<uint4*>(dst + (size_t)i * Cp) = make_uint4(px[i][0], px[i][1], px[i][2], px[i][3]);
        else              *reinterpret_cast<uint32_t*>(dst + (size_t)i * Cp) = px[i][0];   // Cp = 4
    }
}

// Everything else (channels-last with C % 4 != 0; images of fewer than four pixels): one dword of the copy per thread.
template <int LAYOUT>
__global__ __launch_bounds__(256) void channels_last_kernel(const int8_t* __restrict__ x, int8_t* __restrict__ out, int C, int Cp, int HW,
                                                            uint32_t total, uint32_t fill) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;   // [pixel of the batch][Cp / 4]
    if (i >= total) return;
    const uint32_t per = (uint32_t)Cp >> 2, pixel = i / per;
    const int c = 4 * (int)(i - pixel * per);
    uint32_t word = 0;
    if (LAYOUT == WG_NHWC && c + 4 <= C) {
        word = load_word(x + (size_t)pixel * C + c);
    } else {
        const uint32_t n = pixel / (uint32_t)HW;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const size_t at = LAYOUT == WG_NHWC ? (size_t)pixel * C + c + j : ((size_t)n * C + c + j) * HW + (pixel - n * (uint32_t)HW);
            word |= (c + j < C ? (uint32_t)(uint8_t)x[at] : fill & 0xffu) << (8 * j);
        }
    }
    reinterpret_cast<uint32_t*>(out)[i] = word;
}

}  // namespace

hipError_t launch_channels_last(const int8_t* x, int8_t* out, const Problem& p, int layout, int padded, uint8_t fill_byte, hipStream_t s) {
    const int HW = p.H * p.W;
    const uint32_t fill = 0x01010101u * fill_byte;
    if (layout == WG_NCHW && HW >= 4 && p.N <= 65535) {
        channels_last_from_planes_kernel<<<dim3(ceil_div(ceil_div(HW, 4), 64), ceil_div(padded, 64), p.N), 256, 0, s>>>(x, out, p.C, padded, HW, fill);
        return hipGetLastError();
    }
    const size_t total = (size_t)p.N * HW * (padded / 4);
    const unsigned blocks = (unsigned)((total + 255) / 256);
    if (layout == WG_NHWC) channels_last_kernel<WG_NHWC><<<blocks, 256, 0, s>>>(x, out, p.C, padded, HW, (uint32_t)total, fill);
    else                   channels_last_kernel<WG_NCHW><<<blocks, 256, 0, s>>>(x, out, p.C, padded, HW, (uint32_t)total, fill);
    return hipGetLastError();
}

}  // namespace wg
