// Which int32 outputs are written through the L2 (write_out, kernel_common.h): rules on their number, their lines and where they lie.  Host only.
#pragma once
#include "wg_internal.h"

namespace wg {

// Where writing through pays.  Few outputs are written back in no time (64 -> 64 at 56x56, N = 1, 0.8 MB, scaled 7.43 us,
// through 7.54, direct 4.13 and 4.18); of more than 64 MB most are written back while the kernel runs (102 and 205 MB 0.98 - 1.04 of the time);
// lines that are written in parts (channels-last, K % 32 != 0) cost the memory a read each where they are many (direct convolution,
// K = 100, 18 MB 0.87, 38 MB 0.95 of the time, 50 MB 2.1).  Channel-major rows of W outputs are parts of lines: from 16 outputs on (7x7 1.05,
// 14x14 1.03 of the time, 28x28 0.98), and above 16 MB from 48 on (128 -> 128, N = 128 at 28x28, 51 MB, 1.04 - 1.06; 64 -> 64, N = 64 at
// 56x56 0.91).
// Memory takes 64 bytes at a time: outputs that start 16 bytes after a multiple of 64, as a view may, are all written in parts (of the
// time, plain / through: scaled, lossless, both scaled, F(2x2) and direct, 64 -> 64 at 56x56, N = 64 1.21, 1.15, 1.30, 1.25, 1.29, 128 -> 128, N = 40
// 1.25, 1.20, 1.35, 1.10, 1.50; channel-major 64 -> 64 at 32x64, N = 61 1.12, 1.16; 64 bytes after one 0.87 - 1.03).
constexpr int kThroughRows = 1, kThroughPlanes = 2, kThroughFewest = 512 << 10;   // outputs
inline bool on_unit(const void* y) { return reinterpret_cast<uintptr_t>(y) % 64 == 0; }
inline int writes_through(const Problem& p, const void* y) {
    const long long outputs = (long long)p.N * p.H * p.W * p.K;
    if (outputs < kThroughFewest || outputs > (p.K % 32 == 0 && on_unit(y) ? 16 << 20 : 6 << 20)) return 0;
    return kThroughRows | (p.W >= 16 && ((p.W >= 48 && on_unit(y)) || outputs <= 4 << 20) ? kThroughPlanes : 0);
}
inline bool f4_through(const Problem& p, const void* y, int layout) { return writes_through(p, y) & (layout == WG_NHWC ? kThroughRows : kThroughPlanes); }
inline bool f2_through(const Problem& p, const void* y) { return writes_through(p, y) & kThroughRows; }   // channels-last
bool direct_through(const Problem& p, const int32_t* y, int layout);   // direct_gemm.hip

}  // namespace wg
