// Which outputs are written through the L2 (write_out, kernel_common.h): rules on their number, their lines and where they lie.  Host only.
#pragma once
#include "wg_internal.h"

namespace wg {

// Where writing through pays.  Few outputs are written back in no time (64 -> 64 at 56x56, N = 1, 0.8 MB, scaled 7.43 us,
// through 7.54, direct 4.13 and 4.18); of more than 64 MB most are written back while the kernel runs (102 and 205 MB 0.98 - 1.04 of the time);
// lines that are written in parts (channels-last, K % 32 != 0) cost the memory a read each where they are many.  Where a kernel stores 32 filters of a
// pixel at once, that begins at 20 MB (of the time, scaled, lossless, both scaled, K = 36 .. 200: 17 MB 0.93 - 1.03, 20 MB 0.97 - 1.08, 24 MB
// 1.06 - 1.21), unless 64-byte units are whole (K % 16 = 0: 24 MB 0.88 - 0.99, 60 MB 0.91 - 1.03); F(2x2) and direct kernels store 64, 20 MB 0.87 - 1.02,
// 24 MB 0.93 - 1.13 (K % 16 = 0 0.90 - 1.03, F(2x2) with K = 16 1.05).
// Channel-major rows of W outputs are whole units where W % 16 = 0, whatever K is (16 -> 256 at most, to 60 MB 0.87 - 1.01), else parts: from 20 outputs on,
// where they are few (8 MB, W = 20 .. 56 0.91 - 1.03; W = 15 .. 19 up to 1.05; 7x7 1.05), from 28 on up to 16 MB (0.91 - 1.03; W = 20 and 24 up to 1.08), not
// above (W = 28 .. 75, 28 MB 1.02 - 1.21, 60 MB 1.04 - 1.49: 64 -> 64 at 56x56, N = 62, lossless 45.3 us plain, 54.0 through).
// Memory takes 64 bytes at a time: outputs that start 16 bytes after a multiple of 64, as a view may, are all written in parts (through, of the
// time: scaled, lossless, both scaled, F(2x2) and direct, 64 -> 64 at 56x56, N = 64 1.21, 1.15, 1.30, 1.25, 1.29, 128 -> 128, N = 40
// 1.25, 1.20, 1.35, 1.10, 1.50; channel-major 64 -> 64 at 32x64, N = 61 1.12, 1.16; 64 bytes after one 0.87 - 1.03).  With 32 filters of
// a pixel at once that does not pay in any number (2 - 8 MB 0.97 - 1.01, 16 MB 0.97 - 1.06), with 64 up to 20 MB (0.88 - 1.00).
constexpr int kThroughFewest = 512 << 10;   // outputs
inline long long outputs_of(const Problem& p) { return (long long)p.N * p.H * p.W * p.K; }
inline bool on_unit(const void* y) { return reinterpret_cast<uintptr_t>(y) % 64 == 0; }
// Channels-last outputs, `filters` of a pixel stored at once.
inline bool rows_through(const Problem& p, const void* y, int filters) {
    const bool wide = filters == 64;
    const long long parts = wide ? 5 << 20 : on_unit(y) ? 4 << 20 : 0;
    const long long most = !on_unit(y) ? parts : p.K % 32 == 0 ? 16 << 20 : p.K % 16 == 0 && 2 * p.K >= filters ? 6 << 20 : parts;
    return outputs_of(p) >= kThroughFewest && outputs_of(p) <= most;
}
// The most channel-major outputs that are written through.
inline long long planes_most(const Problem& p, const void* y) {
    if (on_unit(y) && p.W % 16 == 0) return 16 << 20;
    return on_unit(y) && p.W >= 28 ? 4 << 20 : p.W >= 20 ? 2 << 20 : 0;
}
inline bool planes_through(const Problem& p, const void* y) { return outputs_of(p) >= kThroughFewest && outputs_of(p) <= planes_most(p, y); }
inline bool f4_through(const Problem& p, const void* y, int layout) { return layout == WG_NHWC ? rows_through(p, y, 32) : planes_through(p, y); }
inline bool f2_through(const Problem& p, const void* y) { return rows_through(p, y, 64); }   // channels-last
// Limb-pair kernel, channel-major outputs, which are not many: few pay as well (plain / through, us, 64 -> 64 at 28x28, N = 4, 7.54 / 7.42, 56x56, N = 8 9.8 / 9.1, 16 -> 16
// at 16x16 level), but no narrow rows (8x7x7 7.32 / 7.72, 60x14x7 7.60 / 7.96, 14x14 1.01, W = 17 and 18 1.00 - 1.02 of the time).
inline bool pair_planes_through(const Problem& p, const void* y) { return outputs_of(p) <= planes_most(p, y); }
// First layers on the matrix cores, channels-last, `bytes` 4 (int32) or 1 (int8): 64 filters of the pixels of a tile's row are stored together, so that
// up to 64 filters are whole units also where one pixel's are not.  Whole, any number of them pays (224x224, N = 1 .. 16, K = 32 .. 256, 6 - 200 MB
// 0.83 - 1.01 of the time, int8 0.87 - 1.02); int32 parts up to 20 MB (K = 68 .. 200 0.84 - 0.95, 25 MB 0.95 - 1.11; above, up to 1.4: K = 52 at 223x225, N = 16,
// 49.3 us plain, 69.4 through, 168 at 112x112, N = 24, lossless 71.1 / 89.2), int8 parts up to 32 MB (0.83 - 0.98; 38 - 100 MB 1.01 - 1.09).
inline bool first_layer_through(const Problem& p, const void* out, int bytes, bool pool) {
    const long long row = (pool ? 2 : 4) * (long long)p.K * bytes, outputs = pool ? outputs_of(p) / 4 : outputs_of(p);
    const bool whole = p.K * bytes % 64 == 0 || (p.K <= 64 && p.W % 4 == 0 && row % 64 == 0);
    return (whole && on_unit(out)) || outputs <= (bytes == 4 ? 5 << 20 : 32 << 20);
}
bool direct_through(const Problem& p, const int32_t* y);   // channels-last (direct_gemm.hip)

}  // namespace wg
