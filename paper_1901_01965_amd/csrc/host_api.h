// What the Python extension (torch_binding.cpp) calls beyond the C ABI of winograd_c.h: entry points that take their
// scratch memory as an option.  Plain host declarations, no HIP types.
#pragma once
#include "winograd_c.h"

namespace wg {

// Scratch memory with which the single-kernel path runs this convolution best (0: it has no use for any), and its entry
// points with that memory: 256-byte aligned, for this call alone while it runs; null / fewer bytes are accepted and only
// cost time.
size_t conv2d_scratch_bytes(int N, int C, int H, int W, int K, int layout, int mode, int is_unsigned);
int conv2d_int8_with_scratch(const int8_t* x, const void* packed, int32_t* y, int N, int C, int H, int W, int K, int layout,
                             int mode, void* scratch, size_t scratch_bytes, void* stream);
int conv2d_int8_requant_with_scratch(const int8_t* x, const void* packed, int8_t* out, int N, int C, int H, int W, int K, int layout,
                                     int mode, int shift, int relu, int pool, void* scratch, size_t scratch_bytes, void* stream);
int conv2d_u8_with_scratch(const uint8_t* x, int zero_point, const void* packed, int32_t* y, int N, int C, int H, int W, int K,
                           int layout, int mode, void* scratch, size_t scratch_bytes, void* stream);
size_t act_scaled_scratch_bytes(int N, int C, int H, int W, int K, int layout);
int conv2d_int8_act_scaled_with_scratch(const int8_t* x, const void* packed, int32_t* y, int N, int C, int H, int W, int K, int layout,
                                        int32_t* act_table, void* scratch, size_t scratch_bytes, void* stream);
size_t f2x2_conv2d_scratch_bytes(int N, int C, int H, int W, int K, int layout);
int f2x2_conv2d_with_scratch(const void* x, int is_unsigned, int zero_point, const void* packed, int32_t* y, int N, int C, int H, int W,
                             int K, int layout, int mode, void* scratch, size_t scratch_bytes, void* stream);
int f2x2_conv2d_int8_requant_with_scratch(const int8_t* x, const void* packed, int8_t* out, int N, int C, int H, int W, int K,
                                          int layout, int mode, int shift, int relu, int pool, void* scratch, size_t scratch_bytes,
                                          void* stream);
size_t direct_conv2d_scratch_bytes(int N, int C, int H, int W, int K, int layout);
int direct_conv2d_with_scratch(const int8_t* x, const int8_t* w, int32_t* y, int N, int C, int H, int W, int K, int layout, void* scratch,
                               size_t scratch_bytes, void* stream);

}  // namespace wg
