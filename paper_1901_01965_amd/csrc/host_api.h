// What the Python extension (torch_binding.cpp) calls beyond the C ABI of winograd_c.h: entry points that take their
// scratch memory as an option.  Plain host declarations, no HIP types.
#pragma once
#include "winograd_c.h"

namespace wg {

// winograd_conv2d_int8 where winograd_conv2d_path() is the single kernel, which needs no workspace.
int conv2d_int8_single_kernel(const int8_t* x, const void* packed, int32_t* y, int N, int C, int H, int W, int K, int layout,
                              int mode, void* stream);

}  // namespace wg
