// The streaming role-specialised kernel, lossless mode (a file of its own so that the modes compile side by side).
#include "stream_kernel.h"

namespace wg {

hipError_t launch_stream_lossless(const RolesCall& c, StreamForm form, hipStream_t s) { return launch_stream_mode<WG_LOSSLESS>(c, form, s); }

}  // namespace wg
