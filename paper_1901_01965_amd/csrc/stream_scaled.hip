// The streaming role-specialised kernel, scaled mode (a file of its own so that the modes compile side by side).
#include "stream_kernel.h"

namespace wg {

hipError_t launch_stream_scaled(const RolesCall& c, StreamForm form, hipStream_t s) { return launch_stream_mode<WG_SCALED>(c, form, s); }

}  // namespace wg
