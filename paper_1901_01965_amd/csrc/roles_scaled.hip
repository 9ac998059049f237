// The role-specialised kernel, scaled mode (a file of its own so that the modes compile side by side).
#include "roles_kernel.h"

namespace wg {

hipError_t launch_roles_scaled(const RolesCall& c, bool wide, hipStream_t s) { return launch_roles_mode<WG_SCALED>(c, wide, s); }
}  // namespace wg
