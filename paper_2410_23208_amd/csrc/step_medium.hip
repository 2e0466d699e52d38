// step_medium.hip -- the step kernel of the Medium capacity class (Table 4).
#include "step_kernel.h"

namespace k2d_impl {
int launch_step_medium(const StepLaunch& s) { return launch_step_class<6, 3, 2, 2>(s); }
}  // namespace k2d_impl
