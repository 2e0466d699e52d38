// step_large.hip -- the step kernel of the Large capacity class (Table 4).
#include "step_kernel.h"

namespace k2d_impl {
int launch_step_large(const StepLaunch& s) { return launch_step_class<12, 4, 6, 2>(s); }
}  // namespace k2d_impl
