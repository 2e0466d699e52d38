// step_small.hip -- the step kernel of the Small capacity class (Table 4).
#include "step_kernel.h"

namespace k2d_impl {
int launch_step_small(const StepLaunch& s) { return launch_step_class<5, 2, 1, 1>(s); }
}  // namespace k2d_impl
