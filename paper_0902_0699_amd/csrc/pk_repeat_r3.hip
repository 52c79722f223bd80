// Kernel instances (repeat, 3 register bits) of the templates in pk_pass.h, in a
// translation unit of their own so that the build compiles them in parallel.
#include "pk_pass.h"

namespace pk {
template hipError_t launch_repeat_r<double, 3>(int, const KArgs&, const RepeatArgs&, unsigned, hipStream_t);
template hipError_t launch_repeat_r<float, 3>(int, const KArgs&, const RepeatArgs&, unsigned, hipStream_t);
template int repeat_occupancy_r<double, 3>(int);
template int repeat_occupancy_r<float, 3>(int);
}  // namespace pk
