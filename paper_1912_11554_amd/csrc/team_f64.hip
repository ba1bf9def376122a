// The grid path's kernels for data held in LDS (sampler_team_kernel),
// instantiated for double data (their own
// translation unit keeps the build parallel).
#include "sampler_impl.h"

namespace nuts {

const void* team_kernel_f64(int D) { return sampler::team_kernel_for<double, false>(D); }

}  // namespace nuts
