// The grid path's kernels for data held in LDS (sampler_team_kernel),
// instantiated for float data with the optional features compiled in (their own
// translation unit keeps the build parallel).
#include "sampler_impl.h"

namespace nuts {

const void* team_kernel_ext_f32(int D) { return sampler::team_kernel_for<float, true>(D); }

}  // namespace nuts
