// FP64 sweep (project_fp64_sweep_kernel.hpp) with 1 column: the plain, sampled and scaled
// variants on double sources and the plain one on float sources.
#include "project_fp64_sweep_launch.hpp"

namespace los {

hipError_t project_sweep_launch_n1(const ProjectArgs &a, const SweepShape &sh, bool f32, bool scaled,
                                   hipStream_t s) {
  return sweep::launch<1>(a, sh, f32, scaled, s);
}

}  // namespace los
