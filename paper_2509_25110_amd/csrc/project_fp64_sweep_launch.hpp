// Launches of the FP64 sweep for one source count.
#pragma once

#include "project_fp64_sweep_kernel.hpp"

namespace los {
namespace sweep {

template <typename T, int NSRC, bool SMP, bool SC>
hipError_t launch_t(const ProjectArgs &a, const SweepShape &sh, hipStream_t s) {
  auto kern = project_fp64_sweep_kernel<T, NSRC, SMP, SC>;
  if (sh.waves < 1 || sh.waves > max_waves(NSRC) || sh.nodes < 64 || sh.nodes > 64 * 128)
    return hipErrorInvalidValue;
  if (sh.lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void *)kern,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh.lds);
    if (e != hipSuccess) return e;
  }
  ProjectArgs b = a;
  // A launch counts its threads in 32 bits and takes a larger grid without an error, modulo
  // 2^32: from 2^26 / waves rows on (2^24 with 4 waves) the rows go in several launches.
  const int64_t rows = ((int64_t)1 << 26) / sh.waves - 1;
  for (int64_t n0 = 0; n0 < a.ntau; n0 += sh.nodes) {
    b.n0 = (int)n0;
    b.ncnt = (int)(a.ntau - n0 < sh.nodes ? a.ntau - n0 : sh.nodes);
    b.accumulate = n0 > 0;
    for (b.kend = a.nk; b.kend > 0; b.kend -= rows) {
      const int64_t cnt = b.kend < rows ? b.kend : rows;
      hipLaunchKernelGGL(kern, dim3((unsigned)cnt), dim3(64 * sh.waves), sh.lds, s, b);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

template <int NSRC, bool SC>
hipError_t launch_f64(const ProjectArgs &a, const SweepShape &sh, hipStream_t s) {
  if (!a.lsel) return launch_t<double, NSRC, false, SC>(a, sh, s);
  if (!a.bmask) return hipErrorInvalidValue;
  return launch_t<double, NSRC, true, SC>(a, sh, s);
}

template <int NSRC>
hipError_t launch(const ProjectArgs &a, const SweepShape &sh, bool f32, bool scaled,
                  hipStream_t s) {
  if (f32) {
    if (scaled || a.lsel) return hipErrorInvalidValue;
    return launch_t<float, NSRC, false, false>(a, sh, s);
  }
  return scaled ? launch_f64<NSRC, true>(a, sh, s) : launch_f64<NSRC, false>(a, sh, s);
}

}  // namespace sweep
}  // namespace los
