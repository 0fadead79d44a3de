// FP64 sweep: launch shape and dispatch over the source count.  The kernel and its
// description are in project_fp64_sweep_kernel.hpp; project_fp64_sweep_n{1..4}.hip
// instantiate it.
#include <algorithm>

#include "project_fp64_sweep_kernel.hpp"

namespace los {

hipError_t project_sweep_launch_n1(const ProjectArgs &a, const SweepShape &sh, bool f32, bool scaled,
                                   hipStream_t s);
hipError_t project_sweep_launch_n2(const ProjectArgs &a, const SweepShape &sh, bool f32, bool scaled,
                                   hipStream_t s);
hipError_t project_sweep_launch_n3(const ProjectArgs &a, const SweepShape &sh, bool f32, bool scaled,
                                   hipStream_t s);
hipError_t project_sweep_launch_n4(const ProjectArgs &a, const SweepShape &sh, bool f32, bool scaled,
                                   hipStream_t s);

namespace {

// LDS of a workgroup: per node the pair, 1/x and the block of R; per wave the reduction
// stage and the progress word; two thresholds per slot.
size_t sweep_lds(int W, int64_t nodes, int nsrc) {
  return (size_t)nodes * (2 * sizeof(double) + sizeof(double) + sizeof(short)) +
         (size_t)W * (sizeof(double) * sweep::stage_doubles(nsrc) + sizeof(int)) +
         2 * sizeof(short) * (size_t)(nodes / 64);
}

}  // namespace

// Waves per workgroup.  More waves share a row's blocks, more workgroups on a CU work on
// rows that do not wait for each other.  Measured over W = 2 .. 16 on 41 shapes (1 to 4
// columns, 30 to 2999 multipoles, 165 to 4096 nodes, 66 to 5000 rows), from 7 blocks of
// multipoles on a multiple of 4 (every SIMD has the same number) is always within 4 % of the
// best, and the best is the largest
//   W g / (1 + W / 10),  g = workgroups on a CU: what LDS and registers allow, at most nk / 256
// e.g. 1751 nodes, 4 columns, 1253 rows: 4 waves 246 us (two workgroups), 8 waves 291 us (one);
// 565 nodes, 4 columns, 382 rows: 190 and 141 us; C2 in one pass (3000 nodes, one workgroup
// by LDS): 4, 8, 12 waves 2.86, 2.00, 1.78 ms; 1777 nodes, 2 columns, 1501 rows: 4, 8, 12
// waves 327, 244, 281 us.  With up to 6 blocks 2 waves count too (5 blocks keep 4 waves busy for
// 5/8 of the time, 2 for 5/6; 5 % off, so that near ties stay with 4): l <= 70, 3000 rows, 600
// nodes: 4 columns 148 -> 119 us, 3 columns 95 -> 82; l <= 80, 2000 x 1000, 4 columns 134 -> 115.
//
// Passes.  A row's nodes hold 26 bytes of LDS each for its whole time, so a long tau axis keeps
// other rows off the CU and the waves of one row wait for each other (each for the block above,
// all for the setup).  With rows enough for two rounds of as many 4-wave workgroups as the
// registers allow (g), the nodes therefore go in as many passes as give every one of the g its
// LDS; a pass adds to delta.  3 columns: C2 (2499 multipoles, 4000 k, 3000 nodes) 1776 us in one
// pass of 12 waves, 1672 in two of 4 (sampled: 1350, 1198); 899, 3000, 4000: 915, 848 in three;
// 249, 4000, 4096: 823, 736; but 899, 1200, 4000: 373, 445; 1499, 1000, 4000: 396, 668.  4
// columns (two workgroups): 1499, 2000, 3000: 931, 876.  1 column: 1499, 3000, 4000: 811, 713
// in four.  2 columns: 2499, 4000, 2500: 1115, 1004 in three.  With up to 8 blocks 16 or 12 waves
// mostly wait, and 3 rows a CU are enough: 1 column, 100, 800, 3000: 102, 94 in three; 3 columns
// 127, 110 in two; 4 columns 177, 167 in two; but 60, 600, 3500 (1 to 4 columns) 3 to 14 % slower.
SweepShape project_sweep_shape(int nsrc, int nl, int64_t nk, int64_t ntau, int force_waves) {
  constexpr size_t kLds = 160 * 1024;
  const int wmax = sweep::max_waves(nsrc);
  int64_t passes = 1;
  const int nblk = (nl + kSweepBlock - 1) / kSweepBlock;
  if (force_waves <= 0 && nk >= (nblk <= 8 ? 768 : 512 * (wmax / 4))) {
    const int64_t fit = (int64_t)(kLds / (wmax / 4) - sweep_lds(4, 0, nsrc)) /
                        (int64_t)sweep_lds(0, 64, nsrc) * 64;
    if (ntau > fit) {
      passes = (ntau + fit - 1) / fit;
      force_waves = 4;
    }
  }
  // nodes per pass: all of them if 4 waves fit beside their LDS, else equal shares
  int64_t nodes = 0;
  for (;; ++passes) {
    nodes = ((ntau + passes - 1) / passes + 63) / 64 * 64;
    if (nodes <= 64 * 128 && sweep_lds(4, nodes, nsrc) <= kLds) break;
  }
  int W = force_waves < wmax ? force_waves : wmax;
  if (force_waves <= 0) {
    double best = 0.0;
    for (int w = nblk <= 6 ? 2 : 4; w <= wmax; w += w < 4 ? 2 : 4) {
      const size_t lds = sweep_lds(w, nodes, nsrc);
      if (lds > kLds) break;
      double g = (double)std::min<size_t>(kLds / lds, (size_t)(wmax / w));
      g = std::min(g, (double)nk / 256.0);
      const double score = w * g / (1.0 + 0.1 * w) * (w < 4 ? 0.95 : 1.0);
      if (score > best) {
        best = score;
        W = w;
      }
    }
  }
  while (sweep_lds(W, nodes, nsrc) > kLds) --W;
  SweepShape sh{};
  sh.waves = W;
  sh.nodes = (int)nodes;
  sh.lds = sweep_lds(W, nodes, nsrc);
  return sh;
}

hipError_t project_sweep_launch(const ProjectArgs &a, int nsrc, const SweepShape &sh, bool f32,
                                hipStream_t s) {
  // scaled columns or remapped source planes take the scaled variants
  bool sc = (a.emask | a.x1mask | a.x2mask) != 0u;
  for (int q = 0; q < nsrc && q < 4; ++q) sc = sc || a.splane[q] != q;
  switch (nsrc) {
    case 1: return project_sweep_launch_n1(a, sh, f32, sc, s);
    case 2: return project_sweep_launch_n2(a, sh, f32, sc, s);
    case 3: return project_sweep_launch_n3(a, sh, f32, sc, s);
    case 4: return project_sweep_launch_n4(a, sh, f32, sc, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace los
