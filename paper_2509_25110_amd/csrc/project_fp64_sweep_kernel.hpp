// FP64 line-of-sight projection, one descending sweep per k row (gCAMB paper
// Sec. 2.1 Eq. 2-3; Sec. 3.2 / Algorithm 1 for the k / l / tau loops):
//
//   delta[k][l][s] = sum_n w_n S[s][k][n] j_l(k (tau0 - tau_n))
//
// One workgroup of W waves per k row, the largest k first.  The tau nodes go in
// slots of 64 (one node per lane), the multipoles in blocks of 16 rows counted
// from lmin.
//   * setup (all waves, slots dealt out): each node finds the pair w (j_R, j_{R+1})
//     at its top row R, the top row of the block that holds min(ltop(x), lmax).
//     For x >= lmax + 1 the upward recurrence from j_{-1} = cos x / x, j_0 =
//     sin x / x runs to R + 1 (stable on the oscillatory side; R is at most 15 rows
//     past lmax, and those rows are never stored).  Otherwise, for x >= kXDebye,
//     Debye's expansion gives the pair at Ls = max(ltop(x), R) and the recurrence
//     runs down to R; for smaller x the upward run goes to m = floor(x) for j_m, and
//     Miller's recurrence with seeds (0, 1) from Ls runs down to m and is scaled there
//     to j_m (j_m is near the last maximum in l, never near a zero).  The pair, 1/x and
//     the block of R go to LDS.
//   * sweep: wave w takes the blocks first - w, first - w - W, ... and walks all
//     slots that are live in its block, so the sums of a block over every node stay in
//     one wave's registers (16 x NSRC accumulators per lane).  For a slot it reads the
//     nodes' pairs from LDS, runs j_{l-1} = (2l+1)/x j_l - j_{l+1} down the 16 rows
//     (downward is stable above the turning point and neutral below it) and writes the
//     pairs back for the wave that owns the next lower block.  That wave follows one
//     slot or more behind: each wave publishes how far it is in LDS (prog), and waits
//     only when it has caught up with the wave above.
//   * a block's sums are reduced over the lanes once, by its wave, and stored.
//   * a row with at most half as many live blocks as waves (a small lmax, or the small k of
//     any grid) is swept by groups of waves, each taking all blocks over its share of the
//     slots; the groups' sums meet in LDS.  C2 1905 -> 1770 us, sampled 1455 -> 1355, the
//     tensor case 988 -> 949, C3 in FP32 7.19 -> 6.83 ms.
// Scalar registers are spilled (94 to 159 by variant), all of them in the setup and between
// blocks; 32 bytes of scratch a lane in the sampled variants.
// The upward runs of two slots side by side in a wave's setup were 2 to 5 % slower at every size:
// these runs are a small part of the setup.
// Why this split: the sweep is bound by FP64 VALU issue.  With the nodes of a row
// divided among the waves instead (each wave walking every block, the pairs in
// registers), every wave reduces every block over its lanes, which was 30 % of the
// VALU instructions, the unrolled slots take 220 registers (2 waves per SIMD), each
// block re-reads the row's sources from L2, and a short row keeps one wave busy for
// its whole length.  Here a block is reduced once, W blocks in flight share each
// slot's sources through the L1 cache, and a row of few slots still spreads over W
// waves.
//
// E-mode sources (bit s of emask; Sec. 2.1, Eq. 3: eps_l(x) =
// sqrt((l+2)!/(l-2)!) j_l(x) / x^2): their values are scaled by 1/x^2 per node
// as they are used and their output rows by sqrt((l-1) l (l+1) (l+2)); a node
// with x below kXTiny adds its limit w S sqrt(24)/15 to l = 2 only.
// Columns of x1mask / x2mask are scaled by 1/x / 1/x^2 per node with no row
// factor (the tensor-mode projection combines them afterwards); their x -> 0
// limits go to l = 1 (w S / 3) and l = 2 (w S / 15).  Column s reads source
// plane splane[s], so one source can feed several columns.
#pragma once

#include "bessel_dev.hpp"
#include "fp64_common.hpp"
#include "los_internal.hpp"

#include <type_traits>

namespace los {
namespace sweep {

using fp64::wave_max;
using fp64::wave_min;

constexpr int B = kSweepBlock;

// Most waves of a workgroup: their registers bound the waves a SIMD can hold.
constexpr int max_waves(int nsrc) { return nsrc <= 2 ? 16 : nsrc == 3 ? 12 : 8; }

// One slot over the block of rows top .. top-15, descending.  (p1, p0) =
// (w j_{l+1}, w j_l) at l = top on entry, at l = top - 16 on return.
template <int NSRC>
__device__ __forceinline__ void sweep_slot(double (&acc)[B * NSRC], double &p1, double &p0,
                                           double ix, const double (&sv)[NSRC], int top) {
  double t = 0.0;
  const double d2 = ix + ix;
#pragma unroll
  for (int i = 0; i < B; ++i) {
    // the coefficient (2l+1)/x is formed exactly every 8 rows and stepped by
    // -2/x in between (at most 7 rounding steps)
    if (i % 8 == 0) t = (double)(2 * (top - i) + 1) * ix;
    const int q = (B - 1 - i) * NSRC;
#pragma unroll
    for (int s = 0; s < NSRC; ++s) acc[q + s] = fma(p0, sv[s], acc[q + s]);
    const double nx = rec_step(t, p0, p1);
    p1 = p0;
    p0 = nx;
    t -= d2;
  }
}

// Sampled multipoles: C sampled rows of a block, off[r] rows below its top (uniform).  The
// recurrence alone runs through the block (2 FP64 instructions a row instead of 2 + NSRC), its
// 16 values stay in registers and the sampled ones are picked by a uniform index; no branch.
// C2 at 91 multipoles, one pass: 1.87 -> 1.46 ms against sweeping every block densely.  (A test
// per row in sweep_slot costs the compiler 300 spilled registers; runs from sample to sample
// with loops in between were no faster than the dense sweep: 80 scalar instructions and 20
// branches a slot.)
template <int NSRC, int C, int N>
__device__ __forceinline__ void sampled_slot(double (&acc)[N], double &p1,
                                             double &p0, double ix, const double (&sv)[NSRC],
                                             int top, const int (&off)[C ? C : 1]) {
  double t = 0.0, P[B];
  const double d2 = ix + ix;
#pragma unroll
  for (int i = 0; i < B; ++i) {
    if (i % 8 == 0) t = (double)(2 * (top - i) + 1) * ix;
    P[i] = p0;
    const double nx = rec_step(t, p0, p1);
    p1 = p0;
    p0 = nx;
    t -= d2;
  }
#pragma unroll
  for (int r = 0; r < C; ++r) {
    const double v = P[off[r]];
#pragma unroll
    for (int s = 0; s < NSRC; ++s) acc[r * NSRC + s] = fma(v, sv[s], acc[r * NSRC + s]);
  }
}

// Orders a wave's LDS accesses and keeps its lanes together: a wave's LDS operations are
// performed in order, so no wait is needed, but the compiler must neither move accesses
// across this point nor let one side of a divergent branch run ahead of it.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// NV values summed over a wave's lanes (16 NSRC for a whole block).  Two exchange steps
// (lanes 32 and 16 apart) leave NV / 4 values per lane, summed over 4 lanes; these go through
// the wave's LDS stage, [16][NV / H + 1] (the pad keeps both its accesses free of bank
// conflicts), in H rounds.  f(e, total) is called by the lane that holds the total of value e.  Two rounds
// (from 2 columns on) halve the stage, which decides how many waves fit a CU's LDS.
constexpr int reduce_rounds(int nv) { return nv <= 16 ? 1 : 2; }
constexpr int stage_doubles(int nsrc) { return 16 * (B * nsrc / reduce_rounds(B * nsrc) + 1); }

template <int NV, typename F>
__device__ __forceinline__ void reduce_block(double (&v)[NV], double *stage, int lane, F f) {
  constexpr int H = reduce_rounds(NV), P = NV / 4 / H, LD = NV / H + 1;
  static_assert(NV % (4 * H) == 0, "whole rounds");
  double u[NV / 2], q[NV / 4];
#pragma unroll
  for (int p = 0; p < NV / 2; ++p) u[p] = fp64::swap_add32(v[p], v[p + NV / 2]);
#pragma unroll
  for (int p = 0; p < NV / 4; ++p) q[p] = fp64::swap_add16(u[p], u[p + NV / 4]);
  // lane (r, c) now holds, for value p + r NV / 4, the sum over the 4 lanes of column c
  const int r = lane >> 4, c = lane & 15;
  double tot[H] = {};
#pragma unroll
  for (int h = 0; h < H; ++h) {
#pragma unroll
    for (int p = 0; p < P; ++p) stage[c * LD + r * P + p] = q[h * P + p];
    wave_sync();
    if (lane < 4 * P) {
#pragma unroll
      for (int cc = 0; cc < 16; ++cc) tot[h] += stage[cc * LD + lane];
    }
    wave_sync();
  }
  if (lane < 4 * P) {  // (f may write to the stage)
#pragma unroll
    for (int h = 0; h < H; ++h) f(lane / P * (NV / 4) + h * P + lane % P, tot[h]);
  }
}

// The members of a set of up to 128 slots in increasing order (uniform).
struct SlotList {
  uint64_t a, b;
  __device__ int pop() {  // the next one, or -1
    if (a) {
      const int s = __builtin_ctzll(a);
      a &= a - 1;
      return s;
    }
    if (b) {
      const int s = 64 + __builtin_ctzll(b);
      b &= b - 1;
      return s;
    }
    return -1;
  }
};

// T: type of the sources and of delta (float: the sources are widened as they are
// used, a pass's sums are FP64, and delta is rounded at the end of each pass, of which there
// are as many as the launch shape gives the tau axis).  SMP: multipole sampling.
// SC: the variant with per-column scalings (E-mode, 1/x, 1/x^2) and source planes;
// without it every column s reads plane s unscaled.
template <typename T, int NSRC, bool SMP, bool SC>
__global__ void __launch_bounds__(64 * max_waves(NSRC)) project_fp64_sweep_kernel(ProjectArgs a) {
  constexpr int NV = B * NSRC;
  extern __shared__ __attribute__((aligned(16))) double lds[];

  const int W = blockDim.x >> 6;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t ki = a.kend - 1 - (int64_t)blockIdx.x;  // large k (most work) first
  const int lmin = a.lmin, lmax = a.lmax;
  const int nblk = (a.nl + B - 1) / B;
  const int n0 = a.n0, ncnt = a.ncnt;  // this pass's nodes
  const int nslot = (ncnt + 63) >> 6, npad = nslot << 6;

  double *ixs = lds;                                // [npad] 1/x
  double2 *st = (double2 *)(ixs + npad);            // [npad] (w j_l, w j_{l+1}) at the next row
  double *stages = ixs + 3 * npad, *stage = stages + w * stage_doubles(NSRC);  // per wave
  short *rb = (short *)(stages + W * stage_doubles(NSRC));  // [npad] block of R
  short *th = rb + npad, *tf = th + nslot;          // per slot: live / every lane live up to here
  int *prog = (int *)(tf + nslot);                  // [W] progress of each wave

  const double kk = a.k[ki];
  const T *srow[NSRC];
#pragma unroll
  for (int s = 0; s < NSRC; ++s)
    srow[s] = (const T *)a.S + ((int64_t)(SC ? a.splane[s] : s) * a.nk + ki) * a.ntau + n0;

  // ---------------- per-node setup: the pair at the top row ----------------
  // Every node's top row R is the top row of a block, so in any block a lane is
  // either live throughout or not at all.  Rows between the band edge and R hold
  // values below the band cut; rows above lmax are swept but never stored.
  const int top_all = lmin + (lmax - lmin) / B * B + (B - 1);
  const bool lim1 = SC && a.x1mask != 0 && lmin <= 1;
  const bool lim2 = SC && (a.emask | a.x2mask) != 0 && lmin <= 2;
  constexpr int kTinyNode = -2;  // rb of a node below kXTiny with a limit term
  for (int s = w; s < nslot; s += W) {
    const int i = s * 64 + lane;
    const int nc = i < ncnt ? i : ncnt - 1, n = n0 + nc;
    // The slot's sources, so that the sweep finds them in L2: it loads them one slot ahead, and
    // with 3 and 4 columns too few waves share a SIMD to cover more.  Tensor case 901 -> 877 us,
    // sampled 1190 -> 1157; 3 columns, l <= 60, 4000 x 4096: 552 -> 502 (1 column, 1000 x 2500:
    // 94 -> 97, so not there).
    T ahead[NSRC];
    if (NSRC >= 3) {
#pragma unroll
      for (int q = 0; q < NSRC; ++q) ahead[q] = srow[q][nc];
    }
    const double x = kk * (a.tau0 - a.tau[n]), wn = a.w[n];
    const bool live = i < ncnt && x >= kXTiny && wn != 0.0;
    const bool tiny = i < ncnt && (lim1 || lim2) && x < kXTiny;
    const double ix = live ? 1.0 / x : 0.0;
    const int m = live ? (int)floor(x) : 0;
    const bool osc = m >= lmax + 1;  // every row up to R is on the oscillatory side
    int R = -1;
    double cur = 0.0, nxt = 0.0;
    if (live) {
      const int L0 = ltop_of(x);
      const int Rc = osc || L0 > lmax ? lmax : L0;  // last row kept (band edge or lmax)
      if (Rc >= lmin) {
        // top row of the block holding Rc; Debye's and Miller's seeds sit at or above it
        R = lmin + (Rc - lmin) / B * B + (B - 1);
        const int Ls = L0 > R ? L0 : R;
        if (!osc && x >= kXDebye) {
          double h[2];  // j_Ls, j_{Ls+1}
          debye_n<2>(Ls, x, ix, h);
          run_down(h[1], h[0], Ls, R, ix);
          cur = wn * h[0];
          nxt = wn * h[1];
        } else {
          double sn, cs;
          sincos(x, &sn, &cs);
          cur = wn * (cs * ix);  // w j_{-1}
          nxt = wn * (sn * ix);  // w j_0
          run_up(cur, nxt, 0, osc ? R + 1 : m, ix);
          if (!osc) {
            double hn = 0.0, hc = 1.0;  // Miller seeds (0, 1) at Ls
            run_down(hn, hc, Ls, R, ix);
            const double hR = hc, hR1 = hn;
            run_down(hn, hc, R, m, ix);
            const double sc = nxt / hc;  // w j_m / its Miller value
            cur = sc * hR;
            nxt = sc * hR1;
          }
        }
      }
    }
    const int b = R >= lmin ? (R - lmin) / B : -1;
    const int bmax = wave_max(b), bmin = wave_min(b);
    st[i] = make_double2(cur, nxt);
    ixs[i] = ix;
    rb[i] = (short)(tiny ? kTinyNode : b);
    if (lane == 0) {
      th[s] = (short)bmax;
      tf[s] = (short)bmin;
    }
    if (NSRC >= 3) {  // (keeps the loads)
#pragma unroll
      for (int q = 0; q < NSRC; ++q) asm volatile("" ::"v"(ahead[q]));
    }
  }
  if (lane == 0) prog[w] = 0;
  __syncthreads();

  // Slot thresholds, lane j holding slots j and 64 + j; the highest live block.
  const int th0 = lane < nslot ? th[lane] : -1, th1 = lane + 64 < nslot ? th[lane + 64] : -1;
  const int tf0 = lane < nslot ? tf[lane] : -1, tf1 = lane + 64 < nslot ? tf[lane + 64] : -1;
  int first = wave_max(th0 > th1 ? th0 : th1);

  T *drow = (T *)a.delta + ki * (int64_t)(SMP ? a.nls : a.nl) * NSRC;
  // output offset of row l = b + e / NSRC, source e % NSRC (-1: not stored)
  auto out_at = [&](int b, int e) -> int64_t {
    const int l = b + e / NSRC;
    if (l > lmax) return -1;
    if (!SMP) return (int64_t)(b - lmin) * NSRC + e;
    const int r = a.lsel[l - lmin];
    return r < 0 ? -1 : (int64_t)r * NSRC + e % NSRC;
  };
  // with limit terms, block 0 is summed even when no node reaches it
  if ((lim1 || lim2) && first < 0) first = 0;
  if (!a.accumulate) {  // blocks above every node's top row are zero
    for (int e = (first + 1) * NV + (int)threadIdx.x; e < nblk * NV; e += blockDim.x) {
      const int64_t o = out_at(lmin + e / NV * B, e % NV);
      if (o >= 0) drow[o] = (T)0;
    }
  }

  // ---------------- sweep ----------------
  // Few live blocks: the waves form G groups, each taking every block over its own slots
  // (s % G), and the groups' sums are added at the end.
  const int nlive = first + 1;
  const int G = nlive > 0 && 2 * nlive <= W ? W / nlive : 1;
  const int grp = G > 1 ? w / nlive : 0, wb = G > 1 ? w % nlive : w;
  const int stride = G > 1 ? nlive : W;
  const uint64_t mineA = G > 1 ? __ballot(lane % G == grp) : ~0ull;
  const uint64_t mineB = G > 1 ? __ballot((lane + 64) % G == grp) : ~0ull;
  // row l = b + e / NSRC, source e % NSRC, to its place in delta
  auto put = [&](int b, int e, double tot) {
    const int l = b + e / NSRC;
    if (SC && ((a.emask >> (e % NSRC)) & 1u))
      tot *= sqrt((double)(l - 1) * (double)l * (double)(l + 1) * (double)(l + 2));
    const int64_t o = out_at(b, e);
    if (o >= 0) drow[o] = (T)(a.accumulate ? tot + (double)drow[o] : tot);
  };
  const int pred = w > 0 ? w - 1 : W - 1;  // the wave that owns the block above
  int known = 0;                           // how far it is known to be
  int it = 0;
  const unsigned last = (unsigned)(ncnt - 1) * (unsigned)sizeof(T);
  for (int bi = grp < G ? first - wb : -1; bi >= 0; bi -= stride, ++it) {
    const int b = lmin + bi * B, top = b + B - 1;
    const SlotList slots{__ballot(th0 >= bi) & mineA, __ballot(th1 >= bi) & mineB};  // live in this block
    const uint64_t fullA = __ballot(tf0 >= bi), fullB = __ballot(tf1 >= bi);  // every lane live
    // progress the wave above must have reached for slot s: 128 a block, s + 1 within it;
    // the top block waits for nobody
    const int base = wb > 0 ? it * 128 : (it - 1) * 128;
    // Every live slot in order: body(p1, p0, ix, sv) takes the lane's pair through the block.
    // sum: it uses the sources.
    auto walk = [&](bool sum, auto body) {
      SlotList live = slots;
      auto load = [&](T (&sv)[NSRC], int s) {
        if (!sum) return;  // uniform
        unsigned off = (unsigned)(s * 64 + lane) * (unsigned)sizeof(T);
        off = off < last ? off : last;  // lanes past the end read the last node (not used)
#pragma unroll
        for (int q = 0; q < NSRC; ++q) sv[q] = *(const T *)((const char *)srow[q] + off);
      };
      auto step = [&](int s, const T (&raw)[NSRC], int snext) {
        if (wb > 0 || it > 0) {
          const int need = base + s + 1;
          while (known < need) {
            known = __builtin_amdgcn_readfirstlane(
                __hip_atomic_load(&prog[pred], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
            if (known < need) __builtin_amdgcn_s_sleep(1);
          }
          wave_sync();
        }
        const int i = s * 64 + lane;
        if ((((s < 64 ? fullA : fullB) >> (s & 63)) & 1u) || rb[i] >= bi) {  // the node is live
          const double2 pr = st[i];
          const double ix = ixs[i];
          double p0 = pr.x, p1 = pr.y;
          double sv[NSRC];
#pragma unroll
          for (int q = 0; q < NSRC; ++q) sv[q] = (double)raw[q];
          if (SC) {
            const double i2 = ix * ix;
#pragma unroll
            for (int q = 0; q < NSRC; ++q) {
              if (((a.emask | a.x2mask) >> q) & 1u) sv[q] *= i2;
              else if ((a.x1mask >> q) & 1u) sv[q] *= ix;
            }
          }
          body(p1, p0, ix, sv);
          st[i] = make_double2(p0, p1);
        }
        // the pairs are in place before the progress that announces them: every slot below
        // the next live one is done
        wave_sync();
        __hip_atomic_store(&prog[w], snext >= 0 ? it * 128 + snext : (it + 1) * 128,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      };
      // the next slot's sources are loaded while this one is swept
      T sa[NSRC] = {}, sb[NSRC] = {};
      int s = live.pop();
      if (s >= 0) load(sa, s);
      else  // a group's slots may all end below: nothing for the next block to wait for
        __hip_atomic_store(&prog[w], (it + 1) * 128, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
      while (s >= 0) {
        const int s2 = live.pop();
        if (s2 >= 0) load(sb, s2);
        step(s, sa, s2);
        if (s2 < 0) break;
        s = live.pop();
        if (s >= 0) load(sa, s);
        step(s2, sb, s);
      }
    };
    // Limits at x -> 0 of the scaled columns (the nodes below kXTiny are not swept), for
    // block 0: j_2(x)/x^2 -> 1/15 for E-mode and 1/x^2 columns at l = 2, j_1(x)/x -> 1/3
    // for 1/x columns at l = 1; every other row -> 0.  add(row, q, term), row = l - lmin.
    auto limits = [&](auto add) {
      if (!SC || bi != 0 || grp != 0 || !(lim1 || lim2)) return;
      const uint32_t m2 = a.emask | a.x2mask, m1 = a.x1mask;
      for (int sl = 0; sl < nslot; ++sl) {
        const int n = sl * 64 + lane;
        if (rb[n] != kTinyNode) continue;
        const double wn = a.w[n0 + n];
#pragma unroll
        for (int q = 0; q < NSRC; ++q) {
          if (lim2 && ((m2 >> q) & 1u)) add(2 - lmin, q, wn * (double)srow[q][n] * (1.0 / 15.0));
          if (lim1 && ((m1 >> q) & 1u)) add(1 - lmin, q, wn * (double)srow[q][n] * (1.0 / 3.0));
        }
      }
    };
    auto store = [&](int e, double tot) {
      if (G > 1) stage[e] = tot;  // uniform
      else put(b, e, tot);
    };
    const uint32_t rows = SMP ? __builtin_amdgcn_readfirstlane(a.bmask[bi]) : 0xffffu;
    const int nrow = __builtin_popcount(rows);
    if (SMP && nrow <= 4) {  // few sampled rows (uniform)
      auto few = [&](auto count) {
        constexpr int C = decltype(count)::value, C1 = C ? C : 1;
        constexpr int N = (C1 * NSRC + 3) / 4 * 4;  // (reduce_block takes multiples of 4)
        int off[C1] = {};
        uint32_t m = rows;  // bit r: row b + r
#pragma unroll
        for (int r = 0; r < C; ++r) {
          off[r] = m ? __builtin_clz(m) - (32 - B) : B - 1;
          m &= ~((1u << (B - 1)) >> off[r]);
        }
        double acc[N];
#pragma unroll
        for (int q = 0; q < N; ++q) acc[q] = 0.0;
        walk(C > 0, [&](double &p1, double &p0, double ix, const double (&sv)[NSRC]) {
          sampled_slot<NSRC, C>(acc, p1, p0, ix, sv, top, off);
        });
        if constexpr (C > 0) {
          limits([&](int row, int q, double term) {
#pragma unroll
            for (int r = 0; r < C; ++r)
              acc[r * NSRC + q] += r < nrow && off[r] == B - 1 - row ? term : 0.0;
          });
          reduce_block<N>(acc, stage, lane, [&](int e, double tot) {
            int o = off[0];
#pragma unroll
            for (int r = 1; r < C; ++r) o = e / NSRC == r ? off[r] : o;
            if (e / NSRC < nrow) store((B - 1 - o) * NSRC + e % NSRC, tot);
          });
        }
      };
      using std::integral_constant;
      if (nrow == 0) few(integral_constant<int, 0>{});
      else if (nrow == 1) few(integral_constant<int, 1>{});
      else few(integral_constant<int, 4>{});
    } else {
      double acc[NV];
#pragma unroll
      for (int q = 0; q < NV; ++q) acc[q] = 0.0;
      walk(true, [&](double &p1, double &p0, double ix, const double (&sv)[NSRC]) {
        sweep_slot<NSRC>(acc, p1, p0, ix, sv, top);
      });
      limits([&](int row, int q, double term) {  // row 0 or 1
        acc[q] += row == 0 ? term : 0.0;
        acc[NSRC + q] += row == 1 ? term : 0.0;
      });
      reduce_block<NV>(acc, stage, lane, store);
    }
  }
  if (G > 1) {  // uniform over the workgroup
    __syncthreads();
    for (int e = threadIdx.x; e < nlive * NV; e += blockDim.x) {
      const double *part = stages + e / NV * stage_doubles(NSRC) + e % NV;
      double tot = 0.0;
      for (int g = 0; g < G; ++g) tot += part[g * nlive * stage_doubles(NSRC)];
      put(lmin + (first - e / NV) * B, e % NV, tot);
    }
  }
}

}  // namespace sweep
}  // namespace los
