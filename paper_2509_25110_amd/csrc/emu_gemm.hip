// FP32 matrix products of the emulator on the matrix cores: the network's layers (all members
// in one launch), their gradients, and the reconstruction of the spectra fused with the
// ensemble statistics.  Definitions of every quantity are in emu_api.cpp.
//
// Every output element is one chain of v_mfma_f32_16x16x4 in increasing k, four k at a time,
// from zero, whatever the tile: tiles change the speed only, never a bit of the result.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "emu_internal.hpp"

namespace los {
namespace emu {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ inline float gelu_f(float x) { return 0.5f * x * (1.f + erff(x * 0.70710678118654752f)); }
__device__ inline float gelu_grad_f(float x) {
  return 0.5f * (1.f + erff(x * 0.70710678118654752f)) +
         x * expf(-0.5f * x * x) * 0.39894228040143268f;
}

// An operand's tile of T rows (of A, or columns of B) by KT k in LDS: [row][KT + 4] when k is
// its contiguous axis, else [k][T + 16].  Both pitches keep the fragment reads (16 rows x 4 k)
// free of bank conflicts.  The tile moves in 16-byte pieces along the contiguous axis, F per
// thread; pieces that are not wholly inside, or not aligned, go element by element.
template <bool KC, int T, int KT, int NTH>
struct Operand {
  static constexpr int LD = KC ? KT + 4 : T + 16;
  static constexpr int size = KC ? T * LD : KT * LD;
  static constexpr int P = T * KT / 4, F = (P + NTH - 1) / NTH;
  // piece i of a thread exists (P may not fill the last round)
  __device__ static bool has(int i, int tid) { return P % NTH == 0 || i * NTH + tid < P; }

  __device__ static void at(int f, int &row, int &k) {
    if (KC) {
      row = f / (KT / 4);
      k = f % (KT / 4) * 4;
    } else {
      k = f / (T / 4);
      row = f % (T / 4) * 4;
    }
  }
  // X(row, k) = X[row * sr + k * sk]; rows r0 .. of `rows`, k0 .. of `K`; zeros outside
  __device__ static void load(f4 (&v)[F], const float *X, int64_t sr, int64_t sk, int64_t r0,
                              int64_t rows, int64_t k0, int64_t K, bool vec, int tid) {
#pragma unroll
    for (int i = 0; i < F; ++i) {
      if (!has(i, tid)) break;
      int row, k;
      at(i * NTH + tid, row, k);
      const int64_t r = r0 + row, kk = k0 + k;
      const float *p = X + r * sr + kk * sk;
      const bool in = KC ? r < rows && kk + 3 < K : r + 3 < rows && kk < K;
      if (vec && in) {
        v[i] = *(const f4 *)p;
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          v[i][u] = (KC ? r < rows && kk + u < K : r + u < rows && kk < K) ? p[u] : 0.f;
      }
    }
  }
  __device__ static void store(const f4 (&v)[F], float *lds, int tid) {
#pragma unroll
    for (int i = 0; i < F; ++i) {
      if (!has(i, tid)) break;
      int row, k;
      at(i * NTH + tid, row, k);
      *(f4 *)(lds + (KC ? row * LD + k : k * LD + row)) = v[i];
    }
  }
  __device__ static float get(const float *lds, int row, int k) {
    return KC ? lds[row * LD + k] : lds[k * LD + row];
  }
};

__host__ __device__ inline bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

// One workgroup's tile of C(m, n) = sum_k A(m, k) B(k, n): 4 waves in a 2 x 2 arrangement,
// each MB x MB blocks of 16 x 16.  Two LDS stages; the tile after next is loaded into
// registers while the matrix cores work on this one, one barrier per k tile.
// MB = 2 (64 x 64, 32 k) where that gives every CU its workgroups, MB = 1 (32 x 32, 64 k)
// where it does not: a layer of 512 x 512 for 256 rows is 32 or 128 workgroups.
template <int MB>
struct Tile {
  static constexpr int T = 32 * MB, KT = MB == 1 ? 64 : 32;
  template <bool AK, bool BK>
  static constexpr int floats() {
    return 2 * (Operand<AK, T, KT, 256>::size + Operand<BK, T, KT, 256>::size);
  }
};

template <bool AK, bool BK, int EPI, int MB>
__device__ __forceinline__ void gemm_tile(const GemmF32 &g, int bx, int by, int bz, float *lds) {
  constexpr int T = Tile<MB>::T, KT = Tile<MB>::KT;
  typedef Operand<AK, T, KT, 256> OA;
  typedef Operand<BK, T, KT, 256> OB;
  float *As = lds, *Bs = lds + 2 * OA::size;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int r16 = lane & 15, kq = lane >> 4;
  const int64_t mb = (int64_t)by * T, nb = (int64_t)bx * T;
  const int mw = (w >> 1) * (16 * MB), nw = (w & 1) * (16 * MB);
  const float *A = g.A + bz * g.a_bs, *Bp = g.B + bz * g.b_bs;
  const int64_t asr = AK ? g.sam : 1, ask = AK ? 1 : g.sak;
  const int64_t bsr = BK ? g.sbn : 1, bsk = BK ? 1 : g.sbk;
  const bool av = aligned16(A) && (AK ? asr : ask) % 4 == 0;
  const bool bv = aligned16(Bp) && (BK ? bsr : bsk) % 4 == 0;
  f4 ra[OA::F], rb[OB::F];
  f4 acc[MB][MB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < MB; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
  float rsum = 0.f;
  const bool sums = g.rowsum && bx == 0;  // uniform
  auto load = [&](int64_t k0) {
    OA::load(ra, A, asr, ask, mb, g.M, k0, g.K, av, tid);
    OB::load(rb, Bp, bsr, bsk, nb, g.N, k0, g.K, bv, tid);
  };
  load(0);
  OA::store(ra, As, tid);
  OB::store(rb, Bs, tid);
  if (KT < g.K) load(KT);
  __syncthreads();
  int st = 0;
  for (int64_t k0 = 0; k0 < g.K; k0 += KT, st ^= 1) {
    const float *a_ = As + st * OA::size, *b_ = Bs + st * OB::size;
    if (k0 + KT < g.K) {
      OA::store(ra, As + (st ^ 1) * OA::size, tid);
      OB::store(rb, Bs + (st ^ 1) * OB::size, tid);
      if (k0 + 2 * KT < g.K) load(k0 + 2 * KT);
    }
    const int kn = g.K - k0 < KT ? (int)(g.K - k0) : KT;
    auto products = [&](int kk) {
      float a[MB], b[MB];
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        a[i] = OA::get(a_, mw + 16 * i + r16, kk + kq);
        b[i] = OB::get(b_, nw + 16 * i + r16, kk + kq);
      }
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
    };
    if (kn == KT) {
#pragma unroll
      for (int kk = 0; kk < KT; kk += 4) products(kk);
    } else {
      for (int kk = 0; kk < kn; kk += 4) products(kk);
    }
    if (sums && tid < T)
      for (int kk = 0; kk < kn; ++kk) rsum += OA::get(a_, tid, kk);
    __syncthreads();
  }
  if (sums && tid < T && mb + tid < g.M) g.rowsum[mb + tid] = rsum;
  float *C = g.C + bz * g.c_bs;
  const float *bias = g.bias ? g.bias + bz * g.bias_bs : nullptr;
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < MB; ++j) {
      const int64_t n = nb + nw + 16 * j + r16;
      if (n >= g.N) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t m = mb + mw + 16 * i + 4 * kq + v;
        if (m >= g.M) continue;
        float x = acc[i][j][v];
        float *c = C + m * g.ldc + n;
        if (EPI == kEpiStore) {
          *c = x;
        } else if (EPI == kEpiBias) {
          *c = x + bias[n];
        } else if (EPI == kEpiBiasGelu) {  // keep the pre-activation in Z for the backward pass
          x += bias[n];
          if (g.Z) g.Z[m * g.ldc + n] = x;
          *c = gelu_f(x);
        } else if (EPI == kEpiBiasUnwhiten) {
          x += bias[n];
          *c = (float)((double)x * g.scale[n]);
        } else {  // kEpiGeluBack
          *c = x * gelu_grad_f(g.Z[m * g.ldc + n]);
        }
      }
    }
}

template <bool AK, bool BK, int EPI, int MB>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmF32 g) {
  __shared__ __attribute__((aligned(16))) float lds[Tile<MB>::template floats<AK, BK>()];
  gemm_tile<AK, BK, EPI, MB>(g, blockIdx.x, blockIdx.y, blockIdx.z, lds);
}

// A layer's weight gradient and the gradient of its input need each other for nothing: one
// launch, the first tw workgroups on the former.
template <int MB>
__global__ __launch_bounds__(256) void gemm_backward_kernel(GemmF32 dw, GemmF32 dx, int tw, int wx,
                                                            int xx) {
  constexpr int F0 = Tile<MB>::template floats<false, false>();
  constexpr int F1 = Tile<MB>::template floats<true, false>();
  __shared__ __attribute__((aligned(16))) float lds[F0 > F1 ? F0 : F1];
  const int b = blockIdx.x;
  if (b < tw) gemm_tile<false, false, kEpiStore, MB>(dw, b % wx, b / wx, 0, lds);
  else gemm_tile<true, false, kEpiGeluBack, MB>(dx, (b - tw) % xx, (b - tw) / xx, 0, lds);
}

// Tiles of a product at MB blocks a wave.
template <int MB>
int64_t tiles(const GemmF32 &g) {
  constexpr int T = Tile<MB>::T;
  return ((g.N + T - 1) / T) * ((g.M + T - 1) / T) * (g.batch > 1 ? g.batch : 1);
}

template <bool AK, bool BK, int EPI>
hipError_t launch_gemm(const GemmF32 &g, hipStream_t s) {
  const unsigned z = g.batch > 1 ? g.batch : 1;
  auto grid = [&](int t) {
    return dim3((unsigned)((g.N + t - 1) / t), (unsigned)((g.M + t - 1) / t), z);
  };
  // 64 x 64 tiles from two workgroups per CU on
  if (tiles<2>(g) >= 512)
    hipLaunchKernelGGL((gemm_f32_kernel<AK, BK, EPI, 2>), grid(64), dim3(256), 0, s, g);
  else
    hipLaunchKernelGGL((gemm_f32_kernel<AK, BK, EPI, 1>), grid(32), dim3(256), 0, s, g);
  return hipGetLastError();
}

// ------------------------------------------------ reconstruction and ensemble

// exp: (e^r - 1 - r) / r^2 on |r| <= ln 2 / 2, degree 10 (gen_exp.py); then sinh: 1 / k! for
// k = 3, 5, .. 17.
__constant__ const double kExpSinh[19] = {
    0.5, 0.16666666666666671, 0.041666666666666671, 0.0083333333333261411, 0.0013888888888883752,
    0.00019841269874800683, 2.4801587325533502e-05, 2.75572554255029e-06, 2.7557273661174726e-07,
    2.5105206475334834e-08, 2.091467944897855e-09,
    0.16666666666666666, 0.008333333333333333, 0.0001984126984126984, 2.7557319223985893e-06,
    2.505210838544172e-08, 1.6059043836821613e-10, 7.647163731819816e-13, 2.8114572543455206e-15};

// Uniform coefficients by scalar loads: as literals they would sit in vector registers.
typedef const __attribute__((address_space(4))) double *coef_ptr;
__device__ inline coef_ptr exp_sinh_coef() {
  coef_ptr p = (coef_ptr)(const double *)kExpSinh;
  asm volatile("" : "+s"(p));  // an address the compiler does not look through
  return p;
}

// e^y = (hi + lo) 2^n, hi = 1 + r rounded, |lo| < 0.07: y = n ln 2 + r, |r| <= ln 2 / 2, with ln 2
// as the sum of its first 42 bits (n times them is exact) and the next 53; r's own rounding
// error and the polynomial's terms, from r^2 on, go to lo.  Past +-800 e^y is inf or 0 as there.
__device__ __forceinline__ int exp_parts(float yf, coef_ptr c, double &hi, double &lo) {
  yf = yf > 800.f ? 800.f : yf;
  yf = yf < -800.f ? -800.f : yf;
  const double y = (double)yf, n = rint(y * 1.4426950408889634);
  const double r0 = fma(-n, 0x1.62e42fefa3800p-1, y);
  const double r = fma(-n, 0x1.ef35793c76730p-45, r0);
  const double rl = fma(-n, 0x1.ef35793c76730p-45, r0 - r);
  double q = c[10];
#pragma unroll
  for (int k = 9; k >= 0; --k) q = fma(q, r, c[k]);
  hi = 1.0 + r;
  lo = ((1.0 - hi) + r) + fma(r * r, q, rl);
  return (int)n;
}

// e^y: at most 0.64 units in the last place from it (the library's exp: 0.864), over 5.3 million
// arguments against 113 bits; overflows to inf, underflows to 0, NaN stays NaN.  About 2/3 of the
// library's instructions.
__device__ __forceinline__ double exp_f64(float y, coef_ptr c) {
  double hi, lo;
  const int n = exp_parts(y, c, hi, lo);
  return ldexp(hi + lo, n);
}

// sinh y: (e^|y| - e^-|y|) / 2 from |y| = 1 on, Taylor's polynomial below (next term below 9e-18
// of y; y^2 is exact, y having 24 bits).  At most 0.77 units in the last place (the library's,
// which forms e^y in double-double with 4 times the instructions: 0.858), as above.
__device__ __forceinline__ double sinh_f64(float yf, coef_ptr c) {
  double hi, lo;
  const int n = exp_parts(fabsf(yf), c, hi, lo);
  const double s = hi + lo;  // in [0.7, 1.42]: 1 / s by Newton's steps from an estimate
  double g = __builtin_amdgcn_rcp(s);
  g = fma(fma(-s, g, 1.0), g, g);
  g = fma(fma(-s, g, 1.0), g, g);
  const double big = ldexp(hi + (lo - ldexp(g, -2 * n)), n - 1);
  const double y = (double)yf, y2 = y * y;
  double p = c[18];
#pragma unroll
  for (int k = 17; k >= 11; --k) p = fma(p, y2, c[k]);
  return fabsf(yf) < 1.f ? fma(y * y2, p, y) : copysign(big, y);
}

struct Recon {
  const float *cz;     // [MEM][n][4 nc]
  const float *basis;  // [4][nl][nc]
  const float *mean;   // [4][nl]
  const double *t;     // [nl]
  double *cl;          // [n][4][nl]
  unsigned int *err;   // [n][4]
  int64_t n;
  int nl, nc, ctiles;  // ctiles: column tiles per workgroup
};

// Reconstruction y_e = mean + cz_e basis^T of every member, and the ensemble from it:
//   C_e = exp(y_e) (TE: t sinh(y_e)),  cl = member mean,
//   err = max over the multipoles and members of |C_e - cl| / scale
// (scale |cl|, TE sqrt(C_TT C_EE)) as float bits (an order-independent max).  A workgroup
// takes 16 WM rows by 32 WN multipoles (ctiles times), a wave 16 by 32 of them for all MEM
// members and one spectrum after the other, so the members' values meet in registers: kept in
// memory (16 FP32 values per row and multipole at 4 members) they were written once and read
// twice, and exp and sinh were taken twice.  The division by the scale is monotone, so the
// largest |C_e - cl| is divided once.
// Bound by the FP64 exp and sinh (VALU) beside the matrix cores: 4096 rows x 4999 multipoles
// x 4 members take 1.27 ms (1.66 ms with the library's exp and sinh; 1.22 ms with exp and sinh
// that were less accurate than these), three waves a SIMD at the price of 23 spilled registers
// (96 bytes of scratch a lane); two waves were 0.13 ms slower.
template <int MEM, int WM, int WN, int NB, int KT>
__global__ __launch_bounds__(256, 3) void reconstruct_kernel(Recon a) {
  constexpr int TM = 16 * WM, TN = 16 * NB * WN, LD = KT + 4;
  typedef Operand<true, MEM * TM, KT, 256> OA;
  typedef Operand<true, TN, KT, 256> OB;
  __shared__ __attribute__((aligned(16))) float As[OA::size];
  __shared__ __attribute__((aligned(16))) float Bs[OB::size];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int r16 = lane & 15, kq = lane >> 4;
  const int wm = w % WM, wn = w / WM;
  const int64_t row0 = (int64_t)blockIdx.x * TM;
  const int nout = 4 * a.nc;
  const bool vec = a.nc % 4 == 0 && aligned16(a.cz) && aligned16(a.basis);
  const int64_t m0 = row0 + 16 * wm + 4 * kq;  // the lane's rows m0 .. m0 + 3
  unsigned int worst[4][4] = {};               // [spectrum][row], float bits
  for (int ct = 0; ct < a.ctiles; ++ct) {
    const int64_t col0 = ((int64_t)blockIdx.y * a.ctiles + ct) * TN;
    if (col0 >= a.nl) break;  // uniform
    double keep[NB][4];  // TT mean, then the TE scale
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) keep[j][v] = 0.0;
#pragma unroll 1
    for (int sp = 0; sp < 4; ++sp) {
      f4 acc[MEM][NB];
#pragma unroll
      for (int e = 0; e < MEM; ++e)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[e][j] = f4{0.f, 0.f, 0.f, 0.f};
      f4 ra[OA::F], rb[OB::F];
      auto load = [&](int k0) {
        // row e TM + i of the A tile is row row0 + i of member e
#pragma unroll
        for (int i = 0; i < OA::F; ++i) {
          if (!OA::has(i, tid)) break;
          int row, k;
          OA::at(i * 256 + tid, row, k);
          const int e = row / TM;
          const int64_t r = row0 + row % TM;
          const float *p = a.cz + ((int64_t)e * a.n + r) * nout + sp * a.nc + k0 + k;
          if (vec && r < a.n && k0 + k + 3 < a.nc) {
            ra[i] = *(const f4 *)p;
          } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) ra[i][u] = r < a.n && k0 + k + u < a.nc ? p[u] : 0.f;
          }
        }
        OB::load(rb, a.basis + (int64_t)sp * a.nl * a.nc, a.nc, 1, col0, a.nl, k0, a.nc, vec, tid);
      };
      load(0);
      for (int k0 = 0; k0 < a.nc; k0 += KT) {
        __syncthreads();  // the previous tile is consumed
        OA::store(ra, As, tid);
        OB::store(rb, Bs, tid);
        __syncthreads();
        if (k0 + KT < a.nc) load(k0 + KT);
        const int kn = a.nc - k0 < KT ? a.nc - k0 : KT;
        for (int kk = 0; kk < kn; kk += 4) {
          float b[NB];
#pragma unroll
          for (int j = 0; j < NB; ++j) b[j] = Bs[(16 * (NB * wn + j) + r16) * LD + kk + kq];
#pragma unroll
          for (int e = 0; e < MEM; ++e) {
            const float x = As[(e * TM + 16 * wm + r16) * LD + kk + kq];
#pragma unroll
            for (int j = 0; j < NB; ++j)
              acc[e][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, b[j], acc[e][j], 0, 0, 0);
          }
        }
      }
      // the spectrum's values: TE as t sinh(y), the others as exp(y)
      auto finish = [&](auto te) {
        constexpr bool TE = decltype(te)::value;
        const coef_ptr ck = exp_sinh_coef();
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const int64_t l = col0 + 16 * (NB * wn + j) + r16;
          const bool inl = l < a.nl;
          const float mu = inl ? a.mean[(int64_t)sp * a.nl + l] : 0.f;
          const double tl = TE && inl ? a.t[l] : 0.0;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const bool in = inl && m0 + v < a.n;
            if (!__any(in)) continue;
            double c[MEM], mean = 0.0;
#pragma unroll
            for (int e = 0; e < MEM; ++e) {
              const float y = acc[e][j][v] + mu;
              c[e] = TE ? tl * sinh_f64(y, ck) : exp_f64(y, ck);
              mean += c[e];
            }
            mean /= MEM;
            double scale = fabs(mean);
            if (TE) scale = keep[j][v];
            else if (sp == 0) keep[j][v] = mean;
            else if (sp == 1) keep[j][v] = sqrt(keep[j][v] * mean);
            double d = 0.0;
#pragma unroll
            for (int e = 0; e < MEM; ++e) d = fmax(d, fabs(c[e] - mean));
            d = fmax(0.0, d / scale);
            if (in) {
              a.cl[((m0 + v) * 4 + sp) * a.nl + l] = mean;
              const unsigned int bits = __float_as_uint((float)d);
              // (worst[sp] with sp a constant: the array stays in registers)
#pragma unroll
              for (int q = 0; q < 4; ++q)
                if (q == sp) worst[q][v] = bits > worst[q][v] ? bits : worst[q][v];
            }
          }
        }
      };
      if (sp == 2) finish(std::true_type{});
      else finish(std::false_type{});
    }
  }
  // the 16 lanes of a row, then one atomic per row and spectrum
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      unsigned int x = worst[q][v];
#pragma unroll
      for (int o = 8; o >= 1; o >>= 1) {
        const unsigned int y = __shfl_xor(x, o, 64);
        x = y > x ? y : x;
      }
      if (r16 == 0 && m0 + v < a.n) atomicMax(a.err + (m0 + v) * 4 + q, x);
    }
}

template <int MEM>
hipError_t launch_recon(Recon a, hipStream_t s) {
  // few rows: 16 rows by 64 multipoles a workgroup (3 rows, 2499 multipoles: call 97.7 us, by 128
  // 104.2); else 32 by 64, and several column tiles per workgroup (fewer atomics) as long as
  // every CU has four workgroups
  if (a.n <= 16) {
    a.ctiles = 1;
    hipLaunchKernelGGL((reconstruct_kernel<MEM, 1, 4, 1, 32>), dim3(1, (unsigned)((a.nl + 63) / 64)),
                       dim3(256), 0, s, a);
    return hipGetLastError();
  }
  const int64_t rt = (a.n + 31) / 32, cts = (a.nl + 63) / 64;
  a.ctiles = (int)std::min<int64_t>(16, std::max<int64_t>(1, rt * cts / 1024));
  hipLaunchKernelGGL((reconstruct_kernel<MEM, 2, 2, 2, 32>),
                     dim3((unsigned)rt, (unsigned)((cts + a.ctiles - 1) / a.ctiles)), dim3(256), 0, s,
                     a);
  return hipGetLastError();
}

}  // namespace

hipError_t gemm_f32(const GemmF32 &g, int epi, hipStream_t s) {
  if (g.sak != 1 || g.sbk != 1) return hipErrorInvalidValue;
  switch (epi) {
    case kEpiBias: return launch_gemm<true, true, kEpiBias>(g, s);
    case kEpiBiasGelu: return launch_gemm<true, true, kEpiBiasGelu>(g, s);
    case kEpiBiasUnwhiten: return launch_gemm<true, true, kEpiBiasUnwhiten>(g, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t gemm_backward(const GemmF32 &dw, const GemmF32 &dx, hipStream_t s) {
  if (dw.sam != 1 || dw.sbn != 1 || dx.sak != 1 || dx.sbn != 1) return hipErrorInvalidValue;
  const int64_t big = tiles<2>(dw) + tiles<2>(dx);
  const bool two = big >= 512;
  const int T = two ? 64 : 32;
  const int64_t tw = two ? tiles<2>(dw) : tiles<1>(dw), tx = two ? tiles<2>(dx) : tiles<1>(dx);
  if (tw + tx > 0x7fffffff) return hipErrorInvalidValue;
  const int wx = (int)((dw.N + T - 1) / T), xx = (int)((dx.N + T - 1) / T);
  if (two)
    hipLaunchKernelGGL(gemm_backward_kernel<2>, dim3((unsigned)(tw + tx)), dim3(256), 0, s, dw, dx,
                       (int)tw, wx, xx);
  else
    hipLaunchKernelGGL(gemm_backward_kernel<1>, dim3((unsigned)(tw + tx)), dim3(256), 0, s, dw, dx,
                       (int)tw, wx, xx);
  return hipGetLastError();
}

hipError_t reconstruct_ensemble(const float *cz, int members, int64_t n, int nl, int ncomp,
                                const float *basis, const float *mean, const double *t,
                                double *cl, unsigned int *err_bits, hipStream_t s) {
  if ((n + 31) / 32 > 0x7fffffff) return hipErrorInvalidValue;
  const Recon a{cz, basis, mean, t, cl, err_bits, n, nl, ncomp, 1};
  switch (members) {
    case 1: return launch_recon<1>(a, s);
    case 2: return launch_recon<2>(a, s);
    case 3: return launch_recon<3>(a, s);
    case 4: return launch_recon<4>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace emu
}  // namespace los
