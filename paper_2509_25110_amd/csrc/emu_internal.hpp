// Internal declarations of the C_l emulator kernels (emu_kernels.hip) used by
// its host code (emu_api.cpp).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace los {
namespace emu {

constexpr int kEpiStore = 0;         // C = A B
constexpr int kEpiBias = 1;          // C = A B + bias[n]
constexpr int kEpiBiasGelu = 2;      // Z = A B + bias[n] (kept if Z is given), C = GELU(Z)
constexpr int kEpiBiasUnwhiten = 3;  // C = (A B + bias[n]) scale[n] (the product in FP64)
constexpr int kEpiGeluBack = 4;      // C = (A B) GELU'(Z)
constexpr int kMaxQ = 112;           // largest PCA subspace (ncomp + oversampling)
constexpr int kMaxFused = 4;         // most members of the fused reconstruction

// A(m, k) = A[m * sam + k * sak], B(k, n) = B[k * sbk + n * sbn], each with one of its two
// strides 1; C(m, n) = C[m * ldc + n] (and Z likewise).  `batch` such products, operand X of
// the b-th at X + b * x_bs (bias and scale too; scale is shared).  rowsum (or NULL):
// rowsum[m] = sum_k A(m, k), in increasing k.
struct GemmF32 {
  int64_t M, N, K;
  const float *A;
  int64_t sam, sak;
  const float *B;
  int64_t sbk, sbn;
  float *C;
  int64_t ldc;
  const float *bias;
  float *Z;
  int batch;  // 0 counts as 1
  int64_t a_bs, b_bs, c_bs, bias_bs;
  const double *scale;
  float *rowsum;
};
struct GemmF64 {
  int64_t M, N, K;
  const double *A;
  int64_t sam, sak;
  const double *B;
  int64_t sbk, sbn;
  double *C;
  int64_t ldc;
};

hipError_t gemm_f32(const GemmF32 &g, int epi, hipStream_t s);
// Backward of a layer in one launch: dw (kEpiStore, A and B contiguous along M and N) and dx
// (kEpiGeluBack, A contiguous along K, B along N).
hipError_t gemm_backward(const GemmF32 &dw, const GemmF32 &dx, hipStream_t s);
hipError_t gemm_f64(const GemmF64 &g, hipStream_t s);
hipError_t mse_grad(const float *out, const float *z, int64_t cnt, float *G, float *partial,
                    float *loss, int accumulate, hipStream_t s);
hipError_t adam(float *w, const float *g, float *m, float *v, int64_t n, float lr, int64_t t,
                hipStream_t s);
hipError_t gather_rows(const float *src, const int64_t *idx, int64_t rows, int64_t cols,
                       float *dst, hipStream_t s);
// u = 2 (p - lo) / (hi - lo) - 1; err_bits (or NULL): 4 n words set to 0.
hipError_t scale_params(const double *p, int64_t n, int np, const double *lo, const double *hi,
                        float *u, unsigned int *err_bits, hipStream_t s);
hipError_t transform(const double *cl, int64_t n, int nl, const double *t, double *y,
                     hipStream_t s);
hipError_t te_median(const double *cl, int64_t n, int nl, double *t, hipStream_t s);
hipError_t center(double *X, int64_t rows, int64_t cols, int64_t ld, double *mean, hipStream_t s);
// R^T R = G + shift_rel * trace(G) * I; Rinv = R^{-1}.
hipError_t chol_inv(const double *G, int q, double shift_rel, double *Rinv, int *status,
                    hipStream_t s);
hipError_t jacobi_eig(const double *A, int q, int sweeps, double *V, double *evals, double *U,
                      hipStream_t s);
hipError_t whiten(const double *c, int64_t n, int ncomp, int s_idx, int nout, double *sigma,
                  float *z, hipStream_t s);
// Member mean into cl and the largest deviations into err_bits (4 n words, zeroed before).
hipError_t ensemble(const float *y, int members, int64_t n, int nl, const double *t, double *cl,
                    unsigned int *err_bits, hipStream_t s);
// The same from the members' coefficients cz[e][r][4 ncomp]: reconstruction (basis [4][nl]
// [ncomp], mean [4][nl]) and ensemble in one kernel; members <= kMaxFused.
hipError_t reconstruct_ensemble(const float *cz, int members, int64_t n, int nl, int ncomp,
                                const float *basis, const float *mean, const double *t,
                                double *cl, unsigned int *err_bits, hipStream_t s);
// Estimates and flags from err_bits: per row (err, flag) and / or per (row, spectrum) (err4,
// flag4), any of them NULL.
hipError_t flags(const unsigned int *err_bits, int64_t n, float thr, float *err,
                 unsigned char *flag, float *err4, unsigned char *flag4, hipStream_t s);
// cl[rows[i]][*] = src[i][*] (row_len values each), err[rows[i]] = 0, flag[rows[i]] = 0
// (err, flag may be NULL); rows in [0, n) and distinct (checked by the caller).
hipError_t merge_rows(const int64_t *rows, int64_t nf, const double *src, int64_t row_len,
                      double *cl, float *err, unsigned char *flag, hipStream_t s);
// cl[rows[i]][spec][*] = src[i][*] (nl values each), err4 / flag4 of (rows[i], spec) = 0.
hipError_t merge_spectrum(const int64_t *rows, int64_t nf, const double *src, int nl, int spec,
                          double *cl, float *err4, unsigned char *flag4, hipStream_t s);

}  // namespace emu
}  // namespace los
