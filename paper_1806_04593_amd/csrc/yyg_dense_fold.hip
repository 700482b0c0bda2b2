// Dense FP64 solve folded about both mirror planes of a patch.
//
// On a grid symmetric about its equator (j -> n_t - 1 - j) and its central
// meridian (k -> n_p - 1 - k) every column of the two dense contractions is
// even or odd under each reflection: (-1)^(l + m) about the equator, + for
// cosines and - for sines about the meridian.  The other patch's harmonics,
// taken at the mapped points (x, y, z) -> (-x, z, y), are too, with the two
// parities in each other's place.  So each contraction splits into four over
// a quarter of the cells and a quarter of the columns each: a quarter of the
// products.  Class c = 2 (odd about the equator) + (odd about the meridian).
// The density is folded once before the analysis and the four classes'
// potentials are unfolded after the synthesis, each one pass over memory:
// 82 MB there and back at 2 degrees, 400 shells, 14 us each.  The four
// contractions of a side run in one launch (gemm_nt_f64_quad).
//
// Measured, a whole solve unfolded against folded (degree 25 at 2 degrees, 40
// at 1 degree): 2 degrees and 400 shells 642 and 187 us; 37 shells 301 and
// 48; 1 degree and 550 shells 5800 and 1600; 5 degrees, 50 shells, degree 8
// 75 and 27.  Folding the density in the contraction's own loads instead of
// a pass would fetch every cell once per class and column tile (four to
// twelve times) for the 14 us.  Low degrees save fewer products than the passes
// cost; which plans fold stands where they are made.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "yyg_internal.h"

namespace yyg {

namespace {

// F[c][row][j h_p + k] = the sum of the four mirror cells with class c's signs
// (a middle row or column meets itself: the bases halve it).
__global__ __launch_bounds__(256) void fold_rows_kernel(const double *__restrict__ rho, double *__restrict__ F, int nt,
                                                        int np, int ht, int hp, long stride) {
  const int row = blockIdx.y;
  const long a = (long)blockIdx.x * 256 + threadIdx.x;
  if (a >= (long)ht * hp) return;
  const int j = (int)(a / hp), k = (int)(a - (long)j * hp), jm = nt - 1 - j, km = np - 1 - k;
  const double *__restrict__ r = rho + (long)row * nt * np;
  const double x0 = r[(long)j * np + k], x1 = r[(long)j * np + km];
  const double y0 = r[(long)jm * np + k], y1 = r[(long)jm * np + km];
  const double pe = x0 + x1, po = x0 - x1, qe = y0 + y1, qo = y0 - y1;
  double *__restrict__ f = F + (long)row * ht * hp + a;
  f[0] = pe + qe;
  f[stride] = po + qo;
  f[2 * stride] = pe - qe;
  f[3 * stride] = po - qo;
}

// The four mirror cells of phi from the classes' potentials E[c][row][..].
__global__ __launch_bounds__(256) void unfold_rows_kernel(const double *__restrict__ E, double *__restrict__ phi,
                                                          int nt, int np, int ht, int hp, long stride) {
  const int row = blockIdx.y;
  const long a = (long)blockIdx.x * 256 + threadIdx.x;
  if (a >= (long)ht * hp) return;
  const int j = (int)(a / hp), k = (int)(a - (long)j * hp), jm = nt - 1 - j, km = np - 1 - k;
  const double *__restrict__ e = E + (long)row * ht * hp + a;
  const double e0 = e[0], e1 = e[stride], e2 = e[2 * stride], e3 = e[3 * stride];
  double *__restrict__ r = phi + (long)row * nt * np;
  const double s = e0 + e2, t = e1 + e3, u = e0 - e2, v = e1 - e3;
  r[(long)j * np + k] = s + t;
  if (km != k) r[(long)j * np + km] = s - t;
  if (jm != j) {
    r[(long)jm * np + k] = u + v;
    if (km != k) r[(long)jm * np + km] = u - v;
  }
}

// Folded analysis basis: row n (column q = cols[n] of class c) over the
// quarter's cells, the mean of the four mirror entries with their signs, a
// middle row or column halved.  The flag as below.
__global__ __launch_bounds__(256) void fold_analysis_basis_kernel(const double *__restrict__ Bt, long ldb,
                                                                  const int *__restrict__ cols, int c, int nt, int np,
                                                                  int ht, int hp, double *__restrict__ out, long ldo, int *__restrict__ flag) {
  const long a = (long)blockIdx.x * 256 + threadIdx.x;
  if (a >= ldo) return;
  double v = 0.0;
  if (a < (long)ht * hp) {
    const int j = (int)(a / hp), k = (int)(a - (long)j * hp), jm = nt - 1 - j, km = np - 1 - k;
    const double st = c & 2 ? -1.0 : 1.0, sp = c & 1 ? -1.0 : 1.0;
    const double *__restrict__ b = Bt + (long)cols[blockIdx.y] * ldb;
    const double v0 = b[(long)j * np + k];
    const double r0 = 1e-11 * fabs(v0) + 1e-14;  // entries are at most a cell's solid angle
    if (!(fabs(v0 - sp * b[(long)j * np + km]) <= r0 && fabs(v0 - st * b[(long)jm * np + k]) <= r0)) *flag = 1;
    v = 0.25 * ((b[(long)j * np + k] + sp * b[(long)j * np + km]) +
                st * (b[(long)jm * np + k] + sp * b[(long)jm * np + km]));
    v *= (jm == j ? 0.5 : 1.0) * (km == k ? 0.5 : 1.0);
  }
  out[(long)blockIdx.y * ldo + a] = v;
}

// Folded synthesis basis of one class: cell a of the quarter, column n = the
// unfolded basis' column ycols[n].  Where a mirror entry's magnitude or sign
// is off by more than 1e-11 (entries are O(1)) the flag is raised.
__global__ __launch_bounds__(256) void fold_synthesis_basis_kernel(const double *__restrict__ Y, long ldy,
                                                                   const int *__restrict__ ycols, int n, int c, int nt,
                                                                   int np, int ht, int hp, double *__restrict__ out,
                                                                   long ldo, int *__restrict__ flag) {
  const long a = blockIdx.x;
  const int j = (int)(a / hp), k = (int)(a - (long)j * hp), jm = nt - 1 - j, km = np - 1 - k;
  const double st = c & 2 ? -1.0 : 1.0, sp = c & 1 ? -1.0 : 1.0;
  for (int i = threadIdx.x; i < ldo; i += 256) {
    double v = 0.0;
    if (i < n) {
      const int q = ycols[i];
      v = Y[((long)j * np + k) * ldy + q];
      const double x = Y[((long)j * np + km) * ldy + q], y = Y[((long)jm * np + k) * ldy + q];
      if (!(fabs(v - sp * x) <= 1e-11 && fabs(v - st * y) <= 1e-11)) *flag = 1;
    }
    out[a * ldo + i] = v;
  }
}

}  // namespace

hipError_t launch_fold_rows(const double *rho, double *F, int rows, int nt, int np, hipStream_t s) {
  const int ht = (nt + 1) / 2, hp = (np + 1) / 2;
  const long cells = (long)ht * hp;
  if (rows <= 0) return hipSuccess;
  if (rows > 65535 || (cells + 255) / 256 > INT_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL(fold_rows_kernel, dim3((unsigned)((cells + 255) / 256), rows), dim3(256), 0, s, rho, F, nt, np, ht,
                     hp, rows * cells);
  return hipGetLastError();
}

hipError_t launch_unfold_rows(const double *E, double *phi, int rows, int nt, int np, hipStream_t s) {
  const int ht = (nt + 1) / 2, hp = (np + 1) / 2;
  const long cells = (long)ht * hp;
  if (rows <= 0) return hipSuccess;
  if (rows > 65535 || (cells + 255) / 256 > INT_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL(unfold_rows_kernel, dim3((unsigned)((cells + 255) / 256), rows), dim3(256), 0, s, E, phi, nt, np,
                     ht, hp, rows * cells);
  return hipGetLastError();
}

hipError_t launch_fold_analysis_basis(const double *Bt, long ldb, const int *cols, int n, int c, int nt, int np,
                                      double *out, long ldo, int *flag, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fold_analysis_basis_kernel, dim3((unsigned)((ldo + 255) / 256), n), dim3(256), 0, s, Bt, ldb, cols,
                     c, nt, np, (nt + 1) / 2, (np + 1) / 2, out, ldo, flag);
  return hipGetLastError();
}

hipError_t launch_fold_synthesis_basis(const double *Y, long ldy, const int *ycols, int n, int c, int nt, int np,
                                       double *out, long ldo, int *flag, hipStream_t s) {
  const int ht = (nt + 1) / 2, hp = (np + 1) / 2;
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fold_synthesis_basis_kernel, dim3((unsigned)((long)ht * hp)), dim3(256), 0, s, Y, ldy, ycols, n, c,
                     nt, np, ht, hp, out, ldo, flag);
  return hipGetLastError();
}

}  // namespace yyg
