// Theta transforms and moment rotation of the separable form with their
// operands loaded straight from memory: every intermediate keeps the row
// (patch, shell) contiguous, so 16 rows of one column are a 128-byte run and
// four columns of 16 rows the B operand of v_mfma_f64_16x16x4 as they lie.
//
// The colatitudes are mirror-symmetric about the equator (j -> n_t - 1 - j)
// and T_j^(lm), P_l^m(cos t_j) gain (-1)^(l + m), so each theta transform
// folds: the sum of a mirror pair meets the degrees with l + m even, the
// difference those with l + m odd, over h = ceil(n_t / 2) rows.
//
// The rotation block D_l between the patches maps (x, y, z) -> (-x, z, y):
// a harmonic's parity in x is kept, those in y and z trade places.  So the
// columns of a degree fall into four classes (cos / sin, m even / odd), and
// each class of this patch takes moments of one class of the other patch
// only: a quarter of D_l's products.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>

#include "yyg_internal.h"

namespace yyg {

namespace {

typedef double dbl4t __attribute__((ext_vector_type(4)));
typedef double dbl2t __attribute__((ext_vector_type(2), aligned(16)));

// Analysis of azimuthal column mc: A[l^2 + mc][row] = sum_j T_j X2[mc][j][row].
// A block holds the column's folded basis in LDS, in operand order; each
// wave walks row tiles of 16 rows and loads the next four steps (16 mirror
// pairs) while it multiplies the last four; the products are basis x data,
// so that a store covers 16 consecutive rows.  Every X2 value is read once
// (the tiles read it once per 32 degrees).  Bound by that stream (within whole
// solves, median of 20 traced): 1000 shells at half a degree, lmax 64 (443 MB)
// 136 us in 32 x 32 tiles, 105 here (4.2 TB/s); 800 shells, 180 colatitudes,
// lmax 80 (227 MB) 89 in 32 x 32 tiles, 81 in the best, 59 here (3.8);
// launched alone, its operands in the last-level cache, 46.
template <int T>
__device__ __forceinline__ void theta_ana_sweep(const ThetaArgs &a, const double *Bs, int mc, int m, int ng, int t_beg,
                                                int t_end, int nw) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  int t = t_beg + wave;
  if (t >= t_end) return;
  const double *__restrict__ const col = a.X2 + (long)mc * a.MJ;
  // byte-free element offsets of a step's rows; padding steps repeat the last
  double ra[4], rb[4];
  auto load = [&](int tile, int n) {
    const double *__restrict__ p = col + min(tile * 16 + r16, a.Mr - 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int j = min(16 * n + 4 * i + g, a.h - 1);
      ra[i] = p[(long)j * a.Mr];
      rb[i] = p[(long)(a.nt - 1 - j) * a.Mr];
    }
  };
  load(t, 0);
  for (; t < t_end; t += nw) {
    dbl4t ae[T], ao[T];
#pragma unroll
    for (int k = 0; k < T; ++k) ae[k] = ao[k] = dbl4t{0.0, 0.0, 0.0, 0.0};
    for (int n = 0; n < ng; ++n) {
      double e[4], o[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        e[i] = ra[i] + rb[i];
        o[i] = ra[i] - rb[i];
      }
      __builtin_amdgcn_sched_barrier(0);
      // the next steps, or the first of this wave's next row tile
      const bool last = n + 1 == ng;
      load(last ? min(t + nw, t_end - 1) : t, last ? 0 : n + 1);
#pragma unroll
      for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
        for (int k = 0; k < T; ++k) {
          const double *__restrict__ q = Bs + (((2 * n + i2) * 2) * T + k) * 128 + 2 * lane;
          const dbl2t be = *reinterpret_cast<const dbl2t *>(q), bo = *reinterpret_cast<const dbl2t *>(q + T * 128);
          ae[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(be.x, e[2 * i2], ae[k], 0, 0, 0);
          ao[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(bo.x, o[2 * i2], ao[k], 0, 0, 0);
          ae[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(be.y, e[2 * i2 + 1], ae[k], 0, 0, 0);
          ao[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(bo.y, o[2 * i2 + 1], ao[k], 0, 0, 0);
        }
    }
    const int row = t * 16 + r16;
#pragma unroll
    for (int k = 0; k < T; ++k)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int l = m + 2 * (16 * k + g + 4 * r);
        if (row < a.Mr && l <= a.L) a.Ahat[((long)l * l + mc) * a.Mr + row] = ae[k][r];
        if (row < a.Mr && l + 1 <= a.L) a.Ahat[((long)(l + 1) * (l + 1) + mc) * a.Mr + row] = ao[k][r];
      }
  }
}

// One block: the row tiles of `chunk` (of `chunks`) of column mc.  NW waves,
// TM the most 16-degree tiles a parity holds (m = 0).
template <int TM, int NW>
__device__ __forceinline__ void theta_ana_block(const ThetaArgs &a, double *Bs, int mc, int chunk, int chunks) {
  const int m = (mc + 1) >> 1;
  const int ng = (a.h + 15) / 16, T = ((a.L - m) / 2 + 16) / 16;  // even degrees l = m, m + 2, ..: (L - m) / 2 + 1
  const dbl2t *__restrict__ src = reinterpret_cast<const dbl2t *>(a.TA + (long)m * a.sta);
  for (int e = threadIdx.x; e < ng * 4 * T * 64; e += 64 * NW) *reinterpret_cast<dbl2t *>(Bs + 2 * e) = src[e];
  __syncthreads();
  const int tiles = (a.Mr + 15) / 16, t_beg = (int)((long)tiles * chunk / chunks);
  const int t_end = (int)((long)tiles * (chunk + 1) / chunks);
  if (T == 1)
    theta_ana_sweep<1>(a, Bs, mc, m, ng, t_beg, t_end, NW);
  else if (TM >= 2 && T == 2)
    theta_ana_sweep<(TM >= 2 ? 2 : 1)>(a, Bs, mc, m, ng, t_beg, t_end, NW);
  else if (TM >= 3)
    theta_ana_sweep<(TM >= 3 ? 3 : 1)>(a, Bs, mc, m, ng, t_beg, t_end, NW);
}

template <int TM, int NW>
__global__ __launch_bounds__(64 * NW) void theta_ana_stream(ThetaArgs a, int chunks) {
  extern __shared__ __attribute__((aligned(16))) double Bs[];
  const int mc = blockIdx.x / chunks;
  theta_ana_block<TM, NW>(a, Bs, mc, blockIdx.x - mc * chunks, chunks);
}

// The same over the columns of several plans: items (plan, column, chunk,
// chunks), one a block.  24 plans of 100 to 600 shells at 2 to 4 degrees, lmax
// 10 to 30: analysis 65 us in tiles, 60 here; synthesis 78, 57; rotation 63,
// 40.
template <int TM, int NW>
__global__ __launch_bounds__(64 * NW) void theta_ana_group(const ThetaArgs *__restrict__ args,
                                                           const int4 *__restrict__ items) {
  extern __shared__ __attribute__((aligned(16))) double Bs[];
  const int4 it = items[blockIdx.x];
  const ThetaArgs a = args[it.x];
  theta_ana_block<TM, NW>(a, Bs, it.y, it.z, it.w);
}

// Synthesis of azimuthal column mc: V[mc][j][row] = sum_l P_l^m(t_j)
// Ut[mc][l][row].  A block holds the column's folded basis in LDS; each wave
// walks row tiles, a tile's coefficients (KQ steps of four degrees per
// parity) in registers and the next tile's on their way, and stores 16 rows
// of each colatitude and of its mirror.  Same sizes as above: 152 us in
// 64 x 32 tiles, 139 in the best tile, 98 here (4.5 TB/s); 88, 84 and 69 (3.3).
template <int KQ, int NW>
__device__ __forceinline__ void theta_syn_block(const ThetaArgs &a, double *Bs, int mc, int chunk, int chunks) {
  const int m = (mc + 1) >> 1;
  const int kp = ((a.L - m) / 2 + 8) / 8;  // pairs of steps: ceil(((L - m) / 2 + 1) / 8)
  const int jt = (a.h + 15) / 16;
  const dbl2t *__restrict__ src = reinterpret_cast<const dbl2t *>(a.TS + (long)m * a.sts);
  for (int e = threadIdx.x; e < jt * 2 * kp * 64; e += 64 * NW) *reinterpret_cast<dbl2t *>(Bs + 2 * e) = src[e];
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const int tiles = (a.Mr + 15) / 16, t_beg = (int)((long)tiles * chunk / chunks);
  const int t_end = (int)((long)tiles * (chunk + 1) / chunks);
  int t = t_beg + wave;
  if (t >= t_end) return;
  constexpr int KP = (KQ + 1) / 2;
  double ue[2 * KP], uo[2 * KP], ne[2 * KP], no[2 * KP];
  // degrees past L repeat it (their basis is zero)
  auto load = [&](int tile, double (&e)[2 * KP], double (&o)[2 * KP]) {
    const double *__restrict__ p = a.Ut + (long)mc * (a.L + 1) * a.Mr + min(tile * 16 + r16, a.Mr - 1);
#pragma unroll
    for (int q = 0; q < 2 * KP; ++q)
      if (q < 2 * kp) {  // uniform
        const int l = m + 2 * (4 * q + g);
        e[q] = p[(long)min(l, a.L) * a.Mr];
        o[q] = p[(long)min(l + 1, a.L) * a.Mr];
      }
  };
#pragma unroll
  for (int q = 0; q < 2 * KP; ++q) ne[q] = no[q] = 0.0;
  load(t, ne, no);
  for (; t < t_end; t += NW) {
#pragma unroll
    for (int q = 0; q < 2 * KP; ++q) {
      ue[q] = ne[q];
      uo[q] = no[q];
    }
    load(min(t + NW, t_end - 1), ne, no);
    const int row = t * 16 + r16;
    double *__restrict__ const out = a.V + (long)mc * a.MJ + row;
    for (int k = 0; k < jt; ++k) {
      dbl4t ae = dbl4t{0.0, 0.0, 0.0, 0.0}, ao = ae;
#pragma unroll
      for (int p = 0; p < KP; ++p)
        if (p < kp) {  // uniform
          const double *__restrict__ q = Bs + ((k * kp + p) * 2) * 128 + 2 * lane;
          const dbl2t be = *reinterpret_cast<const dbl2t *>(q), bo = *reinterpret_cast<const dbl2t *>(q + 128);
          ae = __builtin_amdgcn_mfma_f64_16x16x4f64(be.x, ue[2 * p], ae, 0, 0, 0);
          ao = __builtin_amdgcn_mfma_f64_16x16x4f64(bo.x, uo[2 * p], ao, 0, 0, 0);
          ae = __builtin_amdgcn_mfma_f64_16x16x4f64(be.y, ue[2 * p + 1], ae, 0, 0, 0);
          ao = __builtin_amdgcn_mfma_f64_16x16x4f64(bo.y, uo[2 * p + 1], ao, 0, 0, 0);
        }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int j = 16 * k + g + 4 * r, jm = a.nt - 1 - j;
        if (row < a.Mr && j < a.h) {
          out[(long)j * a.Mr] = ae[r] + ao[r];
          if (jm != j) out[(long)jm * a.Mr] = ae[r] - ao[r];
        }
      }
    }
  }
}

template <int KQ, int NW>
__global__ __launch_bounds__(64 * NW) void theta_syn_stream(ThetaArgs a, int chunks) {
  extern __shared__ __attribute__((aligned(16))) double Bs[];
  const int mc = blockIdx.x / chunks;
  theta_syn_block<KQ, NW>(a, Bs, mc, blockIdx.x - mc * chunks, chunks);
}

template <int KQ, int NW>
__global__ __launch_bounds__(64 * NW) void theta_syn_group(const ThetaArgs *__restrict__ args,
                                                           const int4 *__restrict__ items) {
  extern __shared__ __attribute__((aligned(16))) double Bs[];
  const int4 it = items[blockIdx.x];
  const ThetaArgs a = args[it.x];
  theta_syn_block<KQ, NW>(a, Bs, it.y, it.z, it.w);
}

// column (within its degree) of member i of class c: 0 cos m = 2 i, 1 cos
// m = 2 i + 1, 2 sin m = 2 i + 2, 3 sin m = 2 i + 1
__device__ __forceinline__ int class_column(int c, int i) {
  return c == 0 ? max(4 * i - 1, 0) : c == 1 ? 4 * i + 1 : c == 2 ? 4 * i + 4 : 4 * i + 2;
}

// Buffer descriptor of `bytes` from a uniform address: a load at or past the
// end gives zero, a store there is dropped.
typedef unsigned u32x2t __attribute__((ext_vector_type(2)));
constexpr unsigned kNoMember = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t theta_buffer(const double *p, long bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(p), 0, (int)min(bytes, 0x7fffffffL), 0x00020000);
}

// Rotation of degree l: At[l^2 + b][p nR + n] = A_own(n, b) + sum_k
// A_other(n, k) D_l[k][b].  Of the four classes two map onto themselves and
// two onto each other; a block takes one of these three units for both
// patches and a run of row tiles, its blocks of D_l in LDS in operand order.
// A wave loads a row tile's members once (16 shells; lane group g, value q =
// member 4 q + g): they are the B operand for the other patch and, value
// 4 t + r being element r of output tile t, the accumulators' start for
// their own.  So the moments are read once and written once (the tiles read
// them twice): 1000 shells, lmax 64 (135 MB) 67 us in tiles, 45 here (3.0 TB/s;
// launched alone 35, and 59 with a wave per class and patch).  At most KQ steps of four members, NT tiles of 16.
template <int NT, int KQ>
__device__ __forceinline__ void rotation_block(const ThetaArgs &a, double *Ds, int l, int unit, int run, int runs) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  // l even: classes 1 and 2 trade, 0 and 3 stay; l odd: 0 and 3 trade
  const bool odd = l & 1, pair = unit == 0;
  const int c0 = pair ? (odd ? 0 : 1) : unit == 1 ? (odd ? 1 : 0) : (odd ? 2 : 3);
  const int c1 = pair ? (odd ? 3 : 2) : c0;
  const int nb = c0 == 0 ? l / 2 + 1 : c0 == 2 ? l / 2 : (l + 1) / 2;  // members; c1 has as many
  if (nb == 0) return;
  const int kq = (nb + 3) / 4, nt = (nb + 15) / 16;
  for (int e = threadIdx.x; e < nt * kq * 64; e += 256) {
    Ds[e] = a.DR[(4L * l + c0) * a.std + e];
    if (pair) Ds[nt * kq * 64 + e] = a.DR[(4L * l + c1) * a.std + e];
  }
  __syncthreads();
  const int tiles = (a.nR + 15) / 16, t_beg = (int)((long)tiles * run / runs), t_end = (int)((long)tiles * (run + 1) / runs);
  unsigned m0[KQ], m1[KQ];
#pragma unroll
  for (int q = 0; q < KQ; ++q) {
    const int k = 4 * q + g;
    m0[q] = k < nb ? 8u * ((unsigned)class_column(c0, k) * (unsigned)a.Mr + r16) : kNoMember;
    m1[q] = k < nb ? 8u * ((unsigned)class_column(c1, k) * (unsigned)a.Mr + r16) : kNoMember;
  }
  const long base = (long)l * l * a.Mr, bytes = 8L * (2 * l + 1) * a.Mr;
  for (int tile = t_beg + wave; tile < t_end; tile += 4) {
    // x[class][patch][q]
    double x[2][2][KQ];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const long at = (long)p * a.nR + tile * 16;
      const auto rs = theta_buffer(a.Ahat + base + at, bytes - 8 * at);
#pragma unroll
      for (int q = 0; q < KQ; ++q) {
        x[0][p][q] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, m0[q], 0, 0));
        if (pair) x[1][p][q] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, m1[q], 0, 0));
      }
    }
    const bool in = tile * 16 + r16 < a.nR;
    // outputs of class c from its own members (own) and the other patch's (oth)
    auto turn = [&](const double (&own)[2][KQ], const double (&oth)[2][KQ], const double *D, const unsigned (&m)[KQ]) {
      dbl4t acc[2][NT];
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[p][t][r] = 4 * t + r < KQ ? own[p][4 * t + r < KQ ? 4 * t + r : 0] : 0.0;
#pragma unroll
      for (int q = 0; q < KQ; ++q)
        if (q < kq)  // uniform
#pragma unroll
          for (int t = 0; t < NT; ++t)
            if (t < nt) {
              const double d = D[(t * kq + q) * 64 + lane];
              acc[0][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(d, oth[1][q], acc[0][t], 0, 0, 0);
              acc[1][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(d, oth[0][q], acc[1][t], 0, 0, 0);
            }
      if (in)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const long at = (long)p * a.nR + tile * 16;
          const auto rs = theta_buffer(a.At + base + at, bytes - 8 * at);
#pragma unroll
          for (int q = 0; q < KQ; ++q)
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2t, (double)acc[p][q / 4][q % 4]), rs, m[q], 0, 0);
        }
    };
    if (pair) {
      turn(x[0], x[1], Ds, m0);
      turn(x[1], x[0], Ds + nt * kq * 64, m1);
    } else {
      turn(x[0], x[0], Ds, m0);
    }
  }
}

template <int NT, int KQ>
__global__ __launch_bounds__(256, KQ <= 9 ? 3 : 2) void rotation_stream(ThetaArgs a, int runs) {
  extern __shared__ __attribute__((aligned(16))) double Ds[];
  // largest degrees first, the unit of two classes (twice the work) first
  const int run = blockIdx.x % runs, unit = (blockIdx.x / runs) % 3;
  rotation_block<NT, KQ>(a, Ds, a.L - blockIdx.x / (3 * runs), unit, run, runs);
}

// items (plan, 3 degree + unit, run, runs)
template <int NT, int KQ>
__global__ __launch_bounds__(256, KQ <= 9 ? 3 : 2) void rotation_group(const ThetaArgs *__restrict__ args,
                                                                       const int4 *__restrict__ items) {
  extern __shared__ __attribute__((aligned(16))) double Ds[];
  const int4 it = items[blockIdx.x];
  const ThetaArgs a = args[it.x];
  rotation_block<NT, KQ>(a, Ds, it.y / 3, it.y % 3, it.z, it.w);
}

int even_tiles(int L) { return (L / 2 + 16) / 16; }

constexpr int kGroupWaves = 4;  // waves of a batch's theta blocks

// blocks of the theta kernels: chunks of row tiles per column, each of them
// whole passes of the block's waves, about three blocks per CU
int theta_chunks(const ThetaArgs &a, int nw, int cus) {
  const int tiles = (a.Mr + 15) / 16, nmc = 2 * a.L + 1;
  return std::max(1, std::min((tiles + nw - 1) / nw, (3 * cus + nmc - 1) / nmc));
}

template <int NW>
hipError_t launch_theta_ana_w(const ThetaArgs &a, int cus, hipStream_t s) {
  const int chunks = theta_chunks(a, NW, cus);
  const dim3 grid((2 * a.L + 1) * chunks), block(64 * NW);
  const size_t lds = theta_ana_doubles(a.L, a.h) * sizeof(double);
  switch (even_tiles(a.L)) {
    case 1: hipLaunchKernelGGL((theta_ana_stream<1, NW>), grid, block, lds, s, a, chunks); break;
    case 2: hipLaunchKernelGGL((theta_ana_stream<2, NW>), grid, block, lds, s, a, chunks); break;
    case 3: hipLaunchKernelGGL((theta_ana_stream<3, NW>), grid, block, lds, s, a, chunks); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

int theta_steps(int L) {
  const int n = L / 8 + 1;
  return n <= 2 ? 2 : n <= 4 ? 4 : n <= 6 ? 6 : n <= 10 ? 10 : n <= 12 ? 12 : -1;
}

template <int NW>
hipError_t launch_theta_syn_w(const ThetaArgs &a, int cus, hipStream_t s) {
  const int chunks = theta_chunks(a, NW, cus);
  const dim3 grid((2 * a.L + 1) * chunks), block(64 * NW);
  const size_t lds = theta_syn_doubles(a.L, a.h) * sizeof(double);
  switch (theta_steps(a.L)) {
    case 2: hipLaunchKernelGGL((theta_syn_stream<2, NW>), grid, block, lds, s, a, chunks); break;
    case 4: hipLaunchKernelGGL((theta_syn_stream<4, NW>), grid, block, lds, s, a, chunks); break;
    case 6: hipLaunchKernelGGL((theta_syn_stream<6, NW>), grid, block, lds, s, a, chunks); break;
    case 10: hipLaunchKernelGGL((theta_syn_stream<10, NW>), grid, block, lds, s, a, chunks); break;
    case 12: hipLaunchKernelGGL((theta_syn_stream<12, NW>), grid, block, lds, s, a, chunks); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// tiles and steps of the largest class, L / 2 + 1 members
void rotation_shape(int L, int *nt, int *kq) {
  const int nb = L / 2 + 1;
  *kq = nb <= 8 ? 2 : nb <= 16 ? 4 : nb <= 24 ? 6 : nb <= 36 ? 9 : 12;
  *nt = (*kq + 3) / 4;
}

hipError_t launch_rotation(const ThetaArgs &a, int wide, int cus, hipStream_t s) {
  const int tiles = (a.nR + 15) / 16, units = 3 * (a.L + 1);
  const int runs = std::max(1, std::min((tiles + 3) / 4, (4 * wide * cus + units - 1) / units));
  const dim3 grid(units * runs), block(256);
  const size_t lds = 2 * (size_t)a.std * sizeof(double);
  int nt, kq;
  rotation_shape(a.L, &nt, &kq);
  switch (kq) {
    case 2: hipLaunchKernelGGL((rotation_stream<1, 2>), grid, block, lds, s, a, runs); break;
    case 4: hipLaunchKernelGGL((rotation_stream<1, 4>), grid, block, lds, s, a, runs); break;
    case 6: hipLaunchKernelGGL((rotation_stream<2, 6>), grid, block, lds, s, a, runs); break;
    case 9: hipLaunchKernelGGL((rotation_stream<3, 9>), grid, block, lds, s, a, runs); break;
    default: hipLaunchKernelGGL((rotation_stream<3, 12>), grid, block, lds, s, a, runs); break;
  }
  return hipGetLastError();
}

}  // namespace

size_t theta_ana_doubles(int L, int h) { return (size_t)((h + 15) / 16) * 4 * even_tiles(L) * 128; }
size_t theta_syn_doubles(int L, int h) { return (size_t)((h + 15) / 16) * 2 * ((L / 2 + 8) / 8) * 128; }

size_t rotation_doubles(int L) {
  const int nb = L / 2 + 1;
  return (size_t)((nb + 15) / 16) * ((nb + 3) / 4) * 64;
}

bool theta_stream_fits(int phase, int L, int h) {
  if (L > 94) return false;
  const size_t lds = phase == 1 ? theta_ana_doubles(L, h) : phase == 3 ? theta_syn_doubles(L, h) : 0;
  return lds * sizeof(double) <= 160 * 1024;
}

hipError_t launch_theta_stream(int phase, int variant, const ThetaArgs &a, int cus, hipStream_t s) {
  if (a.Mr <= 0 || a.nt <= 0) return hipSuccess;
  switch (phase) {
    case 1: return variant ? launch_theta_ana_w<4>(a, cus, s) : launch_theta_ana_w<8>(a, cus, s);
    case 2: return launch_rotation(a, variant ? 2 : 1, cus, s);
    case 3: return variant ? launch_theta_syn_w<4>(a, cus, s) : launch_theta_syn_w<8>(a, cus, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_theta_group(int phase, int L, size_t lds, const ThetaArgs *args, const int4 *items, int n_items,
                              hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  const dim3 grid(n_items), block(phase == 2 ? 256 : 64 * kGroupWaves);
  int nt, kq;
  rotation_shape(L, &nt, &kq);
#define YYG_COMMA ,
#define YYG_GROUP(K)                                                            \
  do {                                                                          \
    hipLaunchKernelGGL((K), grid, block, lds, s, args, items);                  \
    return hipGetLastError();                                                   \
  } while (0)
  if (phase == 1) switch (even_tiles(L)) {
      case 1: YYG_GROUP(theta_ana_group<1 YYG_COMMA kGroupWaves>);
      case 2: YYG_GROUP(theta_ana_group<2 YYG_COMMA kGroupWaves>);
      case 3: YYG_GROUP(theta_ana_group<3 YYG_COMMA kGroupWaves>);
    }
  if (phase == 2) switch (kq) {
      case 2: YYG_GROUP(rotation_group<1 YYG_COMMA 2>);
      case 4: YYG_GROUP(rotation_group<1 YYG_COMMA 4>);
      case 6: YYG_GROUP(rotation_group<2 YYG_COMMA 6>);
      case 9: YYG_GROUP(rotation_group<3 YYG_COMMA 9>);
      case 12: YYG_GROUP(rotation_group<3 YYG_COMMA 12>);
    }
  if (phase == 3) switch (theta_steps(L)) {
      case 2: YYG_GROUP(theta_syn_group<2 YYG_COMMA kGroupWaves>);
      case 4: YYG_GROUP(theta_syn_group<4 YYG_COMMA kGroupWaves>);
      case 6: YYG_GROUP(theta_syn_group<6 YYG_COMMA kGroupWaves>);
      case 10: YYG_GROUP(theta_syn_group<10 YYG_COMMA kGroupWaves>);
      case 12: YYG_GROUP(theta_syn_group<12 YYG_COMMA kGroupWaves>);
    }
#undef YYG_GROUP
#undef YYG_COMMA
  return hipErrorInvalidValue;
}

int theta_stream_kernel_name(int phase, int variant, const ThetaArgs &a, char *buf, size_t n) {
  const int nw = variant ? 4 : 8;
  int r = -1, nt, kq;
  rotation_shape(a.L, &nt, &kq);
  if (phase == 1) r = snprintf(buf, n, "yyg::(anonymous namespace)::theta_ana_stream<%d, %d>", even_tiles(a.L), nw);
  if (phase == 2) r = snprintf(buf, n, "yyg::(anonymous namespace)::rotation_stream<%d, %d>", nt, kq);
  if (phase == 3) r = snprintf(buf, n, "yyg::(anonymous namespace)::theta_syn_stream<%d, %d>", theta_steps(a.L), nw);
  return r < 0 ? -1 : 0;
}

}  // namespace yyg
