// Phi transforms of the separable form folded about two meridians.
//
// A row of azimuthal cells is mirror-symmetric about the patch's central
// meridian (k -> np - 1 - k: cosines even, sines odd), and on every grid
// whose spacing divides 180 degrees into whole cells also about the
// meridians 90 degrees off it (k -> cc - k on the front half: cos m gains
// (-1)^m, sin m gains -(-1)^m).  Over the cells within 90 degrees of the
// centre (fold index t, front cell f0 + t) the transform then splits into
// four sums of a quarter of the columns each: cosines of even m, cosines of
// odd m, sines of even m, sines of odd m.  Cells without a partner
// (t >= T2: the row ends before 90 degrees past them) enter all four with
// their own value; without any partners (T2 = 0) the four sums are the
// even / odd halves of the single fold, split by the parity of m.
//
// Arithmetic per row and colatitude: (2L + 1) K multiply-adds, K = 180 of
// 542 cells at half a degree (271 folded once), K = np / 4 on the polar grid.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdio>
#include <initializer_list>
#include <type_traits>

#include "yyg_internal.h"

namespace yyg {

namespace {

typedef double dbl4q __attribute__((ext_vector_type(4)));
typedef double dbl2q __attribute__((ext_vector_type(2), aligned(8)));   // rows start at any double
typedef double dbl2a __attribute__((ext_vector_type(2), aligned(16)));

// Contiguous runs of work per XCD (blocks are handed to the 8 XCDs
// round-robin), so that neighbouring rows meet in one L2.
__device__ __forceinline__ int quad_xcd(int b, int total) {
  const int per = total / 8, rem = total % 8, x = b & 7;
  return x * per + min(x, rem) + (b >> 3);
}

// Buffer descriptor of `bytes` (at most 2^31) from a uniform address: 32-bit
// lane offsets, and an access at or past the end reads zero or is dropped,
// so a lane without a place to store carries kNoPlace as its offset.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr unsigned kNoPlace = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const double *p, long bytes) {
  const int n = (int)max(0L, min(bytes, 0x7fffffffL));
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(p), 0, n, 0x00020000 /* 32-bit data format */);
}

// azimuthal column of output o of group gr, and its order m
__device__ __forceinline__ int quad_order(int gr, int o) { return 2 * o + (gr == 0 ? 0 : gr == 2 ? 2 : 1); }
__device__ __forceinline__ int quad_column(int gr, int m) { return gr < 2 ? max(2 * m - 1, 0) : 2 * m; }

constexpr int kAnaLdp = 18;  // a folded row of 16 points in LDS

// Analysis sweep, one row tile per wave: 16 (patch, shell) rows of one
// colatitude, every azimuthal column, so that a density value is read once.
// A stage is 16 folded points.  Its density loads cover 128 contiguous bytes
// of 8 rows each (lane = row, pair of points; loaded straight into the
// operand layout every lane would touch a line of its own, and the address
// unit took 45 cycles per load instead of 16); each lane folds its points in
// registers and passes the folded values to the operand layout through LDS
// of the wave's own.  The basis (the same for every colatitude) passes
// through LDS in operand order, shared by the block's waves, double-buffered
// with one barrier per stage.  Stages without partners (t >= T2) load and
// fold two places only.
// `lds`: phi_ana_quad_lds doubles.  TJ tiles of 16 outputs per group; XC: the even cosines number 16 TJ + 1
// and the last one is summed on the vector units.
template <int TJ, bool XC, int NW, bool WGT>
__device__ __forceinline__ void phi_ana_quad_tiles(const PhiQuadArgs &a, int blk, double *lds) {
  constexpr int NT = 64 * NW, CH = 4 * TJ * 256 + (XC ? 16 : 0), NB = (CH / 2 + NT - 1) / NT, LDP = kAnaLdp;
  double *const Bs[2] = {lds, lds + CH};
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r16 = lane & 15;   // operand layout
  const int lr = lane >> 3, lt = 2 * (lane & 7);  // load layout: rows lr and lr + 8, points lt and lt + 1
  const int total = a.nt * ((a.Mr + 15) / 16);
  const int want = blk * NW + wave, id = min(want, total - 1);
  const int rt = id / a.nt, j = id - rt * a.nt;
  const double *__restrict__ px0 = a.X + (long)min(rt * 16 + lr, a.Mr - 1) * a.ld + (long)j * a.np;
  const double *__restrict__ px1 = a.X + (long)min(rt * 16 + lr + 8, a.Mr - 1) * a.ld + (long)j * a.np;
  const double *__restrict__ pw = a.W + (long)j * 2 * a.Kp + lt;
  double *__restrict__ const ps = lds + 2 * CH + wave * 64 * LDP;

  dbl4q acc[4][TJ];
#pragma unroll
  for (int gr = 0; gr < 4; ++gr)
#pragma unroll
    for (int tj = 0; tj < TJ; ++tj) acc[gr][tj] = dbl4q{0.0, 0.0, 0.0, 0.0};
  double xacc = 0.0;

  dbl2q ra[2], rb[2], rc[2], rd[2], wa, wc;
  dbl2a br[NB];
  // the pairs of stage s; clamped pairs stay inside the row and their values
  // are dropped in the fold
  auto load = [&](int s) {
    const int t = min(16 * s + lt, a.K - 1);
    const int oa = a.f0 + t, ob = a.np - 2 - a.f0 - t;
    ra[0] = *reinterpret_cast<const dbl2q *>(px0 + oa);
    ra[1] = *reinterpret_cast<const dbl2q *>(px1 + oa);
    rb[0] = *reinterpret_cast<const dbl2q *>(px0 + ob);
    rb[1] = *reinterpret_cast<const dbl2q *>(px1 + ob);
    if constexpr (WGT) wa = *reinterpret_cast<const dbl2q *>(pw + 16 * s);
  };
  auto load_partners = [&](int s) {
    const int t = min(16 * s + lt, a.K - 1);
    const int oc = max(a.cc - a.f0 - t - 1, 0), od = min(a.np - 1 - a.cc + a.f0 + t, a.np - 2);
    rc[0] = *reinterpret_cast<const dbl2q *>(px0 + oc);
    rc[1] = *reinterpret_cast<const dbl2q *>(px1 + oc);
    rd[0] = *reinterpret_cast<const dbl2q *>(px0 + od);
    rd[1] = *reinterpret_cast<const dbl2q *>(px1 + od);
    if constexpr (WGT) wc = *reinterpret_cast<const dbl2q *>(pw + a.Kp + 16 * s);
  };
  auto bload = [&](int s) {
    const dbl2a *__restrict__ b = reinterpret_cast<const dbl2a *>(a.bas + (long)s * CH);
#pragma unroll
    for (int i = 0; i < NB; ++i) br[i] = b[min(tid + i * NT, CH / 2 - 1)];
  };
  auto bstash = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (CH / 2 >= (i + 1) * NT || tid + i * NT < CH / 2) *reinterpret_cast<dbl2a *>(&Bs[buf][2 * (tid + i * NT)]) = br[i];
  };
  // the descending places hold their pair in reverse
  auto fold = [&](int s, auto paired) {
    const int t = 16 * s + lt;
    const bool i0 = t >= a.tlo && t < a.K, i1 = t + 1 >= a.tlo && t + 1 < a.K;
    const bool c0 = i0 && t < a.T2, c1 = i1 && t < a.T2;  // T2 is even
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      double p[2], m[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const bool in = i ? i1 : i0;
        const double A = in ? ra[h][i] : 0.0, B = in ? rb[h][1 - i] : 0.0;
        p[i] = WGT ? (A + B) * wa[i] : A + B;
        m[i] = WGT ? (A - B) * wa[i] : A - B;
      }
      double *o = ps + (lr + 8 * h) * LDP + lt;
      if constexpr (decltype(paired)::value) {
        double q[2], n[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const bool in = i ? c1 : c0;
          const double C = in ? rc[h][1 - i] : 0.0, D = in ? rd[h][i] : 0.0;
          q[i] = WGT ? (C + D) * wc[i] : C + D;
          n[i] = WGT ? (C - D) * wc[i] : C - D;
        }
        *reinterpret_cast<dbl2a *>(o) = dbl2a{p[0] + q[0], p[1] + q[1]};
        *reinterpret_cast<dbl2a *>(o + 16 * LDP) = dbl2a{p[0] - q[0], p[1] - q[1]};
        *reinterpret_cast<dbl2a *>(o + 32 * LDP) = dbl2a{m[0] - n[0], m[1] - n[1]};
        *reinterpret_cast<dbl2a *>(o + 48 * LDP) = dbl2a{m[0] + n[0], m[1] + n[1]};
      } else {
        *reinterpret_cast<dbl2a *>(o) = dbl2a{p[0], p[1]};
        *reinterpret_cast<dbl2a *>(o + 32 * LDP) = dbl2a{m[0], m[1]};
      }
    }
  };
  auto compute = [&](int buf, auto paired) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      dbl2a e[4];
#pragma unroll
      for (int gr = 0; gr < 4; ++gr) {
        if (!decltype(paired)::value && (gr & 1))
          e[gr] = e[gr - 1];
        else
          e[gr] = *reinterpret_cast<const dbl2a *>(ps + gr * 16 * LDP + r16 * LDP + 4 * g + 2 * h);
      }
#pragma unroll
      for (int gr = 0; gr < 4; ++gr)
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj) {
          const dbl2a b = *reinterpret_cast<const dbl2a *>(&Bs[buf][((gr * TJ + tj) * 2 + h) * 128 + 2 * lane]);
          acc[gr][tj] = __builtin_amdgcn_mfma_f64_16x16x4f64(b.x, e[gr].x, acc[gr][tj], 0, 0, 0);
          acc[gr][tj] = __builtin_amdgcn_mfma_f64_16x16x4f64(b.y, e[gr].y, acc[gr][tj], 0, 0, 0);
        }
      if constexpr (XC) {
        const dbl2a x = *reinterpret_cast<const dbl2a *>(&Bs[buf][4 * TJ * 256 + 4 * g + 2 * h]);
        xacc = __builtin_fma(x.x, e[0].x, xacc);
        xacc = __builtin_fma(x.y, e[0].y, xacc);
      }
    }
  };

  // paired stages first, then the rest; each stage's loads are issued a
  // stage ahead (ahead: 0 none, 1 the stage's own places, 2 with partners;
  // fixed per loop, since waits behind a conditional load count all loads)
  const int sp = (a.T2 + 15) / 16;
  auto step = [&](int s, auto paired, auto ahead) {
    constexpr int AH = decltype(ahead)::value;
    if constexpr (AH > 0) bload(s + 1);
    fold(s, paired);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (AH > 0) load(s + 1);
    if constexpr (AH > 1) load_partners(s + 1);
    compute(s & 1, paired);
    if constexpr (AH > 0) {
      bstash((s + 1) & 1);
      __syncthreads();
    }
  };
  using yes = std::true_type;
  using no = std::false_type;
  bload(0);
  load(0);
  if (sp > 0) load_partners(0);
  bstash(0);
  __syncthreads();
  int s = 0;
  for (; s + 1 < sp; ++s) step(s, yes{}, std::integral_constant<int, 2>{});
  if (s < sp) {
    if (s + 1 < a.S)
      step(s, yes{}, std::integral_constant<int, 1>{});
    else
      step(s, yes{}, std::integral_constant<int, 0>{});
    ++s;
  }
  for (; s + 1 < a.S; ++s) step(s, no{}, std::integral_constant<int, 1>{});
  if (s < a.S) step(s, no{}, std::integral_constant<int, 0>{});

  // D layout: lane l, element r -> output l / 16 + 4 r of the tile, row l % 16
  const int row = rt * 16 + r16;
  const bool live = want < total && row < a.Mr;
  double *__restrict__ out = a.C + (long)j * a.Mr + row;
#pragma unroll
  for (int gr = 0; gr < 4; ++gr)
#pragma unroll
    for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = quad_order(gr, 16 * tj + g + 4 * r);
        if (live && m <= a.L) out[(long)quad_column(gr, m) * a.MJ] = acc[gr][tj][r];
      }
  if constexpr (XC) {
    xacc += __shfl_xor(xacc, 16);
    xacc += __shfl_xor(xacc, 32);
    if (live && g == 0) out[(long)(2 * a.L - 1) * a.MJ] = xacc;
  }
}

constexpr int phi_ana_quad_lds(int TJ, bool XC, int NW) { return 2 * (4 * TJ * 256 + (XC ? 16 : 0)) + NW * 64 * kAnaLdp; }

template <int TJ, bool XC, int NW, bool WGT>
__global__ __launch_bounds__(64 * NW, TJ == 1 ? 3 : TJ < 4 ? 2 : 1) void phi_ana_quad(PhiQuadArgs a) {
  __shared__ __attribute__((aligned(16))) double lds[phi_ana_quad_lds(TJ, XC, NW)];
  phi_ana_quad_tiles<TJ, XC, NW, WGT>(a, quad_xcd(blockIdx.x, gridDim.x), lds);
}

// The sweep over several plans of up to TM tiles of outputs per group: items
// (plan, block of the plan, shape: 4 tiles + 2 extra output + 1 weights), one
// a block.  Bound by the density's stream and its latency: 24 plans of 100 to
// 600 shells at 2 to 4 degrees, lmax 10 to 30 (0.72 GB there and back, 145 us
// at the copy's rate): tiles folded once 248 us, here 204 with two waves a
// block, 197 with four; the form with the basis in registers, its blocks
// shared out among the plans, 252.
template <int TM, int NW>
__global__ __launch_bounds__(64 * NW, TM == 1 ? 3 : 2) void phi_ana_group(const PhiQuadArgs *__restrict__ args,
                                                                         const int4 *__restrict__ items) {
  __shared__ __attribute__((aligned(16))) double lds[phi_ana_quad_lds(TM, true, NW)];
  const int4 it = items[blockIdx.x];
  const PhiQuadArgs a = args[it.x];
  switch (it.z) {  // uniform
    case 4: phi_ana_quad_tiles<1, false, NW, false>(a, it.y, lds); break;
    case 5: phi_ana_quad_tiles<1, false, NW, true>(a, it.y, lds); break;
    case 6: phi_ana_quad_tiles<1, true, NW, false>(a, it.y, lds); break;
    case 7: phi_ana_quad_tiles<1, true, NW, true>(a, it.y, lds); break;
  }
  if constexpr (TM >= 2) switch (it.z) {
      case 8: phi_ana_quad_tiles<2, false, NW, false>(a, it.y, lds); break;
      case 9: phi_ana_quad_tiles<2, false, NW, true>(a, it.y, lds); break;
      case 10: phi_ana_quad_tiles<2, true, NW, false>(a, it.y, lds); break;
      case 11: phi_ana_quad_tiles<2, true, NW, true>(a, it.y, lds); break;
    }
}

// Lane groups 2 and 3 of a trade places with groups 0 and 1 of b.
__device__ __forceinline__ void quad_swap(double &a, double &b) {
  const unsigned long long ua = __builtin_bit_cast(unsigned long long, a);
  const unsigned long long ub = __builtin_bit_cast(unsigned long long, b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)ua, (unsigned)ub, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
  a = __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]);
  b = __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}

constexpr int phi_syn_quad_lds(int NQ) { return 8 * ((NQ + 1) / 2) * 128; }

// Synthesis sweep, one row tile per wave: the tile's coefficients (every
// azimuthal column of 16 rows of one colatitude) load once into registers
// as A operands; the basis passes through LDS one tile of 16 folded cells
// at a time (double-buffered, shared by the block's waves), and each tile's
// four sums give the four symmetric cells.
// NQ steps of four columns per group (groups 1-3 may hold one fewer).
template <int NQ, int NW, bool PAIR>
__device__ __forceinline__ void phi_syn_quad_tiles(const PhiQuadArgs &a, int blk, double *lds) {
  constexpr int NT = 64 * NW, NP = (NQ + 1) / 2, CH = phi_syn_quad_lds(NQ) / 2, NB = (CH / 2 + NT - 1) / NT;
  double *const Bs[2] = {lds, lds + CH};
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const int total = a.nt * ((a.Mr + 15) / 16);
  const int want = blk * NW + wave, id = min(want, total - 1);
  const int rt = id / a.nt, j = id - rt * a.nt;
  const double *__restrict__ pv = a.X + (long)j * a.Mr + min(rt * 16 + r16, a.Mr - 1);

  dbl2a br[NB];
  auto bload = [&](int c) {
    const dbl2a *__restrict__ b = reinterpret_cast<const dbl2a *>(a.bas + (long)c * CH);
#pragma unroll
    for (int i = 0; i < NB; ++i) br[i] = b[min(tid + i * NT, CH / 2 - 1)];
  };
  auto bstash = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (CH / 2 >= (i + 1) * NT || tid + i * NT < CH / 2) *reinterpret_cast<dbl2a *>(&Bs[buf][2 * (tid + i * NT)]) = br[i];
  };
  bload(0);
  double v[4][NQ];
#pragma unroll
  for (int gr = 0; gr < 4; ++gr)
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      v[gr][q] = pv[(long)min(quad_column(gr, quad_order(gr, 4 * q + g)), 2 * a.L) * a.MJ];
  bstash(0);
  __syncthreads();

  dbl4q acc[2][4];
#pragma unroll
  for (int gr = 0; gr < 4; ++gr) acc[1][gr] = dbl4q{0.0, 0.0, 0.0, 0.0};
  auto compute = [&](const double *b0, dbl4q (&ac)[4]) {
#pragma unroll
    for (int gr = 0; gr < 4; ++gr) ac[gr] = dbl4q{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int gr = 0; gr < 4; ++gr) {
        const dbl2a b = *reinterpret_cast<const dbl2a *>(b0 + (gr * NP + p) * 128 + 2 * lane);
        ac[gr] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[gr][2 * p], b.x, ac[gr], 0, 0, 0);
        if (2 * p + 1 < NQ)
          ac[gr] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[gr][2 * p + 1 < NQ ? 2 * p + 1 : 0], b.y, ac[gr], 0, 0, 0);
      }
  };
  const bool live = want < total, whole = live && rt * 16 + 16 <= a.Mr;
  // this lane's first row of a swapped pair of tiles
  double *__restrict__ const po = a.C + (long)j * a.np + (long)(rt * 16 + (g & 1)) * a.ld;
  // the symmetric cells' sums from the four groups'
  auto sums = [&](const dbl4q (&ac)[4], int r, double (&o)[4]) {
    const double pc = ac[0][r] + ac[1][r], ps = ac[2][r] + ac[3][r];
    o[0] = pc + ps;
    o[1] = pc - ps;
    if constexpr (PAIR) {
      const double mc = ac[0][r] - ac[1][r], ms = ac[3][r] - ac[2][r];
      o[2] = mc + ms;
      o[3] = mc - ms;
    } else {
      o[2] = o[3] = 0.0;
    }
  };
  // D layout: lane l, element r -> row l / 16 + 4 r, cell l % 16.  After
  // swapping half-waves between the two tiles a store instruction writes
  // two rows of 32 consecutive cells instead of four rows of 16: lane group
  // g then holds cell tile g / 2 of rows (g % 2) + 4 r and that + 2.
  // PLACES: how many of the four symmetric cells every lane stores, 0: each
  // cell and row under its own conditions
  auto store = [&](int c, auto places) {
    constexpr int PL = decltype(places)::value, NO = PL == 2 || !PAIR ? 2 : 4;
    const int t = 16 * (c + (g >> 1)) + r16, f = a.f0 + t, cp = a.cc - f;
    const int off[4] = {f, a.np - 1 - f, cp, a.np - 1 - cp};
    bool ok[4];
    if constexpr (PL == 0) {
      ok[0] = live && t < a.K;
      ok[1] = ok[0] && a.np - 1 - f != f;       // a cell that is its own mirror
      ok[2] = ok[3] = ok[0] && t < a.T2 && cp != f;  // or its own partner is stored once
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double o0[4], o1[4];
      sums(acc[0], r, o0);
      sums(acc[1], r, o1);
      double *__restrict__ q0 = po + (long)(4 * r) * a.ld, *__restrict__ q1 = q0 + 2 * a.ld;
      const int row = rt * 16 + 4 * r + (g & 1);
#pragma unroll
      for (int x = 0; x < NO; ++x) {
        quad_swap(o0[x], o1[x]);
        if (PL != 0 || (ok[x] && row < a.Mr)) q0[off[x]] = o0[x];
        if (PL != 0 || (ok[x] && row + 2 < a.Mr)) q1[off[x]] = o1[x];
      }
    }
  };
  for (int c = 0; c < a.S; c += 2) {
    const bool two = c + 1 < a.S, more = c + 2 < a.S;  // uniform
    if (two) bload(c + 1);
    compute(&Bs[0][0], acc[0]);
    if (two) {
      bstash(1);
      __syncthreads();
      if (more) bload(c + 2);
      compute(&Bs[1][0], acc[1]);  // a missing tile's cells are not stored
      if (more) bstash(0);
      __syncthreads();
    }
    const bool inner = whole && 16 * c + 32 < a.K;  // no padding, no cell that is its own mirror
    if (PAIR && inner && 16 * c + 32 <= a.T2 && c > 0)
      store(c, std::integral_constant<int, 4>{});
    else if (inner && 16 * c >= a.T2)
      store(c, std::integral_constant<int, 2>{});
    else
      store(c, std::integral_constant<int, 0>{});
  }
}

template <int NQ, int NW, bool PAIR>
__global__ __launch_bounds__(64 * NW, NQ <= 3 ? 3 : NQ <= 11 ? 2 : 1) void phi_syn_quad(PhiQuadArgs a) {
  __shared__ __attribute__((aligned(16))) double lds[phi_syn_quad_lds(NQ)];
  phi_syn_quad_tiles<NQ, NW, PAIR>(a, quad_xcd(blockIdx.x, gridDim.x), lds);
}

// The sweep over several plans of up to NM steps: items (plan, block of the
// plan, shape: 2 steps + 1 with partners), one a block.  The same batch: 239
// us in tiles, 172 here.
template <int NM, int NW>
__global__ __launch_bounds__(64 * NW, 2) void phi_syn_group(const PhiQuadArgs *__restrict__ args,
                                                            const int4 *__restrict__ items) {
  __shared__ __attribute__((aligned(16))) double lds[phi_syn_quad_lds(NM)];
  const int4 it = items[blockIdx.x];
  const PhiQuadArgs a = args[it.x];
#define YYG_STEPS(NQ)                                                        \
  case 2 * NQ: phi_syn_quad_tiles<NQ, NW, false>(a, it.y, lds); break;       \
  case 2 * NQ + 1: phi_syn_quad_tiles<NQ, NW, true>(a, it.y, lds); break
  switch (it.z) {  // uniform
    YYG_STEPS(1);
    YYG_STEPS(2);
    YYG_STEPS(3);
    YYG_STEPS(4);
  }
  if constexpr (NM >= 9) switch (it.z) {
      YYG_STEPS(5);
      YYG_STEPS(6);
      YYG_STEPS(9);
    }
#undef YYG_STEPS
}

// Synthesis with the basis in registers: wave w of a block owns one tile of
// 16 folded cells for the block's whole life (its basis, NQ steps of four
// columns per group, as B operands) and the block walks row tiles.  A row
// tile's coefficients pass through LDS in operand order; its cells go back
// through LDS, so that the block writes whole rows of phi with 16-byte
// stores, 1 KiB of a row per instruction, while it multiplies the next row
// tile.  What bounded the earlier forms at half a degree (1.58 GB of phi)
// was the store path, not the products (0.26 ms): waves owning row tiles and
// sweeping the cells (phi_syn_quad) keep every row open at four places over
// their life, 0.69 ms; this form storing straight from the operand layout
// (four rows of 16 cells per instruction, each piece across two cache
// lines) 0.50 ms.
// ctp waves share a row tile, rtn row tiles run side by side; NL 16-byte
// coefficient loads and NO 16-byte row pieces per thread and iteration; LDS
// row stride ldr.  EVEN: the even cosines alone hold a last step (L a
// multiple of 8).  16 ld and (2 L + 1) MJ stay below 2^28 (32-bit offsets in
// bytes).
template <int NQ>
constexpr int rows_max_waves() {
  return NQ <= 9 ? 12 : 8;
}

template <int NQ, int NL, int NO, bool EVEN, bool PAIR>
__global__ __launch_bounds__(64 * rows_max_waves<NQ>()) void phi_syn_rows(PhiQuadArgs a, int ctp, int rtn, int ldr) {
  constexpr int NP = (NQ + 1) / 2, NS = 16 * NQ;  // slots: 4 NQ columns of four groups
  extern __shared__ __attribute__((aligned(16))) double lds[];
  const int tid = threadIdx.x, lane = tid & 63, nthr = 64 * ctp * rtn;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const int ib = quad_xcd(blockIdx.x, gridDim.x);
  const int tiles = a.nt * ((a.Mr + 15) / 16), its = (tiles + rtn - 1) / rtn;
  const int beg = (int)((long)its * ib / gridDim.x), end = (int)((long)its * (ib + 1) / gridDim.x);
  const int sub = wave / ctp, ct = wave - sub * ctp;
  if (beg >= end) return;  // uniform over the block

  // this wave's basis
  double b[4][NQ];
  {
    const double *__restrict__ pb = a.bas + (long)min(ct, a.S - 1) * 4 * NP * 128 + 2 * lane;
#pragma unroll
    for (int gr = 0; gr < 4; ++gr)
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        if (gr == 0 || !EVEN || q < NQ - 1) b[gr][q] = pb[(gr * NP + q / 2) * 128 + (q & 1)];
    // waited for here, once: a wait inside the loop would also wait for the
    // loop's stores
#pragma unroll
    for (int gr = 0; gr < 4; ++gr)
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        if (gr == 0 || !EVEN || q < NQ - 1) asm volatile("" : "+v"(b[gr][q]));
  }

  // this thread's share of its row tile's coefficients: two rows of one slot
  // (16 bytes; rows past the last one read what follows or zero and are
  // never stored)
  const int e0 = ct * 64 + lane, est = 64 * ctp;
  const int vsz = 2 * NL * est;  // a row tile's coefficients in LDS, whole loads
  double *__restrict__ const vs = lds + sub * vsz, *__restrict__ const rows = lds + rtn * vsz;
  unsigned voff[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int slot = (e0 + i * est) / 8, gr = slot / (4 * NQ);
    const int mc = min(quad_column(gr, quad_order(gr, slot - gr * 4 * NQ)), 2 * a.L);
    voff[i] = slot < NS ? 8u * ((unsigned)mc * (unsigned)a.MJ + 2 * (e0 & 7)) : kNoPlace;
  }
  const long vbytes = 8 * (2L * a.L + 1) * a.MJ;
  auto vload = [&](int it, u32x4 (&v)[NL]) {
    const int id = min(it * rtn + sub, tiles - 1), rt = id / a.nt, j = id - rt * a.nt;  // uniform
    const long at = (long)j * a.Mr + rt * 16;
    const auto rs = buffer_of(a.X + at, vbytes - 8 * at);
#pragma unroll
    for (int i = 0; i < NL; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, voff[i], 0, 0);
  };
  auto vstash = [&](const u32x4 (&v)[NL]) {
#pragma unroll
    for (int i = 0; i < NL; ++i) *reinterpret_cast<u32x4 *>(vs + 2 * (e0 + i * est)) = v[i];
  };

  // the LDS places of this lane's cell, its mirror, its partner and the
  // partner's mirror in row g of the row tile
  const int t = 16 * ct + r16, f = a.f0 + t, cp = a.cc - f;
  const bool own = t < a.K, par = PAIR && own && t < a.T2;
  double *__restrict__ const row0 = rows + (sub * 16 + g) * ldr;

  // this thread's pieces of its row tile's finished rows: piece u = row
  // u / ppr, two cells from 2 (u % ppr) (the last of an odd row repeats one)
  const int ppr = (a.np + 1) / 2;
  int lo[NO];
  unsigned go[NO];
#pragma unroll
  for (int i = 0; i < NO; ++i) {
    const int u = e0 + i * est, rr = u / ppr, k = min(2 * (u - rr * ppr), a.np - 2);
    lo[i] = (sub * 16 + min(rr, 15)) * ldr + k;
    go[i] = rr < 16 ? 8u * ((unsigned)rr * (unsigned)a.ld + k) : kNoPlace;
  }
  const long cbytes = 8 * (long)a.Mr * a.ld;
  // phi from the first cell of iteration it's row tile (rows past the last
  // one lie past the end); nothing before the first and past the last tile
  auto out = [&](int it) {
    const int id = it * rtn + sub, rt = id / a.nt, j = id - rt * a.nt;
    const long at = (long)rt * 16 * a.ld + (long)j * a.np;
    return buffer_of(a.C + at, it >= beg && id < tiles ? cbytes - 8 * at : 0);
  };
  auto piece = [&](__amdgpu_buffer_rsrc_t rs, int i) {
    const dbl2q x = *reinterpret_cast<const dbl2q *>(rows + lo[i]);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), rs, go[i], 0, 0);
  };

  u32x4 v[NL];
  vload(beg, v);
  vstash(v);
  vload(beg + 1, v);
  __syncthreads();
  // The rows of iteration it - 1 leave between the products of iteration it.
  // No load or store is under a condition (the last loads repeat the last row
  // tile), so that the wait for the coefficients counts the stores issued
  // after them and does not wait for those.
  for (int it = beg; it < end; ++it) {
    const auto rs = out(it - 1);
    dbl4q ac[4];
#pragma unroll
    for (int gr = 0; gr < 4; ++gr) ac[gr] = dbl4q{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
#pragma unroll
      for (int gr = 0; gr < 4; ++gr)
        if (gr == 0 || !EVEN || q < NQ - 1)
          ac[gr] = __builtin_amdgcn_mfma_f64_16x16x4f64(vs[(gr * 4 * NQ + 4 * q) * 16 + lane], b[gr][q], ac[gr], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < NO; ++i)
        if (i * NQ / NO == q) piece(rs, i);
    }
    __syncthreads();  // every wave has read the coefficients and the finished rows
    if (own) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double pc = ac[0][r] + ac[1][r], ps = ac[2][r] + ac[3][r];
        double *__restrict__ q = row0 + 4 * r * ldr;
        q[f] = pc + ps;
        if (a.np - 1 - f != f) q[a.np - 1 - f] = pc - ps;
        if (PAIR && par && cp != f) {
          const double mc = ac[0][r] - ac[1][r], ms = ac[3][r] - ac[2][r];
          q[cp] = mc + ms;
          q[a.np - 1 - cp] = mc - ms;
        }
      }
    }
    vstash(v);
    vload(it + 2, v);
    __syncthreads();
  }
  const auto rs = out(end - 1);
#pragma unroll
  for (int i = 0; i < NO; ++i) piece(rs, i);
}

// Analysis with the basis in registers: wave w of a block owns one tile of
// 16 outputs of one group for the block's whole life (SM stages of four
// steps) and the block walks row tiles.  Its threads load a row tile's
// density one iteration ahead (U pairs of folded points per thread, from
// each of the four symmetric places: whole rows, contiguous across the
// block), fold it and write the folded values to LDS while the waves
// multiply the previous row tile (double-buffered, one barrier per
// iteration).  The basis is then read once per block and not once per four
// row tiles, and a stage costs no barrier.  At half a degree (1000 shells,
// lmax 64: 1.95 GB, 17 GFLOP) 0.47 ms in a solve, 4.2 TB/s, against 0.67 ms for
// the best form folded once (25 GFLOP; the sweep, launched alone, 0.51 against
// 0.45); the products alone would take 0.23 ms.  Less where a block has few
// iterations: 550 shells at 1 degree, lmax 40 (286 MB) 106 us, 2.7 TB/s.
// Four tj waves share a row tile, rtn row tiles run side by side.  LDS holds
// the even cosines' and even sines' inputs of every point (row stride ldp)
// and the odd ones' of the paired stages (stride ldq; past them the two
// agree).  16 ld stays below 2^28 (32-bit offsets in bytes).
template <int SM, int U, bool XC, bool WGT, int NWM>
__global__ __launch_bounds__(64 * NWM) void phi_ana_rows(PhiQuadArgs a, int tj4, int rtn) {
  extern __shared__ __attribute__((aligned(16))) double lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const int ib = quad_xcd(blockIdx.x, gridDim.x);
  const int tiles = a.nt * ((a.Mr + 15) / 16), its = (tiles + rtn - 1) / rtn;
  const int beg = (int)((long)its * ib / gridDim.x), end = (int)((long)its * (ib + 1) / gridDim.x);
  if (beg >= end) return;  // uniform over the block
  const int sub = wave / tj4, w = wave - sub * tj4, gr = w & 3, tj = w >> 2, TJ = tj4 >> 2;
  const int sp = (a.T2 + 15) / 16, ldp = 16 * a.S + 2, ldq = 16 * sp + 2;
  const int psz = 32 * (ldp + ldq);  // a row tile's folded values
  double *__restrict__ const pl = lds + sub * 2 * psz;
  const int ch = 4 * TJ * 256 + (XC ? 16 : 0);

  // this wave's basis: stage s, steps 4 s + 2 h + e, point 16 s + 4 g + 2 h + e
  double b[SM][4];
  {
    const double *__restrict__ pb = a.bas + (gr * TJ + tj) * 256 + 2 * lane;
#pragma unroll
    for (int s = 0; s < SM; ++s)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const dbl2a x = *reinterpret_cast<const dbl2a *>(pb + (long)min(s, a.S - 1) * ch + h * 128);
        b[s][2 * h] = x.x;
        b[s][2 * h + 1] = x.y;
      }
  }
  // XC: the last even cosine's basis, summed by the first wave of a row tile
  double *__restrict__ const xb = lds + rtn * 2 * psz;
  if constexpr (XC) {
    for (int e = tid; e < 16 * a.S; e += 64 * tj4 * rtn) xb[e] = a.bas[(long)(e / 16) * ch + 4 * TJ * 256 + e % 16];
  }

  // this thread's pairs of points: byte offsets of the four places within
  // the row tile (none for padding), of the weights, and the LDS place
  const int e0 = w * 64 + lane, est = 64 * tj4, ppr = 8 * a.S;
  unsigned oa[U], ob[U], oc[U], od[U];
  int ow[U], lo[U], lq[U];
  bool i0[U], i1[U];
#pragma unroll
  for (int i = 0; i < U; ++i) {
    const int u = e0 + i * est, rr = u / ppr, t = 2 * (u - rr * ppr);
    const bool in = rr < 16 && t < a.K, pin = in && t < a.T2;  // T2 is even
    const unsigned ro = 8u * (unsigned)rr * (unsigned)a.ld;
    const int f = min(a.f0 + t, a.np - 2);
    oa[i] = in ? ro + 8 * f : kNoPlace;
    ob[i] = in ? ro + 8 * (a.np - 2 - f) : kNoPlace;
    oc[i] = pin ? ro + 8 * (a.cc - a.f0 - t - 1) : kNoPlace;
    od[i] = pin ? ro + 8 * (a.np - 1 - a.cc + a.f0 + t) : kNoPlace;
    ow[i] = min(t, a.Kp - 2);
    lo[i] = rr < 16 ? rr * ldp + t : -1;
    lq[i] = rr < 16 && t < 16 * sp ? 32 * ldp + rr * ldq + t : -1;
    i0[i] = in && t >= a.tlo;
    i1[i] = in && t + 1 < a.K;
  }
  const long xbytes = 8 * (long)a.Mr * a.ld;
  u32x4 ra[U], rb[U], rc[U], rd[U];
  dbl2q wa[U], wc[U];
  struct From {
    __amdgpu_buffer_rsrc_t rs;
    const double *pw;
  };
  auto from = [&](int it) {  // past the last row tile: the last one again
    const int id = min(it * rtn + sub, tiles - 1), rt = id / a.nt, j = id - rt * a.nt;  // uniform
    const long at = (long)rt * 16 * a.ld + (long)j * a.np;
    return From{buffer_of(a.X + at, xbytes - 8 * at), a.W + (long)j * 2 * a.Kp};
  };
  auto load = [&](const From &fr, int i) {
    ra[i] = __builtin_amdgcn_raw_buffer_load_b128(fr.rs, oa[i], 0, 0);
    rb[i] = __builtin_amdgcn_raw_buffer_load_b128(fr.rs, ob[i], 0, 0);
    rc[i] = __builtin_amdgcn_raw_buffer_load_b128(fr.rs, oc[i], 0, 0);
    rd[i] = __builtin_amdgcn_raw_buffer_load_b128(fr.rs, od[i], 0, 0);
    if constexpr (WGT) {
      wa[i] = *reinterpret_cast<const dbl2q *>(fr.pw + ow[i]);
      wc[i] = *reinterpret_cast<const dbl2q *>(fr.pw + a.Kp + ow[i]);
    }
  };
  // the descending places hold their pair in reverse; padding points fold
  // to zero
  auto fold = [&](int buf, int i) {
    const dbl2a A = __builtin_bit_cast(dbl2a, ra[i]), B = __builtin_bit_cast(dbl2a, rb[i]);
    const dbl2a C = __builtin_bit_cast(dbl2a, rc[i]), D = __builtin_bit_cast(dbl2a, rd[i]);
    double e[4][2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const bool in = k ? i1[i] : i0[i];
      double pp = A[k] + B[1 - k], m = A[k] - B[1 - k], q = C[1 - k] + D[k], n = C[1 - k] - D[k];
      if constexpr (WGT) {
        pp *= wa[i][k];
        m *= wa[i][k];
        q *= wc[i][k];
        n *= wc[i][k];
      }
      e[0][k] = in ? pp + q : 0.0;
      e[1][k] = in ? pp - q : 0.0;
      e[2][k] = in ? m - n : 0.0;
      e[3][k] = in ? m + n : 0.0;
    }
    double *__restrict__ d = pl + buf * psz;
    if (lo[i] >= 0) {
      *reinterpret_cast<dbl2a *>(d + lo[i]) = dbl2a{e[0][0], e[0][1]};
      *reinterpret_cast<dbl2a *>(d + 16 * ldp + lo[i]) = dbl2a{e[2][0], e[2][1]};
    }
    if (lq[i] >= 0) {
      *reinterpret_cast<dbl2a *>(d + lq[i]) = dbl2a{e[1][0], e[1][1]};
      *reinterpret_cast<dbl2a *>(d + 16 * ldq + lq[i]) = dbl2a{e[3][0], e[3][1]};
    }
  };

  const From f0 = from(beg), f1 = from(beg + 1);
#pragma unroll
  for (int i = 0; i < U; ++i) load(f0, i);
#pragma unroll
  for (int s = 0; s < SM; ++s)
#pragma unroll
    for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(b[s][k]));  // waited for here, once
#pragma unroll
  for (int i = 0; i < U; ++i) {
    fold(0, i);
    load(f1, i);
  }
  __syncthreads();
  const int pe = (gr & 2 ? 16 * ldp : 0) + r16 * ldp + 4 * g;                          // every stage, or past the pairs
  const int po = 32 * ldp + (gr & 2 ? 16 * ldq : 0) + r16 * ldq + 4 * g;               // an odd group's paired stages
  for (int it = beg; it < end; ++it) {
    const int buf = (it - beg) & 1;
    const double *__restrict__ src = pl + buf * psz;
    dbl4q ac0 = dbl4q{0.0, 0.0, 0.0, 0.0}, ac1 = ac0;
    double xacc = 0.0;
    const From fn = from(it + 2);
#pragma unroll
    for (int s = 0; s < SM; ++s) {
      if (s < a.S) {  // uniform
        const double *__restrict__ q = src + ((gr & 1) && s < sp ? po : pe) + 16 * s;
        const dbl2a x0 = *reinterpret_cast<const dbl2a *>(q), x1 = *reinterpret_cast<const dbl2a *>(q + 2);
        ac0 = __builtin_amdgcn_mfma_f64_16x16x4f64(b[s][0], x0.x, ac0, 0, 0, 0);
        ac1 = __builtin_amdgcn_mfma_f64_16x16x4f64(b[s][1], x0.y, ac1, 0, 0, 0);
        ac0 = __builtin_amdgcn_mfma_f64_16x16x4f64(b[s][2], x1.x, ac0, 0, 0, 0);
        ac1 = __builtin_amdgcn_mfma_f64_16x16x4f64(b[s][3], x1.y, ac1, 0, 0, 0);
        if constexpr (XC) {
          if (w == 0) {  // uniform
            const dbl2a y0 = *reinterpret_cast<const dbl2a *>(xb + 16 * s + 4 * g);
            const dbl2a y1 = *reinterpret_cast<const dbl2a *>(xb + 16 * s + 4 * g + 2);
            xacc = __builtin_fma(y0.x, x0.x, xacc);
            xacc = __builtin_fma(y0.y, x0.y, xacc);
            xacc = __builtin_fma(y1.x, x1.x, xacc);
            xacc = __builtin_fma(y1.y, x1.y, xacc);
          }
        }
      }
      // the next row tile's values, between the products; each pair is loaded
      // again at once, a whole iteration before it is folded
#pragma unroll
      for (int i = 0; i < U; ++i)
        if ((i + 1) * SM / (U + 1) == s) {
          fold(buf ^ 1, i);
          load(fn, i);
        }
    }
    // D layout: lane l, element r -> output l / 16 + 4 r of the tile, row l % 16
    const int id = it * rtn + sub, rt = id / a.nt, j = id - rt * a.nt, row = rt * 16 + r16;
    double *__restrict__ out = a.C + (long)j * a.Mr + row;
    const bool live = id < tiles && row < a.Mr;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = quad_order(gr, 16 * tj + g + 4 * r);
      if (live && m <= a.L) out[(long)quad_column(gr, m) * a.MJ] = ac0[r] + ac1[r];
    }
    if constexpr (XC) {
      if (w == 0) {
        xacc += __shfl_xor(xacc, 16);
        xacc += __shfl_xor(xacc, 32);
        if (live && g == 0) out[(long)(2 * a.L - 1) * a.MJ] = xacc;
      }
    }
    __syncthreads();
  }
}

// Variants: the basis in registers (row tiles side by side and blocks per
// CU at most; where it does not fit, the sweep with 4 waves), then sweeps
// with so many waves per block.
struct QuadVariant {
  int rtn, per_cu, waves;
};
constexpr QuadVariant kQuad[] = {{4, 4, 4}, {1, 4, 4}, {4, 1, 4}, {0, 0, 4}, {0, 0, 2}, {0, 0, 8}, {0, 0, 1}, {0, 0, 3}};

template <int TJ, bool XC, int NW>
void launch_ana_t(const PhiQuadArgs &a, int blocks, hipStream_t s) {
  if (a.W)
    hipLaunchKernelGGL((phi_ana_quad<TJ, XC, NW, true>), dim3(blocks), dim3(64 * NW), 0, s, a);
  else
    hipLaunchKernelGGL((phi_ana_quad<TJ, XC, NW, false>), dim3(blocks), dim3(64 * NW), 0, s, a);
}

template <int NW>
hipError_t launch_ana_w(const PhiQuadArgs &a, int blocks, hipStream_t s) {
  const int tj = phi_quad_tiles(a.L);
  const bool xc = phi_quad_extra(a.L);
  switch (2 * tj + (xc ? 1 : 0)) {
    case 2: launch_ana_t<1, false, NW>(a, blocks, s); break;
    case 3: launch_ana_t<1, true, NW>(a, blocks, s); break;
    case 4: launch_ana_t<2, false, NW>(a, blocks, s); break;
    case 5: launch_ana_t<2, true, NW>(a, blocks, s); break;
    case 6: launch_ana_t<3, false, NW>(a, blocks, s); break;
    case 7: launch_ana_t<3, true, NW>(a, blocks, s); break;
    case 8: launch_ana_t<4, false, NW>(a, blocks, s); break;
    case 9: launch_ana_t<4, true, NW>(a, blocks, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Launch shape of phi_ana_rows: u = 0 where it does not fit.
struct AnaShape {
  int tj4, rtn, u, sm, per_cu;
  size_t lds;
};
AnaShape ana_rows_shape(const PhiQuadArgs &a, const QuadVariant &v) {
  AnaShape s{};
  const int tj = phi_quad_tiles(a.L), sp = (a.T2 + 15) / 16;
  s.tj4 = 4 * tj;
  s.sm = a.S <= 3 ? 3 : a.S <= 6 ? 6 : 12;
  const int u = (128 * a.S + 64 * s.tj4 - 1) / (64 * s.tj4), wm = tj <= 2 ? 8 : 4 * tj;
  if (a.S > 12 || u > 3 || a.np < 2 || 16 * a.ld >= (1L << 28)) return s;
  if (tj > 2 && s.sm > 6) return s;  // their registers do not hold the basis
  for (s.rtn = std::min(wm / s.tj4, v.rtn); s.rtn >= 1; --s.rtn) {
    s.lds = ((size_t)s.rtn * 64 * (16 * a.S + 2 + 16 * sp + 2) + 16 * a.S) * sizeof(double);
    if (s.lds <= 160 * 1024) {
      s.u = u;
      s.per_cu = std::max(1, std::min({v.per_cu, s.sm <= 6 ? 16 / (s.tj4 * s.rtn) : 1, (int)(160 * 1024 / s.lds)}));
      return s;
    }
  }
  return s;
}

template <int SM, int U, bool XC, int NWM>
void launch_ana_rows_w(const PhiQuadArgs &a, const AnaShape &h, int cus, hipStream_t s) {
  const long tiles = (long)a.nt * ((a.Mr + 15) / 16), its = (tiles + h.rtn - 1) / h.rtn;
  const dim3 grid((unsigned)std::min((long)cus * h.per_cu, its)), block(64 * h.tj4 * h.rtn);
  if (a.W)
    hipLaunchKernelGGL((phi_ana_rows<SM, U, XC, true, NWM>), grid, block, h.lds, s, a, h.tj4, h.rtn);
  else
    hipLaunchKernelGGL((phi_ana_rows<SM, U, XC, false, NWM>), grid, block, h.lds, s, a, h.tj4, h.rtn);
}

template <int SM, int U, int NWM>
void launch_ana_rows_x(const PhiQuadArgs &a, const AnaShape &h, int cus, hipStream_t s) {
  if (phi_quad_extra(a.L))
    launch_ana_rows_w<SM, U, true, NWM>(a, h, cus, s);
  else
    launch_ana_rows_w<SM, U, false, NWM>(a, h, cus, s);
}

template <int SM, int NWM>
hipError_t launch_ana_rows_u(const PhiQuadArgs &a, const AnaShape &h, int cus, hipStream_t s) {
  switch (h.u) {
    case 1: launch_ana_rows_x<SM, 1, NWM>(a, h, cus, s); break;
    case 2: launch_ana_rows_x<SM, 2, NWM>(a, h, cus, s); break;
    default: launch_ana_rows_x<SM, 3, NWM>(a, h, cus, s); break;
  }
  return hipGetLastError();
}

hipError_t launch_ana_rows(const PhiQuadArgs &a, const AnaShape &h, int cus, hipStream_t s) {
  if (h.tj4 > 8) {
    if (h.sm == 3)
      launch_ana_rows_x<3, 1, 16>(a, h, cus, s);
    else
      launch_ana_rows_x<6, 1, 16>(a, h, cus, s);
    return hipGetLastError();
  }
  return h.sm == 3 ? launch_ana_rows_u<3, 8>(a, h, cus, s)
         : h.sm == 6 ? launch_ana_rows_u<6, 8>(a, h, cus, s)
                     : launch_ana_rows_u<12, 8>(a, h, cus, s);
}

// Launch shape of phi_syn_rows: as many row tiles side by side as the waves
// and the LDS of a block hold; nl = 0 where it does not fit (more cell
// tiles than waves, rows longer than the LDS, offsets past 32 bits).
struct RowsShape {
  int ctp, rtn, nl, no, ldr, per_cu;
  size_t lds;
};
RowsShape syn_rows_shape(const PhiQuadArgs &a, const QuadVariant &v) {
  RowsShape s{};
  const int nq = phi_quad_steps(a.L), wm = nq <= 9 ? 12 : 8;
  s.ctp = a.S;
  if (nq < 0 || s.ctp > wm || a.np < 2 || 16 * a.ld >= (1L << 28) || (2L * a.L + 1) * a.MJ >= (1L << 28)) return s;
  const int nl = (2 * nq + s.ctp - 1) / s.ctp, no = (16 * ((a.np + 1) / 2) + 64 * s.ctp - 1) / (64 * s.ctp);
  if (nl > 6 || no > 9) return s;
  s.ldr = (a.np + 15) / 32 * 32 + 16;  // rows g and g + 1 half the banks apart
  for (s.rtn = std::min(wm / s.ctp, v.rtn); s.rtn >= 1; --s.rtn) {
    const int NLT = nl <= 2 ? 2 : nl <= 4 ? 4 : 6;
    s.lds = (size_t)s.rtn * (2 * NLT * 64 * s.ctp + 16 * s.ldr) * sizeof(double);
    if (s.lds <= 160 * 1024) {
      s.nl = NLT;
      s.no = no <= 6 ? 6 : 9;
      s.per_cu = std::max(1, std::min({v.per_cu, wm / (s.ctp * s.rtn), (int)(160 * 1024 / s.lds)}));
      return s;
    }
  }
  return s;
}

template <int NQ>
hipError_t launch_syn_rows_t(const PhiQuadArgs &a, const RowsShape &h, int cus, hipStream_t s) {
  const long tiles = (long)a.nt * ((a.Mr + 15) / 16), its = (tiles + h.rtn - 1) / h.rtn;
  const dim3 grid((unsigned)std::min((long)cus * h.per_cu, its)), block(64 * h.ctp * h.rtn);
#define YYG_ROWS_GO(NL, NO)                                                                                       \
  if (a.L % 8 == 0 && a.T2 > 0)                                                                                   \
    hipLaunchKernelGGL((phi_syn_rows<NQ, NL, NO, true, true>), grid, block, h.lds, s, a, h.ctp, h.rtn, h.ldr);    \
  else if (a.T2 > 0)                                                                                              \
    hipLaunchKernelGGL((phi_syn_rows<NQ, NL, NO, false, true>), grid, block, h.lds, s, a, h.ctp, h.rtn, h.ldr);   \
  else                                                                                                            \
    hipLaunchKernelGGL((phi_syn_rows<NQ, NL, NO, false, false>), grid, block, h.lds, s, a, h.ctp, h.rtn, h.ldr)
  if (h.no == 6 && h.nl == 2) {
    YYG_ROWS_GO(2, 6);
  } else if (h.no == 6 && h.nl == 4) {
    YYG_ROWS_GO(4, 6);
  } else if (h.no == 6) {
    YYG_ROWS_GO(6, 6);
  } else if (h.nl == 2) {
    YYG_ROWS_GO(2, 9);
  } else if (h.nl == 4) {
    YYG_ROWS_GO(4, 9);
  } else {
    YYG_ROWS_GO(6, 9);
  }
#undef YYG_ROWS_GO
  return hipGetLastError();
}

hipError_t launch_syn_rows(const PhiQuadArgs &a, const RowsShape &h, int cus, hipStream_t s) {
  switch (phi_quad_steps(a.L)) {
    case 1: return launch_syn_rows_t<1>(a, h, cus, s);
    case 2: return launch_syn_rows_t<2>(a, h, cus, s);
    case 3: return launch_syn_rows_t<3>(a, h, cus, s);
    case 4: return launch_syn_rows_t<4>(a, h, cus, s);
    case 5: return launch_syn_rows_t<5>(a, h, cus, s);
    case 6: return launch_syn_rows_t<6>(a, h, cus, s);
    case 9: return launch_syn_rows_t<9>(a, h, cus, s);
    case 11: return launch_syn_rows_t<11>(a, h, cus, s);
    case 17: return launch_syn_rows_t<17>(a, h, cus, s);
    default: return hipErrorInvalidValue;
  }
}

template <int NQ, int NW>
void launch_syn_t(const PhiQuadArgs &a, int blocks, hipStream_t s) {
  if (a.T2 > 0)
    hipLaunchKernelGGL((phi_syn_quad<NQ, NW, true>), dim3(blocks), dim3(64 * NW), 0, s, a);
  else
    hipLaunchKernelGGL((phi_syn_quad<NQ, NW, false>), dim3(blocks), dim3(64 * NW), 0, s, a);
}

template <int NW>
hipError_t launch_syn_w(const PhiQuadArgs &a, int blocks, hipStream_t s) {
  switch (phi_quad_steps(a.L)) {
    case 1: launch_syn_t<1, NW>(a, blocks, s); break;
    case 2: launch_syn_t<2, NW>(a, blocks, s); break;
    case 3: launch_syn_t<3, NW>(a, blocks, s); break;
    case 4: launch_syn_t<4, NW>(a, blocks, s); break;
    case 5: launch_syn_t<5, NW>(a, blocks, s); break;
    case 6: launch_syn_t<6, NW>(a, blocks, s); break;
    case 9: launch_syn_t<9, NW>(a, blocks, s); break;
    case 11: launch_syn_t<11, NW>(a, blocks, s); break;
    case 17: launch_syn_t<17, NW>(a, blocks, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

// outputs per group: L / 2 + 1 even cosines, (L + 1) / 2 odd cosines and odd
// sines, L / 2 even sines
int phi_quad_tiles(int L) {
  const int most = L / 2 + 1, others = std::max((L + 1) / 2, 1), tj = (others + 15) / 16;
  return most > 16 * tj + 1 ? tj + 1 : tj;
}
bool phi_quad_extra(int L) { return L / 2 + 1 == 16 * phi_quad_tiles(L) + 1; }
int phi_quad_chunk(int L) { return 4 * phi_quad_tiles(L) * 256 + (phi_quad_extra(L) ? 16 : 0); }
int phi_quad_steps(int L) {
  const int n = L / 8 + 1;  // ceil((L / 2 + 1) / 4)
  for (int k : {1, 2, 3, 4, 5, 6, 9, 11, 17})
    if (n <= k) return k;
  return -1;
}

int phi_quad_variant_count() { return (int)(sizeof(kQuad) / sizeof(kQuad[0])); }

// The registers' form pays for its basis and its first loads once per block:
// the default from four iterations a block on.  Whole solves, us, with this
// form and with the sweep.  Analysis: 4.6 iterations (400 shells at 2 degrees,
// lmax 25) 58 and 59, polar 53 and 56; 9 (800 shells, lmax 25) 93 and 98, lmax
// 40 141 and 155; 6.8 (300 at 1 degree, lmax 30) 101 and 113; below four the two
// lie within 5% either way (200 at 2 degrees, lmax 25 45.1 and 45.5).
// Synthesis: 800 shells at 2 degrees 93 and 93; 300 at 1 degree, lmax 30 101 and
// 105; 400 at 0.75, lmax 40 240 and 271; 1000 at half a degree, lmax 64 441 and
// 674 alone; but not at degrees 48 to 63, whose seven and eight steps run as
// nine: 300 at 1 degree, lmax 50 171 and 167; polar 1.5 degrees, lmax 60 129
// and 94.
int phi_quad_default(bool analysis, const PhiQuadArgs &a, int cus) {
  const long tiles = (long)a.nt * ((a.Mr + 15) / 16);
  long side = 0;
  if (analysis) {
    const AnaShape h = ana_rows_shape(a, kQuad[0]);
    side = h.u > 0 ? (long)h.rtn * h.per_cu * cus : 0;
  } else {
    const RowsShape h = syn_rows_shape(a, kQuad[0]);
    side = h.nl > 0 ? (long)h.rtn * h.per_cu * cus : 0;
  }
  if (side > 0 && tiles >= 4 * side) return 0;
  return analysis ? 4 : 3;
}

hipError_t launch_phi_quad(int v, bool analysis, const PhiQuadArgs &a, int cus, hipStream_t s) {
  if (a.Mr <= 0 || a.nt <= 0 || a.K <= 0) return hipSuccess;
  if (v < 0 || v >= phi_quad_variant_count() || a.np < 2 || a.S < 1) return hipErrorInvalidValue;
  const long tiles = (long)a.nt * ((a.Mr + 15) / 16);
  if (tiles >= INT_MAX / 8) return hipErrorInvalidValue;
  const QuadVariant &k = kQuad[v];
  if (k.rtn > 0) {
    if (analysis) {
      const AnaShape h = ana_rows_shape(a, k);
      if (h.u > 0) return launch_ana_rows(a, h, cus, s);
    } else {
      const RowsShape h = syn_rows_shape(a, k);
      if (h.nl > 0) return launch_syn_rows(a, h, cus, s);
    }
  }
  const int blocks = (int)((tiles + k.waves - 1) / k.waves);
  switch (k.waves) {
    case 1: return analysis ? launch_ana_w<1>(a, blocks, s) : launch_syn_w<1>(a, blocks, s);
    case 2: return analysis ? launch_ana_w<2>(a, blocks, s) : launch_syn_w<2>(a, blocks, s);
    case 3: return analysis ? launch_ana_w<3>(a, blocks, s) : launch_syn_w<3>(a, blocks, s);
    case 8: return analysis ? launch_ana_w<8>(a, blocks, s) : launch_syn_w<8>(a, blocks, s);
    default: return analysis ? launch_ana_w<4>(a, blocks, s) : launch_syn_w<4>(a, blocks, s);
  }
}

// Waves of the batch's blocks: four, so that LDS leaves three waves per SIMD in
// the analysis (two with a single plan's two waves a block).
constexpr int kGroupAna = 4, kGroupSyn = 4;

bool phi_group_fits(bool analysis, const PhiQuadArgs &a) {
  const long tiles = (long)a.nt * ((a.Mr + 15) / 16);
  return a.np >= 2 && a.S >= 1 && a.K > 0 && tiles < INT_MAX / 8 &&
         (analysis ? phi_quad_tiles(a.L) <= 2 : phi_quad_steps(a.L) >= 1 && phi_quad_steps(a.L) <= 9);
}

int phi_group_blocks(bool analysis, const PhiQuadArgs &a) {
  const int nw = analysis ? kGroupAna : kGroupSyn;
  return (int)(((long)a.nt * ((a.Mr + 15) / 16) + nw - 1) / nw);
}

int phi_group_shape(bool analysis, const PhiQuadArgs &a) {
  return analysis ? 4 * phi_quad_tiles(a.L) + 2 * (phi_quad_extra(a.L) ? 1 : 0) + (a.W ? 1 : 0)
                  : 2 * phi_quad_steps(a.L) + (a.T2 > 0 ? 1 : 0);
}

hipError_t launch_phi_group(bool analysis, int max_shape, const PhiQuadArgs *args, const int4 *items, int n_items,
                            hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  const dim3 grid(n_items), block(64 * (analysis ? kGroupAna : kGroupSyn));
  if (analysis && max_shape < 8)
    hipLaunchKernelGGL((phi_ana_group<1, kGroupAna>), grid, block, 0, s, args, items);
  else if (analysis)
    hipLaunchKernelGGL((phi_ana_group<2, kGroupAna>), grid, block, 0, s, args, items);
  else if (max_shape < 10)
    hipLaunchKernelGGL((phi_syn_group<4, kGroupSyn>), grid, block, 0, s, args, items);
  else
    hipLaunchKernelGGL((phi_syn_group<9, kGroupSyn>), grid, block, 0, s, args, items);
  return hipGetLastError();
}

int phi_quad_kernel_name(int v, bool analysis, const PhiQuadArgs &a, char *buf, size_t n) {
  if (v < 0 || v >= phi_quad_variant_count()) return -1;
  auto tf = [](bool x) { return x ? "true" : "false"; };
  const QuadVariant &k = kQuad[v];
  const char *ns = "yyg::(anonymous namespace)::";
  int r;
  if (analysis) {
    const AnaShape h = ana_rows_shape(a, k);
    if (k.rtn > 0 && h.u > 0)
      r = snprintf(buf, n, "%sphi_ana_rows<%d, %d, %s, %s, %d>", ns, h.sm, h.u, tf(phi_quad_extra(a.L)), tf(a.W != nullptr),
                   h.tj4 > 8 ? 16 : 8);
    else
      r = snprintf(buf, n, "%sphi_ana_quad<%d, %s, %d, %s>", ns, phi_quad_tiles(a.L), tf(phi_quad_extra(a.L)), k.waves,
                   tf(a.W != nullptr));
  } else {
    const RowsShape h = syn_rows_shape(a, k);
    if (k.rtn > 0 && h.nl > 0)
      r = snprintf(buf, n, "%sphi_syn_rows<%d, %d, %d, %s, %s>", ns, phi_quad_steps(a.L), h.nl, h.no,
                   tf(a.L % 8 == 0 && a.T2 > 0), tf(a.T2 > 0));
    else
      r = snprintf(buf, n, "%sphi_syn_quad<%d, %d, %s>", ns, phi_quad_steps(a.L), k.waves, tf(a.T2 > 0));
  }
  return r < 0 ? -1 : 0;
}

}  // namespace yyg
