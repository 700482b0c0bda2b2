// C ABI of the Yin-Yang multipole solver: plan creation (tables), density
// upload, solve, exports.  See include/yyg.h for the contract.
#include "yyg.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <unordered_map>
#include <new>
#include <vector>

#include "yyg_internal.h"
#include "yyg_tables.h"

namespace {

constexpr int kSlots = 8;

struct TimedLaunch {
  int slot;
  hipEvent_t start, stop;
};

long round_up(long v, long m) { return (v + m - 1) / m * m; }

// Device memory the library holds, process-wide, against an optional cap:
// the environment variable YYG_MAX_DEVICE_BYTES (a decimal byte count; unset,
// empty, 0 or not a plain number: no cap), read at every allocation.  An
// allocation that would take the total past the cap fails like a failed
// hipMalloc, before the runtime is asked.  The buffers of folded dense solves
// (struct Fold) are spare: they are kept within the cap, but given up for any
// other allocation that does not fit beside them, and not part of the figure.
std::mutex g_mem_mu;
struct MemBlock {
  size_t bytes;
  bool spare;
};
std::unordered_map<void *, MemBlock> g_mem_blocks;
size_t g_mem_held = 0, g_mem_spare = 0;

size_t mem_cap() {
  const char *e = std::getenv("YYG_MAX_DEVICE_BYTES");
  if (!e || !*e) return 0;
  char *end = nullptr;
  const unsigned long long v = std::strtoull(e, &end, 10);
  return (end && *end == '\0' && e[0] != '-') ? (size_t)v : 0;
}

// One attempt; *beside: it failed with spare blocks held, without which it
// could fit.
hipError_t dev_malloc_once(void **p, size_t bytes, bool spare, bool *beside) {
  std::lock_guard<std::mutex> lock(g_mem_mu);
  const size_t cap = mem_cap();
  *p = nullptr;
  *beside = false;
  if (cap && (bytes > cap || g_mem_held > cap - bytes)) return hipErrorOutOfMemory;
  *beside = g_mem_spare > 0;
  if (cap && g_mem_held + g_mem_spare > cap - bytes) return hipErrorOutOfMemory;
  const hipError_t e = hipMalloc(p, bytes);
  if (e != hipSuccess) {
    *p = nullptr;
    return e;
  }
  if (*p) {
    g_mem_blocks[*p] = MemBlock{bytes, spare};
    (spare ? g_mem_spare : g_mem_held) += bytes;
  }
  return hipSuccess;
}

// The buffers of one folded dense solve are given up; false: none can be.
bool fold_reclaim();

hipError_t dev_malloc(void **p, size_t bytes) {
  bool beside;
  hipError_t e = dev_malloc_once(p, bytes, false, &beside);
  while (e == hipErrorOutOfMemory && beside && fold_reclaim()) {
    (void)hipGetLastError();
    e = dev_malloc_once(p, bytes, false, &beside);
  }
  return e;
}

hipError_t dev_free(void *p) {
  if (!p) return hipSuccess;
  {
    std::lock_guard<std::mutex> lock(g_mem_mu);
    auto it = g_mem_blocks.find(p);
    if (it != g_mem_blocks.end()) {
      (it->second.spare ? g_mem_spare : g_mem_held) -= it->second.bytes;
      g_mem_blocks.erase(it);
    }
  }
  return hipFree(p);
}

struct DeviceGuard {
  int prev = -1;
  bool ok = false;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    ok = hipSetDevice(dev) == hipSuccess;
  }
  ~DeviceGuard() {
    if (prev >= 0) (void)hipSetDevice(prev);
  }
};

}  // namespace

struct yyg_grid {
  int device = 0;
  int kind = YYG_GRID_YINYANG;
  int n_patch = 2;       // patches: 2 (Yin-Yang) or 1 (polar)
  int n_r = 0, n_t = 0, n_p = 0, L = 0, Q = 0;
  double G = 1.0;
  long nang = 0, ldb = 0, ldy = 0;
  int nsplit = 1;        // split-K factor of the analysis contraction
  int var_ana = 0;       // tile variant of the analysis contraction
  int var_syn = 0;       // tile variant of the synthesis contraction
  int part_cap = 1;      // splits the partial-moment buffer can hold
  int part_gen = 0;      // bumped whenever the partial-moment buffer moves
  std::vector<double> r_edges, w_host, nrm_q;
  yyg::PatchGeom geom;

  double *d_Bt = nullptr;    // analysis basis [Q][ldb]
  double *d_Y = nullptr;     // synthesis basis [nang][ldy], self | cross (cross on Yin-Yang only)
  double *d_coef = nullptr;  // radial coefficients [n_r][L+1][4]
  int *d_qdeg = nullptr;     // degree l of each column
  double *d_part = nullptr;  // split-K partial moments [nsplit][P n_r][Q]
  double *d_Ahat = nullptr;  // reduced moments (sqrt(N) scaled) [P n_r][Q], or [Q][P n_r] after a separable solve
  bool ahat_cols = false;    // d_Ahat holds the column-major layout
  double *d_U = nullptr;     // synthesis operand [P n_r][ldy]
  double *d_rho_owned = nullptr;
  bool ahat_fold = false;  // d_Ahat's columns are in the fold's order

  // dense FP64 solve folded about both mirror planes (yyg_dense_fold.hip);
  // class c holds columns cols[co[c] .. co[c] + N[c]).  Built where a density
  // is handed to a plan in the dense form, the form is chosen or FP64 prepared
  // or tuned (fold_try), so that plans of another form do not hold it, and
  // given back when memory runs short (fold_reclaim).
  struct Fold {
    std::atomic<bool> ready{false};  // the solve runs folded
    std::atomic<bool> tried{false};  // built, not to be had, or given back for memory: only asked for again
    bool captured = false;   // a recorded graph holds the buffers: kept to the plan's end
    int users = 0;           // calls on this plan that use them now
    int var_ana = 0, var_syn = 0, nsplit = 1;  // the contractions' tiles and split
    int splits = 0;          // splits that part holds
    double *part = nullptr;  // partial moments, where d_part holds fewer splits than nsplit
    long hq = 0;             // cells of a quarter patch
    long ldb = 0, ldy[4] = {};
    int N[4] = {}, co[4] = {};  // columns of a class, first one
    int K[4] = {}, ko[4] = {};  // synthesis contraction length of a class, first column in U
    std::vector<int> cols;   // column q at each place (kept when the buffers go: ahat_fold)
    int *d_cols = nullptr, *d_deg = nullptr;
    int2 *d_ucol = nullptr;
    double *Bt = nullptr;    // [Q][ldb]
    double *Y[4] = {};       // [hq][ldy[c]]
    double *F = nullptr;     // folded densities, then the classes' potentials [4][P n_r][hq]
  } fold;
  int cus = 256;  // compute units of the device (persistent grids)
  // opt-in check of the density for NaN / infinity before each solve
  bool check_finite = false;
  int *d_flag = nullptr;
  const double *rho = nullptr;

  // reduced-precision tables, index prec - 1 (FP32, BF16x3, FP16x2)
  struct Lp {
    bool ready = false;
    void *Bt = nullptr;  // analysis basis planes [parts][Q][ldb]
    int *eBt = nullptr;  // row exponents of the analysis basis
    long ldb = 0;
    void *Y = nullptr;   // synthesis basis planes [parts][nang][ldy]
    int *eY = nullptr;
    long ldy = 0;
    void *Ar = nullptr;  // density planes [parts][2 n_r][lda], split per solve
    long lda = 0;
    void *Ur = nullptr;  // synthesis-operand planes [parts][2 n_r][ldu]
    long ldu = 0;
    int var_ana = 0, nsplit = 1, var_syn = 0;
  } lp[3];
  int *d_eA = nullptr;  // row exponents of the density (FP16x2)
  int *d_eU = nullptr;  // row exponents of the synthesis operand (FP16x2)

  // separable form
  int method = YYG_METHOD_DENSE;
  struct Sep {
    bool ready = false;
    long ldk = 0, ldm = 0, ldl = 0;
    double *Wcs = nullptr;   // weighted phi-analysis basis [n_t][2L+1][ldk]: w_jk C/S_k^(m)
    double *trig = nullptr;  // phi-synthesis basis [n_p][ldm]
    double *T2 = nullptr;    // theta-analysis basis [mc][l][n_t]: sqrt(N) T_j^(lm)
    double *P2 = nullptr;    // theta-synthesis basis [mc][j][ldl]: sqrt(N) P_l^m(cos t_j)
    double *Drot = nullptr;  // per degree l: the rotation block D_l (d x d), one after the other
    double *X2 = nullptr;    // phi-analysis output [mc][j][row]
    double *V = nullptr;     // theta-synthesis output [mc][j][row]
    double *At = nullptr;    // own + rotated other moments, column-major [Q][row] (Yin-Yang)
    double *Ut = nullptr;    // potential coefficients of own + rotated other moments [mc][l][row]
    double *coefS = nullptr; // radial recurrence coefficients [L+1][4][n_r]
    // phi phases, strided batches over the colatitudes j: analysis (C
    // stored column-major) and synthesis (A stored k-major)
    yyg::GemmF64Args phi_ana{}, phi_syn{};
    // the same two as LDS-basis kernels
    yyg::PhiDirectArgs phi_ana_d{}, phi_syn_d{};
    // the same two folded about the patch's central meridian (the tile
    // variants use these when the grid is mirror-symmetric: fold = true)
    bool fold = false;
    long h = 0, ldkh = 0, ks = 0, ldtf = 0;  // folded length, its row stride; synthesis split and row stride
    long kcs = 0, nks = 0;   // LDS-free synthesis: cos slots and all slots
    double *WF = nullptr;    // folded analysis basis [n_t][2][L+1][ldkh]: even (cos) / odd (sin) halves
    double *TF = nullptr;    // folded synthesis basis [h][ldtf]: cos m at m, sin m at ks + m - 1
    yyg::GemmF64Args phi_ana_f{}, phi_syn_f{};
    yyg::PhiStreamArgs phi_syn_s{};  // streaming folded synthesis
    yyg::PhiAnaStreamArgs phi_ana_s{};  // streaming folded analysis
    double *CSF = nullptr;  // its colatitude-independent folded basis [16 (nte + nto)][ldcs]
    double *Wt = nullptr;   // its folded overlap weights [n_t][ldcs]
    // folded analysis, both halves per block: basis rows cos m at slot m
    // (m <= L), sin m at slot ks + m - 1, [n_t][ks + L][ldkh], exact weights
    double *WFAB = nullptr;
    yyg::GemmF64Args phi_ana_ab{};
    // folded about the central meridian and, where the grid allows, the
    // meridians 90 degrees off it
    yyg::PhiQuadArgs quad_ana{}, quad_syn{};
    double *QA = nullptr, *QS = nullptr, *QW = nullptr;  // their bases and the analysis weights
    // folded phi synthesis with the fragments loaded straight from memory
    double *BK = nullptr;    // its basis, slot-major [kcs + 4 ceil(L/4)][hp]
    long hp = 0;             // h padded to a multiple of 32
    yyg::PhiLeanArgs phi_syn_l{};
    // theta phases and rotation: one launch each over their problems
    yyg::SepPhaseArgs args{};
    // the same three with their operands straight from memory (stream[r]:
    // phase r = 1..3 can run so on this plan)
    yyg::ThetaArgs theta{};
    bool stream[4] = {false, false, false, false};
    double *TA = nullptr, *TS = nullptr, *DR = nullptr;  // folded theta bases, rotation blocks by class
    // variant per phase (0 phi analysis, 1 theta analysis, 2 moment
    // rotation, 3 theta synthesis, 4 phi synthesis): v < V the tile v,
    // V + v the same with the deep prefetch, 2V + d (phi phases) the
    // LDS-basis kernel d, 2V + D + f (phi phases, fold) the kernel f folded
    // about two meridians, 2V + D + F + e (phi synthesis, fold) the LDS-free
    // kernel e
    // defaults (before autotuning): 32 x 32 tiles, 64 x 32 for the theta
    // synthesis; the phi phases of a folded grid as sep_default_phi
    int var[5] = {10, 10, 10, 9, 10};
    // reduced-precision phi transforms (FP32, BF16 x 3): tile of the phi
    // analysis and of the phi synthesis (yyg::sep_lp_tile_count() shapes)
    int lpt[2][2] = {{0, 1}, {0, 1}};
  } sep;

  bool timing = false;
  std::vector<TimedLaunch> launches;
};

namespace {


hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

// Release the separable form's device buffers (after a failed build too,
// so that a retry starts from nothing).
void sep_release(yyg_grid *g) {
  auto &S = g->sep;
  double **b[] = {&S.Wcs, &S.trig, &S.T2, &S.P2, &S.Drot, &S.X2, &S.V,   &S.Ut,  &S.coefS,
                  &S.At,  &S.WF,   &S.TF, &S.QA, &S.QS, &S.QW, &S.TA, &S.TS, &S.DR, &S.BK, &S.WFAB, &S.CSF, &S.Wt};
  for (double **x : b) {
    if (*x) (void)dev_free(*x);
    *x = nullptr;
  }
}

// Release the operand planes of one reduced precision of the dense form.
template <class LpPlan>
void lp_release(LpPlan &l) {
  void **b[] = {reinterpret_cast<void **>(&l.Bt), reinterpret_cast<void **>(&l.eBt), reinterpret_cast<void **>(&l.Y),
                reinterpret_cast<void **>(&l.eY), reinterpret_cast<void **>(&l.Ar), reinterpret_cast<void **>(&l.Ur)};
  for (void **x : b) {
    if (*x) (void)dev_free(*x);
    *x = nullptr;
  }
}

// Plans whose fold is built, the oldest first.  The lock covers this list and
// the state of every fold in it; it is held over no launch and no table build.
std::mutex g_fold_mu;
std::vector<yyg_grid *> g_folds;

// Free a fold's buffers (under g_fold_mu once it is in the list).
void fold_free(yyg_grid *g) {
  auto &f = g->fold;
  void *b[] = {f.d_cols, f.d_deg, f.d_ucol, f.Bt, f.Y[0], f.Y[1], f.Y[2], f.Y[3], f.F, f.part};
  for (void *x : b)
    if (x) (void)dev_free(x);
  f.d_cols = f.d_deg = nullptr;
  f.d_ucol = nullptr;
  f.Bt = f.F = f.part = nullptr;
  for (double *&y : f.Y) y = nullptr;
  f.splits = 0;
  f.ready = false;
}

// Give back a fold that no call uses and no recorded graph holds, after the
// work on its device (under g_fold_mu).
bool fold_drop(yyg_grid *g) {
  auto &f = g->fold;
  if (!f.ready || f.users > 0 || f.captured) return false;
  DeviceGuard dg(g->device);
  if (!dg.ok || hipDeviceSynchronize() != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  fold_free(g);
  g_folds.erase(std::remove(g_folds.begin(), g_folds.end(), g), g_folds.end());
  return true;
}

bool fold_reclaim() {
  std::lock_guard<std::mutex> lock(g_fold_mu);
  for (yyg_grid *g : g_folds)
    if (fold_drop(g)) return true;
  return false;
}

// A plan's own fold, given back if it can be; `again`: to be built again when
// the dense form is next used.
void fold_release(yyg_grid *g, bool again) {
  std::lock_guard<std::mutex> lock(g_fold_mu);
  if (fold_drop(g) && again) g->fold.tried = false;
}

// Whether s is being recorded into a graph (the default stream cannot be).
bool capturing(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (s && hipStreamIsCapturing(s, &st) != hipSuccess) {
    (void)hipGetLastError();
    return true;  // not known
  }
  return st != hipStreamCaptureStatusNone;
}

// The fold of one call, held until the call has enqueued its work; `s` is the
// stream it goes to.
struct FoldUse {
  yyg_grid *g = nullptr;
  FoldUse(yyg_grid *plan, hipStream_t s) {
    if (!plan) return;
    std::lock_guard<std::mutex> lock(g_fold_mu);
    if (!plan->fold.ready) return;
    plan->fold.captured = plan->fold.captured || capturing(s);
    plan->fold.users += 1;
    g = plan;
  }
  void end() {
    if (!g) return;
    std::lock_guard<std::mutex> lock(g_fold_mu);
    g->fold.users -= 1;
    g = nullptr;
  }
  explicit operator bool() const { return g != nullptr; }
  ~FoldUse() { end(); }
  FoldUse(const FoldUse &) = delete;
  FoldUse &operator=(const FoldUse &) = delete;
};

void free_grid(yyg_grid *g) {
  if (!g) return;
  {
    std::lock_guard<std::mutex> lock(g_fold_mu);
    fold_free(g);
    g_folds.erase(std::remove(g_folds.begin(), g_folds.end(), g), g_folds.end());
  }
  double *bufs[] = {g->d_Bt, g->d_Y, g->d_coef, g->d_part, g->d_Ahat, g->d_U, g->d_rho_owned};
  (void)dev_free(g->d_flag);
  for (double *b : bufs)
    if (b) (void)dev_free(b);
  if (g->d_qdeg) (void)dev_free(g->d_qdeg);
  for (auto &l : g->lp) lp_release(l);
  if (g->d_eA) (void)dev_free(g->d_eA);
  if (g->d_eU) (void)dev_free(g->d_eU);
  sep_release(g);
  for (auto &t : g->launches) {
    (void)hipEventDestroy(t.start);
    (void)hipEventDestroy(t.stop);
  }
  delete g;
}

template <class T>
int dmalloc(T **p, size_t count) {
  if (dev_malloc(reinterpret_cast<void **>(p), count * sizeof(T)) != hipSuccess) {
    *p = nullptr;
    (void)hipGetLastError();
    return YYG_ERR_OUT_OF_MEMORY;
  }
  return YYG_OK;
}

// Record a start event if timing is on; returns the index of the record.
int timing_begin(yyg_grid *g, int slot, hipStream_t s) {
  if (!g->timing) return -1;
  TimedLaunch t{slot, nullptr, nullptr};
  if (hipEventCreate(&t.start) != hipSuccess || hipEventCreate(&t.stop) != hipSuccess) return -1;
  (void)hipEventRecord(t.start, s);
  g->launches.push_back(t);
  return (int)g->launches.size() - 1;
}
void timing_end(yyg_grid *g, int idx, hipStream_t s) {
  if (idx >= 0) (void)hipEventRecord(g->launches[idx].stop, s);
}

}  // namespace

namespace yyg {
int choose_split(long tiles, long K) {
  // Blocks resident at once: 256 CUs x 2 blocks.  Pick the smallest split
  // whose wave-quantised cost is within 10% of the best, keeping at least
  // four 16-wide k stages per split.
  const long slots = 512;
  long smax = std::max(1L, std::min(32L, K / 64));
  double best = 1e30;
  std::vector<double> cost(smax + 1);
  for (long s = 1; s <= smax; ++s) {
    long waves = (tiles * s + slots - 1) / slots;
    cost[s] = (double)waves / s;
    best = std::min(best, cost[s]);
  }
  for (long s = 1; s <= smax; ++s)
    if (cost[s] <= 1.1 * best) return (int)s;
  return 1;
}
}  // namespace yyg

namespace {

// Timing of one launch configuration: one warm-up, then the
// minimum over `reps` event-timed launches (timings are data-independent).
template <class F>
double time_launch(F launch, hipStream_t s, int reps) {
  hipEvent_t a, b;
  if (hipEventCreate(&a) != hipSuccess) return 1e30;
  if (hipEventCreate(&b) != hipSuccess) {
    (void)hipEventDestroy(a);
    return 1e30;
  }
  double best = 1e30;
  if (launch() == hipSuccess && hipStreamSynchronize(s) == hipSuccess) {
    for (int r = 0; r < reps; ++r) {
      (void)hipEventRecord(a, s);
      hipError_t e = launch();
      (void)hipEventRecord(b, s);
      if (e != hipSuccess || hipEventSynchronize(b) != hipSuccess) {
        best = 1e30;
        break;
      }
      float ms = 0.f;
      (void)hipEventElapsedTime(&ms, a, b);
      best = std::min(best, (double)ms);
    }
  }
  (void)hipGetLastError();
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  return best;
}

// Cells of the quarter patch.
long fold_cells(const yyg_grid *g) { return (long)((g->n_t + 1) / 2) * ((g->n_p + 1) / 2); }

// Columns of class c: the degrees l = m, m + 2, .. (odd: m + 1, ..) of its orders.
int fold_columns(int L, int c) {
  int n = 0;
  for (int m = c & 1; m <= L; ++m) n += c & 2 ? (L - m + 1) / 2 : (L - m) / 2 + 1;
  return n;
}

// Tiles of the four analysis contractions.
long fold_analysis_tiles(const yyg_grid *g, int bm, int bn) {
  const long M = (long)g->n_patch * g->n_r;
  long t = 0;
  for (int c = 0; c < 4; ++c) t += ((M + bm - 1) / bm) * ((fold_columns(g->L, c) + bn - 1) / bn);
  return t;
}

// Tile shapes and split of a new plan's folded contractions: 64 x 64 tiles of
// eight waves (variant 11), and 32 x 32 (variant 10) where those pad the
// product by over a tenth more, or give the synthesis under four tiles a CU.
// Measured (fold, contraction and scan; contraction and unfold): 2 degrees,
// 400 shells, degree 25: 64-wide 87 and 100 us, 32-wide 87 and 102, 128-wide
// 118 and 135; 4 degrees, 100 shells, degree 12: 29 and 13, 27 and 12, 42 and
// 30; 1 degree, 100 shells, degree 40 (rows pad by 1.14): 155 and 249, 151
// and 233, 187 and 297.  The split of 64-wide tiles is at least 2 over long
// contractions, where one wave of blocks leaves the last CUs idle.
void fold_shape(const yyg_grid *g, int *var_ana, int *var_syn, int *nsplit) {
  const long M = (long)g->n_patch * g->n_r, hq = fold_cells(g);
  const auto pad = [](long n, long b) { return (n + b - 1) / b * b; };
  const double rows = (double)pad(M, 64) / pad(M, 32);
  const long t64 = fold_analysis_tiles(g, 64, 64), t32 = fold_analysis_tiles(g, 32, 32);
  *var_ana = 4.0 * t64 <= 1.1 * t32 ? 11 : 10;
  *var_syn = rows * pad(hq, 64) / pad(hq, 32) <= 1.1 && 4 * (pad(M, 64) / 64) * (pad(hq, 64) / 64) >= 4L * g->cus ? 11 : 10;
  *nsplit = yyg::choose_split(*var_ana == 11 ? t64 : t32, hq);
  if (*var_ana == 11 && hq >= 1024) *nsplit = std::max(*nsplit, 2);
}

// Whether the dense FP64 solve of this plan is to run folded: a column in every
// class (L >= 2), rows within a launch's reach, and work enough to pay for two
// more launches (tuned plans: 1.0e6 products 22.7 us folded against 19.0,
// 1.2e7 26.4 against 30.0) ...
constexpr double kFoldMinMacs = 4e6;
bool fold_large(const yyg_grid *g) {
  const long M = (long)g->n_patch * g->n_r;
  return g->L >= 2 && M <= 65535 && (double)M * g->nang * g->Q * (1 + g->n_patch) >= kFoldMinMacs;
}

// ... and for the two passes over the density and the potential, which at low
// degrees cost more than the products that they save.  Solves, us, unfolded
// and folded: from degree 8 on the fold is always the faster (900 shells, 92 x
// 272 x 2: 611 and 572); at degrees 5 to 7 while the density, its fold and the
// potential fit the last-level cache together (degree 6, 200 shells of 47 x
// 137 x 2, 21 MB each: 61 and 58; 92 x 272 x 2, 80 MB: 130 and 122 to 129;
// 900 shells of 47 x 137 x 2, 93 MB: 145 and 177; of 92 x 272 x 2: 418 and
// 531; degree 5 at 80 MB: 109 and 129); below, only where few rows of many
// cells leave the unfolded analysis' CUs idle (degree 3, 50 shells of 92 x 272
// x 2: 65 and 61; 100 shells: 71 and 77; 200 of 24 x 70 x 2: 25 and 31).
bool fold_wanted(const yyg_grid *g) {
  if (!fold_large(g)) return false;
  const long M = (long)g->n_patch * g->n_r;
  if (g->L >= 5) return g->L >= 8 || 8.0 * M * g->nang <= (g->L == 5 ? 64e6 : 85e6);
  return g->n_patch == 2 && M <= 50 * g->L && g->nang > 12000;
}

// Tiles and split of a new plan of that size that solves unfolded: 32 x 32
// tiles, 64 x 64 (variant 11) where the columns and the rows fill them, and
// splits that grow with the root of the contraction and shrink with the rows,
// since the scan reads every split's moments.  Degree 3, us, splits 4 / 8 / 16
// / 32: 200 shells of 24 x 70 x 2 27 / 25 / 28 / 38, of 47 x 137 x 2 76 / 53 / 44
// / 48, of 92 x 272 x 2 243 / 144 / 97 / 85; 900 shells: 57 / 60 / 74 / 106, 113 /
// 100 / 106 / 134 and 467 / 340 / 302 / 337.
void low_degree_shape(const yyg_grid *g, int *var_ana, int *var_syn, int *nsplit) {
  const long M = (long)g->n_patch * g->n_r;
  *var_ana = g->L >= 5 ? 11 : 10;
  *var_syn = 8.0 * M * g->nang > 64e6 ? 11 : 10;
  const double split = std::sqrt((double)g->nang) / 4.75 * std::sqrt(std::min(1.0, 600.0 / M));
  *nsplit = std::max(1, std::min(32, (int)std::lround(split)));
}

// The fold's tables, built on a stream of their own (no other stream has to
// wait, and a capture under way elsewhere is not disturbed).  No other fold is
// given up for this one.  False (not wanted, memory short, or a table without
// the symmetry): the plan solves unfolded.
bool fold_build(yyg_grid *g, hipStream_t s) {
  auto &f = g->fold;
  const int Q = g->Q, P = g->n_patch;
  const long M = (long)P * g->n_r;
  f.hq = fold_cells(g);
  f.ldb = round_up(f.hq, 16);
  std::vector<int> deg, ycols, cols;
  std::vector<int2> ucol;
  int yo[4];
  const auto swapped = [](int c) { return (c >> 1) | (c & 1) << 1; };
  try {
    const auto tab = yyg::column_table(g->L);
    for (int c = 0; c < 4; ++c) {
      f.co[c] = (int)cols.size();
      for (int q = 0; q < Q; ++q)
        if ((((tab[q].l + tab[q].m) & 1) << 1 | (tab[q].is_sin ? 1 : 0)) == c) cols.push_back(q);
      f.N[c] = (int)cols.size() - f.co[c];
    }
    for (int c = 0, at = 0; c < 4; at += f.K[c++]) {
      f.ko[c] = at;
      f.K[c] = f.N[c] + (P == 2 ? f.N[swapped(c)] : 0);
      f.ldy[c] = round_up(f.K[c], 16);
      yo[c] = (int)ycols.size();
      for (int i = 0; i < f.N[c]; ++i) ycols.push_back(cols[f.co[c] + i]);
      for (int i = 0; P == 2 && i < f.N[swapped(c)]; ++i) ycols.push_back(Q + cols[f.co[swapped(c)] + i]);
    }
    for (int c = 0; c < 4; ++c)
      for (int i = 0; i < f.N[c]; ++i) {
        deg.push_back(tab[cols[f.co[c] + i]].l);
        ucol.push_back(int2{f.ko[c] + i, f.ko[swapped(c)] + f.N[swapped(c)] + i});
      }
  } catch (const std::bad_alloc &) {
    return false;
  }
  int *d_ycols = nullptr, *d_flag = nullptr;
  auto take = [](auto **p, size_t n) {
    bool beside;
    if (dev_malloc_once(reinterpret_cast<void **>(p), n * sizeof(**p), true, &beside) == hipSuccess) return YYG_OK;
    (void)hipGetLastError();
    return YYG_ERR_OUT_OF_MEMORY;
  };
  int st = take(&f.d_cols, (size_t)Q);
  if (st == YYG_OK) st = take(&f.d_deg, (size_t)Q);
  if (st == YYG_OK) st = take(&f.d_ucol, (size_t)Q);
  if (st == YYG_OK) st = take(&f.Bt, (size_t)Q * f.ldb);
  for (int c = 0; c < 4 && st == YYG_OK; ++c) st = take(&f.Y[c], (size_t)f.hq * f.ldy[c]);
  if (st == YYG_OK) st = take(&f.F, (size_t)4 * M * f.hq);
  if (st == YYG_OK && f.nsplit > g->part_cap) {
    st = take(&f.part, (size_t)f.nsplit * M * Q);
    f.splits = f.nsplit;
  }
  if (st == YYG_OK) st = take(&d_ycols, ycols.size());
  if (st == YYG_OK) st = take(&d_flag, 1);
  hipError_t e = st == YYG_OK ? hipSuccess : hipErrorOutOfMemory;
  auto chk = [&](hipError_t r) {
    if (e == hipSuccess && r != hipSuccess) e = r;
  };
  int bad = 0;
  if (e == hipSuccess) {
    chk(hipMemcpyAsync(f.d_cols, cols.data(), Q * sizeof(int), hipMemcpyHostToDevice, s));
    chk(hipMemcpyAsync(f.d_deg, deg.data(), Q * sizeof(int), hipMemcpyHostToDevice, s));
    chk(hipMemcpyAsync(f.d_ucol, ucol.data(), Q * sizeof(int2), hipMemcpyHostToDevice, s));
    chk(hipMemcpyAsync(d_ycols, ycols.data(), ycols.size() * sizeof(int), hipMemcpyHostToDevice, s));
    chk(hipMemcpyAsync(d_flag, &bad, sizeof(int), hipMemcpyHostToDevice, s));
    for (int c = 0; c < 4 && e == hipSuccess; ++c) {
      chk(yyg::launch_fold_analysis_basis(g->d_Bt, g->ldb, f.d_cols + f.co[c], f.N[c], c, g->n_t, g->n_p,
                                          f.Bt + f.co[c] * f.ldb, f.ldb, d_flag, s));
      chk(yyg::launch_fold_synthesis_basis(g->d_Y, g->ldy, d_ycols + yo[c], f.K[c], c, g->n_t, g->n_p, f.Y[c],
                                           f.ldy[c], d_flag, s));
    }
    chk(hipMemcpyAsync(&bad, d_flag, sizeof(int), hipMemcpyDeviceToHost, s));
    chk(hipStreamSynchronize(s));
  }
  if (d_ycols) (void)dev_free(d_ycols);
  if (d_flag) (void)dev_free(d_flag);
  if (e != hipSuccess) (void)hipGetLastError();
  if (e == hipSuccess && bad == 0) f.cols.swap(cols);
  return e == hipSuccess && bad == 0;
}

// Build the fold of a plan that has none.
void fold_try(yyg_grid *g) {
  auto &f = g->fold;
  if (f.ready || !fold_wanted(g)) return;
  DeviceGuard dg(g->device);
  if (!dg.ok) return;
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
  hipStream_t s = nullptr;
  bool ok = hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess;
  if (ok) {
    ok = fold_build(g, s);
    (void)hipStreamDestroy(s);
  }
  if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
  (void)hipGetLastError();
  std::lock_guard<std::mutex> lock(g_fold_mu);
  f.tried = true;
  if (ok) try {
      g_folds.push_back(g);
    } catch (const std::bad_alloc &) {
      ok = false;
    }
  if (!ok) fold_free(g);
  f.ready = ok;
}


// The four classes' analysis contractions over the folded densities in F;
// part [nsplit][M][Q], columns in the fold's order.
hipError_t fold_analysis(yyg_grid *g, int variant, int nsplit, double *part, hipStream_t s) {
  const auto &f = g->fold;
  const long M = (long)g->n_patch * g->n_r;
  yyg::GemmF64Quad q{};
  for (int c = 0; c < 4; ++c)
    q.g[c] = yyg::GemmF64Args{(int)M, f.N[c], (int)f.hq, f.F + c * M * f.hq, f.hq, f.Bt + f.co[c] * f.ldb, f.ldb,
                              part + f.co[c], g->Q, M * g->Q, 0, 0};
  return yyg::launch_gemm_f64_quad(variant, 0, q, nsplit, s);
}

// The four classes' potentials on the quarter patch, into F.
hipError_t fold_synthesis(yyg_grid *g, int variant, hipStream_t s) {
  const auto &f = g->fold;
  const long M = (long)g->n_patch * g->n_r;
  yyg::GemmF64Quad q{};
  for (int c = 0; c < 4; ++c)
    q.g[c] = yyg::GemmF64Args{(int)M, (int)f.hq, f.K[c], g->d_U + f.ko[c], g->ldy, f.Y[c], f.ldy[c],
                              f.F + c * M * f.hq, f.hq, 0, 0, 0};
  return yyg::launch_gemm_f64_quad(variant, 1, q, 1, s);
}

std::string tune_key(int prec, int role, long M, long N, long K) {
  char buf[128];
  std::snprintf(buf, sizeof buf, "p%d r%d %ld %ld %ld", prec, role, M, N, K);
  return buf;
}

std::map<std::string, std::pair<int, int>> read_tune_cache(const char *path) {
  std::map<std::string, std::pair<int, int>> m;
  if (!path) return m;
  std::FILE *f = std::fopen(path, "r");
  if (!f) return m;
  char line[256];
  while (std::fgets(line, sizeof line, f)) {
    int p, r, v, sp;
    long M, N, K;
    if (std::sscanf(line, "p%d r%d %ld %ld %ld -> %d %d", &p, &r, &M, &N, &K, &v, &sp) == 7)
      m[tune_key(p, r, M, N, K)] = {v, sp};
  }
  std::fclose(f);
  return m;
}

}  // namespace


namespace {

// Variants of separable phase r: v < V the tile v, V + v the same with
// three stages of loads in flight (V = the FP64 tile variants); the phi
// phases (0, 4) also 2V + d, the LDS-basis kernel variant d (d < D), and
// 2V + D + f, the kernel f folded about two meridians (F of them;
// mirror-symmetric grids only);
// the phi synthesis also 2V + D + F + e, the LDS-free folded kernel e.
// Every phase then takes X = yyg::x4_variant_count() tiles on the 4x4x4
// FP64 MFMA at the end of its range (sep_x4_base).
int sep_x4_base(int r) {
  const int v = 2 * yyg::gemm_f64_variant_count();
  const int phi = yyg::phi_direct_variant_count() + yyg::phi_quad_variant_count();
  return r == 0 ? v + phi : r == 4 ? v + phi + yyg::phi_lean_variant_count() : v;
}

// The phi transforms then take the streaming kernels after those (folded
// grids only): yyg::phi_ana_stream_variant_count() for the analysis,
// yyg::phi_stream_variant_count() for the synthesis.
int sep_stream_base(int r) { return sep_x4_base(r) + yyg::x4_variant_count(r); }

int sep_stream_count(int r) {
  return r == 0 ? yyg::phi_ana_stream_variant_count() : r == 4 ? yyg::phi_stream_variant_count() : 0;
}

// The phi analysis last takes yyg::fold_xcol_variant_count() folded tiles
// whose last output column is summed on the vector units (folded grids only).
int sep_xcol_base(int r) { return sep_stream_base(r) + sep_stream_count(r); }

int sep_variant_count(int r) { return sep_xcol_base(r) + (r == 0 ? yyg::fold_xcol_variant_count() : 0); }

bool sep_fold_variant(int r, int v) {
  if ((r == 0 || r == 4) && v >= sep_stream_base(r)) return true;
  if (v >= sep_x4_base(r)) return yyg::x4_fold_only(r, v - sep_x4_base(r)) != 0;
  return (r == 0 || r == 4) && v >= 2 * yyg::gemm_f64_variant_count() + yyg::phi_direct_variant_count();
}

// Whether variant v of phase r can run on this plan's grid and degree.
bool sep_variant_available(const yyg_grid *g, int r, int v) {
  if (r < 0 || r > 4 || v < 0 || v >= sep_variant_count(r)) return false;
  if (sep_fold_variant(r, v) && !g->sep.fold) return false;
  if (r == 4 && v >= sep_stream_base(4)) return yyg::phi_stream_supports(v - sep_stream_base(4), g->L);
  if (r == 0 && v >= sep_xcol_base(0)) return true;
  if (r == 0 && v >= sep_stream_base(0))
    return yyg::phi_ana_stream_supports(v - sep_stream_base(0), (int)g->sep.h, g->n_p);
  return true;
}

int sep_set_variant(yyg_grid *g, int r, int v) {
  if (r < 0 || r > 4 || v < 0 || v >= sep_variant_count(r)) return YYG_ERR_INVALID_ARG;
  if (!sep_variant_available(g, r, v)) return YYG_ERR_UNSUPPORTED;
  g->sep.var[r] = v;
  return YYG_OK;
}

// Variants V + 4 and V + 5 of phases 1-3 (the two largest tiles with three
// stages in flight, far wider than these problems) run the kernels of
// yyg_theta.hip where the plan allows.
int sep_theta_variant(const yyg_grid *g, int r, int v) {
  const int u = v - yyg::gemm_f64_variant_count() - 4;
  return r >= 1 && r <= 3 && (u == 0 || u == 1) && g->sep.stream[r] ? u : -1;
}

hipError_t sep_launch_phase(yyg_grid *g, int r, hipStream_t s) {
  auto &S = g->sep;
  if (const int u = sep_theta_variant(g, r, S.var[r]); u >= 0) {
    if (r == 2 && g->n_patch != 2) return hipSuccess;
    return yyg::launch_theta_stream(r, u, S.theta, g->cus, s);
  }
  const int nv = yyg::gemm_f64_variant_count(), nd = yyg::phi_direct_variant_count();
  const int nf = yyg::phi_quad_variant_count();
  if (r == 4 && S.var[r] >= sep_stream_base(4))
    return yyg::launch_phi_syn_stream(S.var[r] - sep_stream_base(4), S.phi_syn_s, g->cus, s);
  if (r == 0 && S.var[r] >= sep_xcol_base(0)) return yyg::launch_fold_xcol(S.var[r] - sep_xcol_base(0), S.phi_ana_f, s);
  if (r == 0 && S.var[r] >= sep_stream_base(0))
    return yyg::launch_phi_ana_stream(S.var[r] - sep_stream_base(0), S.phi_ana_s, g->cus, s);
  if (S.var[r] >= sep_x4_base(r)) {
    if (r == 2 && g->n_patch != 2) return hipSuccess;
    const yyg::GemmF64Args &phi = r == 0 ? (S.fold ? S.phi_ana_f : S.phi_ana) : (S.fold ? S.phi_syn_f : S.phi_syn);
    return yyg::launch_x4_sep_phase(S.var[r] - sep_x4_base(r), r, S.fold, phi, S.phi_ana_ab, S.args, s);
  }
  if (r == 4 && S.var[r] >= 2 * nv + nd + nf) return yyg::launch_phi_syn_lean(S.var[r] - 2 * nv - nd - nf, S.phi_syn_l, s);
  if (sep_fold_variant(r, S.var[r])) {
    return yyg::launch_phi_quad(S.var[r] - 2 * nv - nd, r == 0, r == 0 ? S.quad_ana : S.quad_syn, g->cus, s);
  }
  if ((r == 0 || r == 4) && S.var[r] >= 2 * nv)
    return yyg::launch_phi_direct(S.var[r] - 2 * nv, r == 0, r == 0 ? S.phi_ana_d : S.phi_syn_d, s);
  const int v = S.var[r] % nv;
  const bool deep = S.var[r] >= nv;
  const int dr = deep ? yyg::kRoleDeep : 0;
  if (r == 0) return yyg::launch_gemm_f64_batched(v, (S.fold ? 2 : 0) + dr, S.fold ? S.phi_ana_f : S.phi_ana, s);
  if (r == 4) return yyg::launch_gemm_f64_batched(v, (S.fold ? 3 : 1) + dr, S.fold ? S.phi_syn_f : S.phi_syn, s);
  if (r == 2 && g->n_patch != 2) return hipSuccess;  // one patch: nothing to rotate
  return yyg::launch_gemm_f64_sep(v, r, deep, S.args, s);
}

// Work buffers of the separable form: the plan's own, or (allocation-free
// solve) regions of the device scratch array.
struct SepWork {
  double *X2, *V, *Ut, *At, *Ahat;
};

SepWork sep_work(const yyg_grid *g) { return {g->sep.X2, g->sep.V, g->sep.Ut, g->sep.At, g->d_Ahat}; }

// Point every launch argument of the separable form at the work buffers w.
void sep_bind_work(yyg_grid *g, const SepWork &w) {
  auto &S = g->sep;
  S.X2 = w.X2;
  S.V = w.V;
  S.Ut = w.Ut;
  S.At = w.At;
  g->d_Ahat = w.Ahat;
  S.phi_ana.C = S.phi_ana_f.C = S.phi_ana_ab.C = w.X2;
  S.phi_ana_d.C = S.quad_ana.C = w.X2;
  S.phi_syn.A = S.phi_syn_f.A = w.V;
  S.phi_syn_s.V = w.V;
  S.phi_ana_s.X2 = w.X2;
  S.phi_syn_d.X = S.quad_syn.X = w.V;
  S.phi_syn_l.V = w.V;
  S.args.X2 = w.X2;
  S.args.Ut = w.Ut;
  S.args.Ahat = w.Ahat;
  S.args.At = w.At;
  S.args.V = w.V;
  S.theta.X2 = w.X2;
  S.theta.Ut = w.Ut;
  S.theta.Ahat = w.Ahat;
  S.theta.At = w.At;
  S.theta.V = w.V;
}

// Doubles of the separable form's work buffers, each region rounded up to
// 256 bytes.
size_t sep_work_doubles(const yyg_grid *g) {
  const long M = (long)g->n_patch * g->n_r, nmc = 2L * g->L + 1;
  auto r32 = [](long v) { return (size_t)((v + 31) / 32 * 32); };
  return 2 * r32(nmc * g->n_t * M) + r32(nmc * (g->L + 1) * M) + (g->n_patch == 2 ? r32(M * g->Q) : 0) +
         r32(M * g->Q);
}

// Point the phi phases at this solve's density and potential (kernel
// arguments: nothing is copied).
int sep_set_pointers(yyg_grid *g, const double *rho, double *phi, hipStream_t) {
  g->sep.phi_ana.A = rho;
  g->sep.phi_syn.C = phi;
  g->sep.phi_ana_d.X = rho;
  g->sep.phi_syn_d.C = phi;
  g->sep.phi_ana_f.A = rho;
  g->sep.phi_ana_s.rho = rho;
  g->sep.phi_ana_ab.A = rho;
  g->sep.phi_syn_f.C = phi;
  g->sep.phi_syn_s.phi = phi;
  g->sep.quad_ana.X = rho;
  g->sep.quad_syn.C = phi;
  g->sep.phi_syn_l.C = phi;
  return YYG_OK;
}

// The fold about two meridians (yyg::PhiQuadArgs): its index ranges, bases
// and weights.  The central fold holds (S.fold); the one about the meridians
// 90 degrees off the centre pairs front cells k and cc - k where the cell
// spacing divides 180 degrees (cc = np - 1 - 180 / spacing) and the C / S and
// trig tables show the parity to 1e-12 of their largest entry.  The tables
// halve a cell that is its own mirror or partner.
void sep_quad_tables(yyg_grid *g, const std::vector<double> &CSt, const std::vector<double> &trig,
                     std::vector<double> &QA, std::vector<double> &QS, std::vector<double> &QW) {
  auto &S = g->sep;
  const int L = g->L, nt = g->n_t, np = g->n_p, h = (int)S.h;
  auto mcol = [](int gr, int o, int *m) {
    *m = 2 * o + (gr == 0 ? 0 : gr == 2 ? 2 : 1);
    return gr < 2 ? std::max(2 * *m - 1, 0) : 2 * *m;
  };
  const double spacing = g->geom.ph[1] - g->geom.ph[0], ccx = np - 1 - M_PI / spacing;
  int cc = (int)std::lround(ccx);
  bool pair = std::fabs(ccx - cc) < 1e-6 && cc >= 1 && cc < h;
  if (pair) {
    double cmax = 0.0, bad = 0.0, tbad = 0.0;
    for (double v : CSt) cmax = std::max(cmax, std::fabs(v));
    for (int k = 0; k <= cc; ++k)
      for (int mc = 0; mc < 2 * L + 1; ++mc) {
        const int m = (mc + 1) / 2;
        const double sg = (m % 2 ? -1.0 : 1.0) * ((mc > 0 && mc % 2 == 0) ? -1.0 : 1.0);
        bad = std::max(bad, std::fabs(CSt[(size_t)mc * S.ldk + k] - sg * CSt[(size_t)mc * S.ldk + cc - k]));
        tbad = std::max(tbad, std::fabs(trig[(size_t)k * S.ldm + mc] - sg * trig[(size_t)(cc - k) * S.ldm + mc]));
      }
    pair = bad <= 1e-12 * cmax && tbad <= 1e-12;
  }
  const int f0 = pair ? (cc + 1) / 2 : 0, T2 = pair ? cc - f0 + 1 : 0, K = h - f0;
  // the analysis loads pairs of points: its partners end on a whole pair
  const int pad = T2 % 2;
  auto &A = S.quad_ana, &B = S.quad_syn;
  A.f0 = f0 - pad;
  A.tlo = pad;
  A.K = K + pad;
  A.T2 = pair ? T2 + pad : 0;
  B.f0 = f0;
  B.tlo = 0;
  B.K = K;
  B.T2 = T2;
  A.cc = B.cc = pair ? cc : 0;
  A.S = (A.K + 15) / 16;
  B.S = (K + 15) / 16;
  A.Kp = 16 * A.S;
  B.Kp = 16 * B.S;
  const int tj = yyg::phi_quad_tiles(L), ch = yyg::phi_quad_chunk(L);
  QA.assign((size_t)A.S * ch, 0.0);
  auto half = [&](int f) { return (np - 1 - f == f ? 0.5 : 1.0) * (pair && cc - f == f ? 0.5 : 1.0); };
  for (int t = A.tlo; t < A.K; ++t) {
    const int f = A.f0 + t, s = t / 16, g4 = t % 16 / 4, hf = t % 4 / 2;
    double *c = &QA[(size_t)s * ch];
    for (int gr = 0; gr < 4; ++gr)
      for (int o = 0, m; o < 16 * tj; ++o) {
        const int mc = mcol(gr, o, &m);
        if (m <= L)
          c[((gr * tj + o / 16) * 2 + hf) * 128 + 2 * (16 * g4 + o % 16) + t % 2] = half(f) * CSt[(size_t)mc * S.ldk + f];
      }
    if (yyg::phi_quad_extra(L)) c[4 * tj * 256 + t % 16] = half(f) * CSt[(size_t)(2 * L - 1) * S.ldk + f];
  }
  const int nq2 = (yyg::phi_quad_steps(L) + 1) / 2;
  QS.assign((size_t)((B.S + 1) / 2 * 2) * 4 * nq2 * 128, 0.0);
  for (int t = 0; t < K; ++t) {
    double *c = &QS[(size_t)(t / 16) * 4 * nq2 * 128];
    for (int gr = 0; gr < 4; ++gr)
      for (int o = 0, m; o < 8 * nq2; ++o) {
        const int mc = mcol(gr, o, &m), q = o / 4;
        if (m <= L) c[(gr * nq2 + q / 2) * 128 + 2 * (16 * (o % 4) + t % 16) + q % 2] = trig[(size_t)(f0 + t) * S.ldm + mc];
      }
  }
  QW.clear();
  if (g->n_patch == 2) {
    QW.assign((size_t)nt * 2 * A.Kp, 0.0);
    auto wmean = [&](int j, int k) {
      return 0.5 * (g->w_host[(size_t)j * np + k] + g->w_host[(size_t)j * np + np - 1 - k]);
    };
    for (int j = 0; j < nt; ++j)
      for (int t = A.tlo; t < A.K; ++t) {
        QW[((size_t)j * 2 + 0) * A.Kp + t] = wmean(j, A.f0 + t);
        if (t < A.T2) QW[((size_t)j * 2 + 1) * A.Kp + t] = wmean(j, cc - A.f0 - t);
      }
  }
}

// Folded bases of the theta phases (yyg::ThetaArgs) from the tables T and P
// [j][q], and which of phases 1-3 can run from memory: the theta phases where
// the tables show the parity (-1)^(l + m) about the equator to 1e-12 of
// their largest entry, the rotation where D_l vanishes outside the parity
// classes to 1e-12 (its entries are at most 1), each where its kernel holds
// the degree.
void sep_theta_tables(yyg_grid *g, const std::vector<double> &T, const std::vector<double> &P,
                      const std::vector<double> &D, std::vector<double> &TA, std::vector<double> &TS,
                      std::vector<double> &DR) {
  auto &S = g->sep;
  const int L = g->L, Q = g->Q, nt = g->n_t, h = (nt + 1) / 2;
  auto odd = [&](const std::vector<double> &X) {
    double top = 0.0, bad = 0.0;
    for (double v : X) top = std::max(top, std::fabs(v));
    for (int l = 0; l <= L; ++l)
      for (int m = 0; m <= l; ++m) {
        const int q = l * l + (m ? 2 * m : 0);
        const double sg = (l + m) % 2 ? -1.0 : 1.0;
        for (int j = 0; j < h; ++j)
          bad = std::max(bad, std::fabs(X[(size_t)j * Q + q] - sg * X[(size_t)(nt - 1 - j) * Q + q]));
      }
    return bad > 1e-12 * top;
  };
  S.stream[1] = yyg::theta_stream_fits(1, L, h) && !odd(T);
  S.stream[3] = yyg::theta_stream_fits(3, L, h) && !odd(P);
  S.stream[2] = g->n_patch == 2 && yyg::theta_stream_fits(2, L, h);
  // the class of a column within its degree (cos / sin, parity of m), the
  // class of the other patch it takes, a class's members
  auto cls = [](int b) {
    const int m = (b + 1) / 2;
    return b > 0 && b % 2 == 0 ? 2 + m % 2 : m % 2;
  };
  auto from = [](int l, int c) { return l % 2 ? (c == 0 ? 3 : c == 3 ? 0 : c) : (c == 1 ? 2 : c == 2 ? 1 : c); };
  auto member = [](int c, int i) { return c == 0 ? std::max(4 * i - 1, 0) : c == 1 ? 4 * i + 1 : c == 2 ? 4 * i + 4 : 4 * i + 2; };
  auto members = [](int l, int c) { return c == 0 ? l / 2 + 1 : c == 2 ? l / 2 : (l + 1) / 2; };
  size_t off = 0;
  for (int l = 0; l <= L && S.stream[2]; ++l) {
    const int d = 2 * l + 1;
    for (int k = 0; k < d; ++k)
      for (int b = 0; b < d; ++b)
        if (cls(k) != from(l, cls(b)) && std::fabs(D[off + (size_t)k * d + b]) > 1e-12) S.stream[2] = false;
    off += (size_t)d * d;
  }
  DR.clear();
  if (S.stream[2]) {
    const size_t std_ = yyg::rotation_doubles(L);
    DR.assign((size_t)4 * (L + 1) * std_, 0.0);
    off = 0;
    for (int l = 0; l <= L; ++l) {
      const int d = 2 * l + 1;
      for (int c = 0; c < 4; ++c) {
        const int nb = members(l, c), kq = (nb + 3) / 4;
        for (int i = 0; i < nb; ++i)
          for (int k = 0; k < nb; ++k)
            DR[(4 * (size_t)l + c) * std_ + ((size_t)(i / 16) * kq + k / 4) * 64 + 16 * (k % 4) + i % 16] =
                D[off + (size_t)member(from(l, c), k) * d + member(c, i)];
      }
      off += (size_t)d * d;
    }
  }
  const size_t sta = yyg::theta_ana_doubles(L, h), sts = yyg::theta_syn_doubles(L, h);
  TA.clear();
  TS.clear();
  if (S.stream[1]) TA.assign((size_t)(L + 1) * sta, 0.0);
  if (S.stream[3]) TS.assign((size_t)(L + 1) * sts, 0.0);
  for (int m = 0; m <= L; ++m) {
    const int t1 = ((L - m) / 2 + 16) / 16, kp = ((L - m) / 2 + 8) / 8;
    for (int l = m; l <= L; ++l) {
      const int par = (l - m) % 2, i = (l - m) / 2, q = l * l + (m ? 2 * m : 0);
      for (int j = 0; j < h; ++j) {
        const int qa = j / 4, qs = i / 4;
        if (S.stream[1])
          TA[m * sta + (((size_t)(qa / 2) * 2 + par) * t1 + i / 16) * 128 + 2 * (16 * (j % 4) + i % 16) + qa % 2] =
              (nt - 1 - j == j ? 0.5 : 1.0) * T[(size_t)j * Q + q];
        if (S.stream[3])
          TS[m * sts + (((size_t)(j / 16) * kp + qs / 2) * 2 + par) * 128 + 2 * (16 * (i % 4) + j % 16) + qs % 2] =
              P[(size_t)j * Q + q];
      }
    }
  }
}

// Default kernels of the phi phases on a folded grid: those of
// yyg_phi_quad.hip, or the 32 x 32 tiles (S.var's start) where a row tile's
// cells, which a wave of the sweep takes in turn, are many and the waves few.
void sep_default_phi(yyg_grid *g) {
  auto &S = g->sep;
  const int base = 2 * yyg::gemm_f64_variant_count() + yyg::phi_direct_variant_count();
  const int ana = yyg::phi_quad_default(true, S.quad_ana, g->cus);
  const int syn = yyg::phi_quad_default(false, S.quad_syn, g->cus);
  const long tiles = (long)g->n_t * (((long)g->n_patch * g->n_r + 15) / 16), cus = g->cus;
  // Analysis.  Without partners a short one gains nothing from the parity
  // split: 131 shells of 61 x 187 cells, lmax 23: 11.2 us in the tiles, 11.6 in
  // the sweep; nor does one of fewer row tiles than four a CU (a solve, us:
  // 100 shells of 90 x 180 cells, one patch, lmax 12 29.5 and 30.6; 200 of
  // 32 x 92, lmax 16 30.8 and 31.5; 400 of 47 x 137, 2350 row tiles, the sweep
  // by 2); nor one of low degree on rows too long for the form with the basis
  // in registers until twelve a CU (400 shells of 90 x 1000, lmax 10 228 and
  // 238; 300 of 180 x 1000, 3420 row tiles, 336 and 330; lmax 30 249 and 248).
  const bool long_ana = S.quad_ana.S > 12 && g->L < 24 && tiles < 12 * cus;
  if (ana == 0 || (S.quad_ana.T2 > 0 && tiles >= 4 * cus && !long_ana)) S.var[0] = base + ana;
  // Synthesis, a solve in the tiles and in the sweep, us.  Few row tiles: 14
  // of 2 x 2000 cells, lmax 8 40 and 64; 160 of 40 x 800, lmax 10 33 and 41; 400
  // of 25 x 320, lmax 10 29.2 and 31.1; 640 of 40 x 320 33.6 and 33.8; 500 of
  // 20 x 840, lmax 20 60 and 57.  Long rows of few columns, which the sweep
  // keeps open all its life: 2250 row tiles of 90 x 1000 cells, lmax 10 206 and
  // 238, lmax 30 238 and 248, lmax 40 292 and 283; 960 of 60 x 1000, lmax 10 71
  // and 73, lmax 20 87 and 78; without partners 5700 of 150 x 450, lmax 10 235
  // and 252, 2500 of 100 x 500, lmax 20 144 and 142; 3420 of 180 x 1600, lmax 10
  // 404 and 375.  One column (lmax 0): three of the sweep's four sums are empty
  // (300 shells of 92 x 272 x 2: 63 and 66).
  const int cells = S.quad_syn.S;
  const bool few = cells >= 3 && 4 * tiles < 7 * cus;
  const bool long_syn = cells > 12 && cells <= 20 && g->L < (S.quad_syn.T2 > 0 && tiles >= 8 * cus ? 32 : 16);
  if (g->L > 0 && (syn == 0 || (!few && !long_syn))) S.var[4] = base + syn;
}

int sep_build(yyg_grid *g) {
  auto &S = g->sep;
  const int L = g->L, Q = g->Q, nmc = 2 * L + 1, nt = g->n_t, np = g->n_p;
  const long M = (long)g->n_patch * g->n_r;
  const long MJ = M * nt;  // (row, j) pairs
  S.ldk = round_up(np, 16);
  S.ldm = round_up(nmc, 16);
  S.ldl = round_up(L + 1, 16);
  if (!yyg::radial_scan_q_supports(g->n_r, g->n_patch)) return YYG_ERR_UNSUPPORTED;
  std::vector<double> CSt, Wcs, trig, T, P, T2, P2, D, coef, coefS, WF, TF, BK, WFAB, CSF, WTF, QA, QS, QW, TA, TS, DR;
  int nte = 0, nto = 0, ldcs = 0;
  try {
    coef.resize((size_t)4 * g->n_r * (L + 1));
    yyg::radial_coefficients(g->n_r, g->r_edges.data(), L, coef.data());
    coefS.resize(coef.size());
    for (int n = 0; n < g->n_r; ++n)
      for (int l = 0; l <= L; ++l)
        for (int k = 0; k < 4; ++k)
          coefS[((size_t)l * 4 + k) * g->n_r + n] = coef[((size_t)n * (L + 1) + l) * 4 + k];
    CSt.resize((size_t)nmc * S.ldk);
    yyg::separable_cs(g->geom, L, S.ldk, CSt.data());
    // the overlap weights folded into one basis copy per colatitude
    Wcs.assign((size_t)nt * nmc * S.ldk, 0.0);
    for (int j = 0; j < nt; ++j)
      for (int mc = 0; mc < nmc; ++mc)
        for (int k = 0; k < np; ++k)
          Wcs[((size_t)j * nmc + mc) * S.ldk + k] = g->w_host[(size_t)j * np + k] * CSt[(size_t)mc * S.ldk + k];
    trig.resize((size_t)np * S.ldm);
    yyg::separable_trig(g->geom, L, S.ldm, trig.data());
    // Mirror symmetry about the central meridian: the cell centres, overlap
    // weights and cos / sin bases are even / odd under k -> n_p - 1 - k (up
    // to rounding), so each phi transform folds into an even and an odd
    // half of ceil(n_p / 2) points.  The bases are closed forms, symmetric
    // to a few ulps; a weight is the covered fraction of a cell, the
    // difference of O(1) terms over the cell's solid angle, so its rounding
    // grows as the cells shrink (1.5e-12 between mirror cells at 0.5 deg):
    // the weights are checked to 1e-10 (an asymmetric grid is off by the
    // partial cells' O(1e-3) and more) and each mirror pair takes their mean,
    // as close to the exact fraction as either.
    {
      double cmax = 0.0, tmax = 0.0, wbad = 0.0, cbad = 0.0, tbad = 0.0;
      for (int mc = 0; mc < nmc; ++mc)
        for (int k = 0; k < np; ++k) {
          cmax = std::max(cmax, std::fabs(CSt[(size_t)mc * S.ldk + k]));
          tmax = std::max(tmax, std::fabs(trig[(size_t)k * S.ldm + mc]));
        }
      for (int k = 0; k < np; ++k) {
        const int km = np - 1 - k;
        for (int j = 0; j < nt; ++j)
          wbad = std::max(wbad, std::fabs(g->w_host[(size_t)j * np + k] - g->w_host[(size_t)j * np + km]));
        for (int mc = 0; mc < nmc; ++mc) {
          const double sg = (mc > 0 && mc % 2 == 0) ? -1.0 : 1.0;  // sin columns are odd
          cbad = std::max(cbad, std::fabs(CSt[(size_t)mc * S.ldk + k] - sg * CSt[(size_t)mc * S.ldk + km]));
          tbad = std::max(tbad, std::fabs(trig[(size_t)k * S.ldm + mc] - sg * trig[(size_t)km * S.ldm + mc]));
        }
      }
      S.fold = np >= 2 && wbad <= 1e-10 && cbad <= 1e-12 * cmax && tbad <= 1e-12 * tmax;
    }
    S.h = (np + 1) / 2;
    S.ldkh = round_up(S.h, 16);
    S.ks = round_up(L + 1, 16);
    S.ldtf = S.ks + round_up(L, 16);
    if (S.fold) {
      const int h = S.h, mid = np % 2 ? h - 1 : -1;
      WF.assign((size_t)2 * nt * (L + 1) * S.ldkh, 0.0);
      TF.assign((size_t)h * S.ldtf, 0.0);
      for (int j = 0; j < nt; ++j)
        for (int k = 0; k < h; ++k) {
          // one weight per mirror pair (equal up to rounding); the middle
          // cell enters the even half twice
          const double wb = 0.5 * (g->w_host[(size_t)j * np + k] + g->w_host[(size_t)j * np + np - 1 - k]);
          const double f = (k == mid ? 0.5 : 1.0) * wb;
          for (int m = 0; m <= L; ++m) {
            WF[(((size_t)j * 2 + 0) * (L + 1) + m) * S.ldkh + k] = f * CSt[(size_t)(m ? 2 * m - 1 : 0) * S.ldk + k];
            if (m > 0)
              WF[(((size_t)j * 2 + 1) * (L + 1) + m - 1) * S.ldkh + k] = f * CSt[(size_t)(2 * m) * S.ldk + k];
          }
        }
      for (int k = 0; k < h; ++k)
        for (int m = 0; m <= L; ++m) {
          TF[(size_t)k * S.ldtf + m] = trig[(size_t)k * S.ldm + (m ? 2 * m - 1 : 0)];
          if (m > 0) TF[(size_t)k * S.ldtf + S.ks + m - 1] = trig[(size_t)k * S.ldm + 2 * m];
        }
      // the streaming analysis: the folded C / S rows without the weights
      // (cos outputs m = 0..L in tiles of 16, then sin outputs m = 1..L) and
      // the weights per colatitude, the middle cell's half in the weight
      nte = (L + 16) / 16;
      nto = (L + 15) / 16;
      ldcs = (int)round_up(h, 16);
      CSF.assign((size_t)16 * (nte + nto) * ldcs, 0.0);
      WTF.assign((size_t)nt * ldcs, 0.0);
      for (int k = 0; k < h; ++k) {
        for (int m = 0; m <= L; ++m) {
          CSF[(size_t)m * ldcs + k] = CSt[(size_t)(m ? 2 * m - 1 : 0) * S.ldk + k];
          if (m > 0) CSF[((size_t)16 * nte + m - 1) * ldcs + k] = CSt[(size_t)(2 * m) * S.ldk + k];
        }
        for (int j = 0; j < nt; ++j)
          WTF[(size_t)j * ldcs + k] =
              (k == mid ? 0.5 : 1.0) * 0.5 * (g->w_host[(size_t)j * np + k] + g->w_host[(size_t)j * np + np - 1 - k]);
      }
      // both halves in one basis for kGemmFoldAB: slot s < ks the cos half,
      // ks <= s < ks + L the sin half
      WFAB.assign((size_t)nt * (S.ks + L) * S.ldkh, 0.0);
      for (int j = 0; j < nt; ++j)
        for (int m = 0; m <= L; ++m)
          for (int k = 0; k < h; ++k) {
            const size_t base = (size_t)j * (S.ks + L);
            WFAB[(base + m) * S.ldkh + k] = WF[(((size_t)j * 2 + 0) * (L + 1) + m) * S.ldkh + k];
            if (m > 0) WFAB[(base + S.ks + m - 1) * S.ldkh + k] = WF[(((size_t)j * 2 + 1) * (L + 1) + m - 1) * S.ldkh + k];
          }
      // the synthesis basis slot-major for the LDS-free kernel: cos m at slot
      // m, sin m at kcs + m - 1, cells padded to a multiple of 32
      S.kcs = round_up(L + 1, 4);
      S.nks = S.kcs + round_up(L, 4);
      S.hp = round_up(h, 32);
      BK.assign((size_t)S.nks * S.hp, 0.0);
      for (int k = 0; k < h; ++k)
        for (int m = 0; m <= L; ++m) {
          BK[(size_t)m * S.hp + k] = TF[(size_t)k * S.ldtf + m];
          if (m > 0) BK[(size_t)(S.kcs + m - 1) * S.hp + k] = TF[(size_t)k * S.ldtf + S.ks + m - 1];
        }
      sep_quad_tables(g, CSt, trig, QA, QS, QW);
    }
    T.resize((size_t)nt * Q);
    yyg::theta_table_normalised(g->geom, L, T.data());
    P.resize((size_t)nt * Q);
    yyg::self_legendre_table(g->geom, L, P.data());
    // azimuthal-column-major copies for the theta GEMMs
    T2.assign((size_t)nmc * (L + 1) * nt, 0.0);
    P2.assign((size_t)nmc * nt * S.ldl, 0.0);
    for (int mc = 0; mc < nmc; ++mc) {
      const int m = (mc + 1) / 2;
      for (int l = m; l <= L; ++l)
        for (int j = 0; j < nt; ++j) {
          T2[((size_t)mc * (L + 1) + l) * nt + j] = T[(size_t)j * Q + l * l + mc];
          P2[((size_t)mc * nt + j) * S.ldl + l] = P[(size_t)j * Q + l * l + mc];
        }
    }
    // per degree: D_l (the rotation phase starts its accumulators from a
    // patch's own moments and adds the other patch's moments times D_l)
    D.resize(yyg::rotation_blocks_size(L));
    yyg::rotation_blocks(L, D.data());
    sep_theta_tables(g, T, P, D, TA, TS, DR);
  } catch (const std::bad_alloc &) {
    return YYG_ERR_OUT_OF_MEMORY;
  }
  int st = YYG_OK;
  if (st == YYG_OK) st = dmalloc(&S.Wcs, Wcs.size());
  if (st == YYG_OK) st = dmalloc(&S.trig, trig.size());
  if (st == YYG_OK) st = dmalloc(&S.T2, T2.size());
  if (st == YYG_OK) st = dmalloc(&S.P2, P2.size());
  if (st == YYG_OK) st = dmalloc(&S.Drot, D.size());
  if (st == YYG_OK) st = dmalloc(&S.X2, (size_t)nmc * MJ);
  if (st == YYG_OK) st = dmalloc(&S.V, (size_t)nmc * MJ);
  if (st == YYG_OK) st = dmalloc(&S.Ut, (size_t)nmc * (L + 1) * M);
  if (st == YYG_OK && g->n_patch == 2) st = dmalloc(&S.At, (size_t)M * Q);
  if (st == YYG_OK) st = dmalloc(&S.coefS, coefS.size());
  if (st == YYG_OK && S.fold) st = dmalloc(&S.WF, WF.size());
  if (st == YYG_OK && S.fold) st = dmalloc(&S.TF, TF.size());
  if (st == YYG_OK && !TA.empty()) st = dmalloc(&S.TA, TA.size());
  if (st == YYG_OK && !TS.empty()) st = dmalloc(&S.TS, TS.size());
  if (st == YYG_OK && !DR.empty()) st = dmalloc(&S.DR, DR.size());
  if (st == YYG_OK && S.fold) st = dmalloc(&S.QA, QA.size());
  if (st == YYG_OK && S.fold) st = dmalloc(&S.QS, QS.size());
  if (st == YYG_OK && !QW.empty()) st = dmalloc(&S.QW, QW.size());
  if (st == YYG_OK && S.fold) st = dmalloc(&S.BK, BK.size());
  if (st == YYG_OK && S.fold) st = dmalloc(&S.WFAB, WFAB.size());
  if (st == YYG_OK && S.fold) st = dmalloc(&S.CSF, CSF.size());
  if (st == YYG_OK && S.fold) st = dmalloc(&S.Wt, WTF.size());
  if (st != YYG_OK) {
    sep_release(g);
    return st;
  }
  hipError_t e = hipSuccess;
  auto chk = [&](hipError_t r) {
    if (e == hipSuccess && r != hipSuccess) e = r;
  };
  chk(hipMemcpy(S.Wcs, Wcs.data(), Wcs.size() * sizeof(double), hipMemcpyHostToDevice));
  chk(hipMemcpy(S.trig, trig.data(), trig.size() * sizeof(double), hipMemcpyHostToDevice));
  if (S.TA) chk(hipMemcpy(S.TA, TA.data(), TA.size() * sizeof(double), hipMemcpyHostToDevice));
  if (S.TS) chk(hipMemcpy(S.TS, TS.data(), TS.size() * sizeof(double), hipMemcpyHostToDevice));
  if (S.DR) chk(hipMemcpy(S.DR, DR.data(), DR.size() * sizeof(double), hipMemcpyHostToDevice));
  chk(hipMemcpy(S.T2, T2.data(), T2.size() * sizeof(double), hipMemcpyHostToDevice));
  chk(hipMemcpy(S.P2, P2.data(), P2.size() * sizeof(double), hipMemcpyHostToDevice));
  chk(hipMemcpy(S.Drot, D.data(), D.size() * sizeof(double), hipMemcpyHostToDevice));
  chk(hipMemcpy(S.coefS, coefS.data(), coefS.size() * sizeof(double), hipMemcpyHostToDevice));
  if (S.fold) {
    chk(hipMemcpy(S.WF, WF.data(), WF.size() * sizeof(double), hipMemcpyHostToDevice));
    chk(hipMemcpy(S.TF, TF.data(), TF.size() * sizeof(double), hipMemcpyHostToDevice));
    chk(hipMemcpy(S.QA, QA.data(), QA.size() * sizeof(double), hipMemcpyHostToDevice));
    chk(hipMemcpy(S.QS, QS.data(), QS.size() * sizeof(double), hipMemcpyHostToDevice));
    if (S.QW) chk(hipMemcpy(S.QW, QW.data(), QW.size() * sizeof(double), hipMemcpyHostToDevice));
    chk(hipMemcpy(S.BK, BK.data(), BK.size() * sizeof(double), hipMemcpyHostToDevice));
    chk(hipMemcpy(S.WFAB, WFAB.data(), WFAB.size() * sizeof(double), hipMemcpyHostToDevice));
    chk(hipMemcpy(S.CSF, CSF.data(), CSF.size() * sizeof(double), hipMemcpyHostToDevice));
    chk(hipMemcpy(S.Wt, WTF.data(), WTF.size() * sizeof(double), hipMemcpyHostToDevice));
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    sep_release(g);
    return YYG_ERR_DEVICE;
  }
  auto kround = [](long k) { return (int)((k + 15) / 16 * 16); };
  // per colatitude j: X2[mc][j][row] = sum_k rho[row][j][k] w_jk CS_k^(mc)   (rho set per solve)
  S.phi_ana = yyg::GemmF64Args{(int)M, nmc, np, nullptr, (long)nt * np, S.Wcs, S.ldk, S.X2, MJ, M, kround(np), 1};
  S.phi_ana.batch = nt;
  S.phi_ana.a_batch = np;
  S.phi_ana.b_batch = (long)nmc * S.ldk;
  // per colatitude j: phi[row][j][k] = sum_mc V[mc][j][row] trig[k][mc]        (phi set per solve)
  S.phi_syn = yyg::GemmF64Args{(int)M, np, nmc, S.V, MJ, S.trig, S.ldm, nullptr, (long)nt * np, np, kround(nmc), 1};
  S.phi_syn.batch = nt;
  S.phi_syn.a_batch = M;
  // folded: even (cos) and odd (sin) halves of every row, h = ceil(n_p / 2)
  S.phi_ana_f = yyg::GemmF64Args{(int)M, L + 1, (int)S.h, nullptr, (long)nt * np, S.WF, S.ldkh, S.X2, MJ, M, kround(S.h), 1};
  S.phi_ana_f.batch = 2 * nt;
  S.phi_ana_f.a_batch = np;
  S.phi_ana_f.b_batch = (long)(L + 1) * S.ldkh;
  S.phi_ana_f.fold_k = np;
  S.phi_ana_f.fold_mc = nmc;
  // both halves per block: slots ks + L, the same density rows and output
  S.phi_ana_ab = yyg::GemmF64Args{(int)M, (int)(S.ks + L), (int)S.h, nullptr, (long)nt * np, S.WFAB, S.ldkh, S.X2, MJ,
                                  M, kround(S.h), 1};
  S.phi_ana_ab.batch = nt;
  S.phi_ana_ab.a_batch = np;
  S.phi_ana_ab.b_batch = (long)(S.ks + L) * S.ldkh;
  S.phi_ana_ab.k_split = (int)S.ks;
  S.phi_ana_ab.fold_k = np;
  S.phi_ana_ab.fold_mc = nmc;
  S.phi_syn_f = yyg::GemmF64Args{(int)M, (int)S.h, (int)S.ldtf, S.V, MJ, S.TF, S.ldtf, nullptr, (long)nt * np, np,
                                 kround(S.ldtf), 1};
  S.phi_syn_f.batch = nt;
  S.phi_syn_f.a_batch = M;
  S.phi_syn_f.k_split = (int)S.ks;
  S.phi_syn_f.fold_k = np;
  S.phi_syn_f.fold_mc = nmc;
  S.phi_syn_s = yyg::PhiStreamArgs{S.V, S.TF, nullptr, MJ, (long)nt * np, (int)M, nt, np, (int)S.h, L, nmc,
                                   (int)S.ldtf, (int)S.ks};
  S.phi_ana_s = yyg::PhiAnaStreamArgs{nullptr, S.CSF, S.Wt, S.X2, MJ, (long)nt * np, (int)M, nt, np, (int)S.h, L,
                                      nmc, ldcs, nte, nto};
  S.phi_ana_d = yyg::PhiDirectArgs{nullptr, S.Wcs, S.X2, (int)M, nt, nmc, np, S.ldk, (long)nmc * S.ldk};
  S.phi_syn_d = yyg::PhiDirectArgs{S.V, S.trig, nullptr, (int)M, nt, np, nmc, S.ldm, 0};
  if (S.fold) {
    for (yyg::PhiQuadArgs *q : {&S.quad_ana, &S.quad_syn}) {
      q->MJ = MJ;
      q->ld = (long)nt * np;
      q->Mr = (int)M;
      q->nt = nt;
      q->np = np;
      q->L = L;
    }
    S.quad_ana.bas = S.QA;
    S.quad_ana.W = S.QW;
    S.quad_ana.C = S.X2;
    S.quad_syn.bas = S.QS;
    S.quad_syn.X = S.V;
    sep_default_phi(g);
  }
  S.phi_syn_l = yyg::PhiLeanArgs{S.V, S.BK, nullptr, (int)M, nt, np, (int)S.h, (int)S.hp, (int)S.nks, (int)S.kcs, nmc};
  // theta analysis, rotation (Yin-Yang) and theta synthesis: problem
  // operands derived in the kernels from these
  S.args = yyg::SepPhaseArgs{L,    g->n_r, g->n_patch, nt,  S.ldl, S.X2, S.T2, S.P2,
                             S.Ut, S.Drot,   g->d_Ahat,  S.At, S.V};
  S.theta = yyg::ThetaArgs{S.X2,     S.TA, S.TS, S.Ut, S.DR, g->d_Ahat, S.At, S.V,
                           MJ,       (long)yyg::theta_ana_doubles(L, (nt + 1) / 2),
                           (long)yyg::theta_syn_doubles(L, (nt + 1) / 2), (long)yyg::rotation_doubles(L), L, g->n_r, (int)M, nt, (nt + 1) / 2};
  // the theta synthesis' waves each run a column's colatitudes in turn: where
  // they are few and the colatitudes many, 32 x 32 tiles (a solve, us: 25
  // columns of 7 row tiles, 90 colatitudes 29.6 and 30.6; 33 of 7, 47
  // colatitudes 29.8 and 30.9; 81 of 7 43.2 and 43.9; 51 of 13 35.7 and 36.5; 21 of
  // 13, 32 colatitudes 25.5 and 26.4; 51 of 25, 47 colatitudes 44.6 and 44.4;
  // 17 of 4, 20 colatitudes 23.9 and 24.2)
  const bool few = (long)nmc * ((M + 15) / 16) < 3L * g->cus && nt > 24;
  for (int r = 1; r <= 3; ++r)
    if (S.stream[r]) S.var[r] = r == 3 && few ? 10 : yyg::gemm_f64_variant_count() + 4;
  S.ready = true;
  return YYG_OK;
}

// Separable solve: phi analysis (a strided batch over the colatitudes),
// theta analysis (one problem per azimuthal column) into the column-major
// moments, own plus rotated other moments (Yin-Yang; one problem per degree
// and patch), radial scan into the azimuthal-column-major coefficients,
// theta synthesis (one problem per azimuthal column), phi synthesis (a
// strided batch over the colatitudes).
// A phi phase (0 or 4) in `precision`: the FP64 variant of the plan, or the
// plan's reduced-precision tile for FP32 / BF16 x 3.
// The opt-in input check: YYG_ERR_NONFINITE if rho holds a NaN or an
// infinity, YYG_OK if not or if the check is off.  Waits for the check on
// stream s; allocates nothing (the flag is the plan's).
int check_rho(yyg_grid *g, const double *rho, hipStream_t s) {
  if (!g->check_finite) return YYG_OK;
  const long n = (long)g->n_patch * g->n_r * g->nang;
  int h = 0;
  hipError_t e = yyg::launch_check_finite(rho, n, g->d_flag, s);
  if (e == hipSuccess) e = hipMemcpyAsync(&h, g->d_flag, sizeof(int), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return YYG_ERR_DEVICE;
  }
  return h ? YYG_ERR_NONFINITE : YYG_OK;
}

// Choices of a reduced-precision phi transform (side 0 analysis, 1
// synthesis): the tile shapes, and in FP32 on a folded grid also the FP32
// streaming kernels after them.
int sep_lp_choices(const yyg_grid *g, int precision, int side) {
  if (precision != YYG_FP32 || !g->sep.fold) return yyg::sep_lp_tile_count();
  return yyg::sep_lp_tile_count() +
         (side == 1 ? yyg::phi_stream32_variant_count() : yyg::phi_ana_stream32_variant_count());
}

bool sep_lp_available(const yyg_grid *g, int precision, int side, int t) {
  if (t < 0 || t >= sep_lp_choices(g, precision, side)) return false;
  const int u = t - yyg::sep_lp_tile_count();
  if (u < 0) return true;
  return side == 1 ? yyg::phi_stream32_supports(u, g->L) : yyg::phi_ana_stream32_supports(u, (int)g->sep.h, g->n_p);
}

hipError_t sep_launch_phi(yyg_grid *g, int r, int precision, hipStream_t s) {
  auto &S = g->sep;
  if (precision == YYG_FP64) return sep_launch_phase(g, r, s);
  if (r == 4 && precision == YYG_FP32 && S.lpt[0][1] >= yyg::sep_lp_tile_count())
    return yyg::launch_phi_syn_stream32(S.lpt[0][1] - yyg::sep_lp_tile_count(), S.phi_syn_s, g->cus, s);
  if (r == 0 && precision == YYG_FP32 && S.lpt[0][0] >= yyg::sep_lp_tile_count())
    return yyg::launch_phi_ana_stream32(S.lpt[0][0] - yyg::sep_lp_tile_count(), S.phi_ana_s, g->cus, s);
  const yyg::GemmF64Args &phi = r == 0 ? (S.fold ? S.phi_ana_f : S.phi_ana) : (S.fold ? S.phi_syn_f : S.phi_syn);
  return yyg::launch_sep_lp_phase(precision, S.lpt[precision - 1][r == 0 ? 0 : 1], r, S.fold, phi, s);
}

hipError_t sep_solve(yyg_grid *g, hipStream_t s, int precision = YYG_FP64) {
  auto &S = g->sep;
  hipError_t e = hipSuccess;
  g->ahat_cols = true;
  g->ahat_fold = false;
  int t = timing_begin(g, 4, s);
  e = sep_launch_phi(g, 0, precision, s);
  timing_end(g, t, s);
  // the scan's input: the moments, or with two patches their rotated sum
  const double *scan_in = g->n_patch == 2 ? S.At : g->d_Ahat;
  if (e == hipSuccess) {
    t = timing_begin(g, 5, s);
    e = sep_launch_phase(g, 1, s);
    if (e == hipSuccess) e = sep_launch_phase(g, 2, s);
    timing_end(g, t, s);
  }
  if (e == hipSuccess) {
    t = timing_begin(g, 1, s);
    e = yyg::launch_radial_scan_q(scan_in, S.coefS, g->d_qdeg, g->n_r, g->L, -g->G, g->n_patch, S.Ut, s);
    timing_end(g, t, s);
  }
  if (e == hipSuccess) {
    t = timing_begin(g, 6, s);
    e = sep_launch_phase(g, 3, s);
    timing_end(g, t, s);
  }
  if (e == hipSuccess) {
    t = timing_begin(g, 7, s);
    e = sep_launch_phi(g, 4, precision, s);
    timing_end(g, t, s);
  }
  return e;
}

}  // namespace


struct yyg_batch {
  int device = 0;
  int precision = 0;
  std::vector<yyg_grid *> grids;
  std::vector<const double *> rho;
  std::vector<double *> phi;
  // per-field argument arrays: pinned host copies (pointer-patched per
  // solve) and their device mirrors, refreshed by a copy at the head of
  // the recorded graph
  yyg::GemmF64Args *h_f64[2] = {nullptr, nullptr}, *d_f64[2] = {nullptr, nullptr};
  yyg::GemmLpArgs *h_lp[2] = {nullptr, nullptr}, *d_lp[2] = {nullptr, nullptr};
  yyg::ScanArgs *d_scan = nullptr;
  yyg::SplitArgs *h_split[2] = {nullptr, nullptr}, *d_split[2] = {nullptr, nullptr};
  int4 *d_items[2] = {nullptr, nullptr};  // analysis / synthesis work items
  int n_items[2] = {0, 0};
  int var[2] = {0, 0};                    // tile variants
  int blocks[2] = {0, 0};                 // resident persistent blocks
  int4 *d_scan_items = nullptr;
  int n_scan_items = 0;
  int2 *d_split_items[2] = {nullptr, nullptr};
  int n_split_items[2] = {0, 0};
  int cus = 256;
  hipGraphExec_t exec = nullptr;
  hipStream_t exec_stream = nullptr;
  hipEvent_t done = nullptr;
  hipStream_t stream = nullptr;  // used when the caller passes the default stream
  bool launched = false;
  std::vector<int> part_gen;     // plans' partial-buffer generations the arguments hold
  // separable batches (FP64, every plan in the separable form): the five
  // phases and the column scans as grouped launches over all plans
  bool sep = false, sep_fold = false;
  // one pinned array and its device mirror hold the phi phases' arguments of
  // the tiles and of the sweeps (analysis / synthesis)
  char *h_args = nullptr, *d_args = nullptr;
  size_t args_bytes = 0;
  yyg::GemmF64Args *h_phi[2] = {nullptr, nullptr}, *d_phi[2] = {nullptr, nullptr};
  yyg::PhiQuadArgs *h_quad[2] = {nullptr, nullptr}, *d_quad[2] = {nullptr, nullptr};
  yyg::ThetaArgs *d_theta = nullptr;
  yyg::SepPhaseArgs *d_sargs = nullptr;
  yyg::ScanQArgs *d_qscan = nullptr;
  int2 *d_qitems = nullptr;
  int n_qitems = 0, max_nr = 0;
  bool scan_two = false;
  int4 *d_sitems[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
  int n_sitems[5] = {0, 0, 0, 0, 0};
  int svar[5] = {0, 0, 0, 0, 0};    // tile of each phase (yyg::sep_batch_tile)
  int sblocks[5] = {0, 0, 0, 0, 0};
  int smax[5] = {0, 0, 0, 0, 0};    // sweeps: the largest shape or degree
  size_t slds[5] = {0, 0, 0, 0, 0};
};

namespace {

void batch_drop_graph(yyg_batch *b) {
  if (b->exec) (void)hipGraphExecDestroy(b->exec);
  b->exec = nullptr;
  b->exec_stream = nullptr;
}

void batch_free(yyg_batch *b) {
  if (!b) return;
  batch_drop_graph(b);
  for (int r = 0; r < 2; ++r) {
    if (b->h_f64[r]) (void)hipHostFree(b->h_f64[r]);
    if (b->h_lp[r]) (void)hipHostFree(b->h_lp[r]);
    if (b->h_split[r]) (void)hipHostFree(b->h_split[r]);
    void *d[] = {b->d_f64[r], b->d_lp[r], b->d_split[r], b->d_items[r], b->d_split_items[r]};
    for (void *x : d)
      if (x) (void)dev_free(x);
  }
  if (b->d_scan) (void)dev_free(b->d_scan);
  if (b->d_scan_items) (void)dev_free(b->d_scan_items);
  if (b->h_args) (void)hipHostFree(b->h_args);
  if (b->d_args) (void)dev_free(b->d_args);
  if (b->d_theta) (void)dev_free(b->d_theta);
  for (int r = 0; r < 5; ++r)
    if (b->d_sitems[r]) (void)dev_free(b->d_sitems[r]);
  if (b->d_sargs) (void)dev_free(b->d_sargs);
  if (b->d_qscan) (void)dev_free(b->d_qscan);
  if (b->d_qitems) (void)dev_free(b->d_qitems);
  if (b->done) (void)hipEventDestroy(b->done);
  if (b->stream) (void)hipStreamDestroy(b->stream);
  delete b;
}

template <class T>
int upload(T **dst, const std::vector<T> &src) {
  if (*dst) (void)dev_free(*dst);
  *dst = nullptr;
  if (src.empty()) return YYG_OK;
  if (dev_malloc(reinterpret_cast<void **>(dst), src.size() * sizeof(T)) != hipSuccess) {
    *dst = nullptr;
    (void)hipGetLastError();
    return YYG_ERR_OUT_OF_MEMORY;
  }
  if (hipMemcpy(*dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice) != hipSuccess) {
    (void)hipGetLastError();
    return YYG_ERR_DEVICE;
  }
  return YYG_OK;
}

// Work items of one contraction phase for tile variant v, largest K first
// so the persistent blocks finish together.
int batch_set_items(yyg_batch *b, int role, int v) {
  const bool lp = b->precision != YYG_FP64;
  int bm, bn;
  if (lp)
    yyg::gemm_lp_variant_tile(v, &bm, &bn);
  else
    yyg::gemm_f64_variant_tile(v, &bm, &bn);
  std::vector<std::pair<long, int4>> work;
  const int n = (int)b->grids.size();
  for (int f = 0; f < n; ++f) {
    const yyg_grid *g = b->grids[f];
    const long M = (long)g->n_patch * g->n_r, N = role == 0 ? g->Q : g->nang, K = role == 0 ? g->nang : (long)g->n_patch * g->Q;
    const int tm = (int)((M + bm - 1) / bm), tn = (int)((N + bn - 1) / bn);
    if (lp) {
      b->h_lp[role][f].tiles_m = tm;
    } else {
      b->h_f64[role][f].tiles_m = tm;
    }
    for (int j = 0; j < tn; ++j)
      for (int i = 0; i < tm; ++i) work.push_back({K, int4{f, i, j, 0}});
  }
  std::stable_sort(work.begin(), work.end(), [](const auto &x, const auto &y) { return x.first > y.first; });
  std::vector<int4> items(work.size());
  for (size_t i = 0; i < work.size(); ++i) items[i] = work[i].second;
  int st = upload(&b->d_items[role], items);
  if (st != YYG_OK) return st;
  b->n_items[role] = (int)items.size();
  b->var[role] = v;
  // resident blocks: LDS-limited occupancy of the variant, four at most
  const int eb = lp ? yyg::lp_elem_bytes(b->precision) : 8;
  const int parts = lp ? yyg::lp_parts(b->precision) : 1;
  const int bk = lp ? yyg::lp_stage_k(b->precision) : 16;
  const long lds = 2L * parts * (bm + bn) * (bk + 16 / eb) * eb;
  int per_cu = (int)std::max(1L, std::min(4L, 160L * 1024 / std::max(1L, lds)));
  b->blocks[role] = std::max(1, std::min(b->n_items[role], b->cus * per_cu));
  // the per-problem tiles_m lives in the argument arrays
  if (lp) {
    std::vector<yyg::GemmLpArgs> h(b->h_lp[role], b->h_lp[role] + n);
    if (hipMemcpy(b->d_lp[role], h.data(), n * sizeof(yyg::GemmLpArgs), hipMemcpyHostToDevice) != hipSuccess)
      return YYG_ERR_DEVICE;
  } else {
    std::vector<yyg::GemmF64Args> h(b->h_f64[role], b->h_f64[role] + n);
    if (hipMemcpy(b->d_f64[role], h.data(), n * sizeof(yyg::GemmF64Args), hipMemcpyHostToDevice) != hipSuccess)
      return YYG_ERR_DEVICE;
  }
  return YYG_OK;
}

hipError_t batch_launch_gemm(yyg_batch *b, int role, hipStream_t s) {
  if (b->precision == YYG_FP64)
    return yyg::launch_gemm_f64_grouped(b->var[role], role, b->d_f64[role], b->d_items[role], b->n_items[role],
                                        b->blocks[role], s);
  return yyg::launch_gemm_lp_grouped(b->precision, b->var[role], role, b->d_lp[role], b->d_items[role],
                                     b->n_items[role], b->blocks[role], s);
}

// Write the current density / potential pointers into the pinned argument
// arrays (their device mirrors are refreshed by the graph's first nodes).
void batch_patch_pointers(yyg_batch *b) {
  const int n = (int)b->grids.size();
  for (int f = 0; f < n; ++f) {
    if (b->sep) {
      b->h_phi[0][f].A = b->rho[f];
      b->h_phi[1][f].C = b->phi[f];
      b->h_quad[0][f].X = b->rho[f];
      b->h_quad[1][f].C = b->phi[f];
    } else if (b->precision == YYG_FP64) {
      b->h_f64[0][f].A = b->rho[f];
      b->h_f64[1][f].C = b->phi[f];
    } else {
      b->h_split[0][f].X = b->rho[f];
      b->h_lp[1][f].C = b->phi[f];
    }
  }
}

hipError_t sep_batch_enqueue(yyg_batch *b, hipStream_t s, hipEvent_t *ev);

// Enqueue the whole batched solve on s (recorded into the graph).
hipError_t batch_enqueue(yyg_batch *b, hipStream_t s) {
  if (b->sep) return sep_batch_enqueue(b, s, nullptr);
  const int n = (int)b->grids.size();
  hipError_t e = hipSuccess;
  const bool lp = b->precision != YYG_FP64;
  if (!lp) {
    e = hipMemcpyAsync(b->d_f64[0], b->h_f64[0], n * sizeof(yyg::GemmF64Args), hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
      e = hipMemcpyAsync(b->d_f64[1], b->h_f64[1], n * sizeof(yyg::GemmF64Args), hipMemcpyHostToDevice, s);
  } else {
    e = hipMemcpyAsync(b->d_split[0], b->h_split[0], n * sizeof(yyg::SplitArgs), hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
      e = hipMemcpyAsync(b->d_lp[1], b->h_lp[1], n * sizeof(yyg::GemmLpArgs), hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
      e = yyg::launch_split_rows_grouped(b->precision, b->d_split[0], b->d_split_items[0], b->n_split_items[0],
                                         std::min(b->n_split_items[0], b->cus * 8), s);
  }
  if (e == hipSuccess) e = batch_launch_gemm(b, 0, s);
  if (e == hipSuccess)
    e = yyg::launch_radial_scan_grouped(b->d_scan, b->d_scan_items, b->n_scan_items,
                                        std::min(b->n_scan_items, b->cus * 2), s);
  if (e == hipSuccess && lp)
    e = yyg::launch_split_rows_grouped(b->precision, b->d_split[1], b->d_split_items[1], b->n_split_items[1],
                                       std::min(b->n_split_items[1], b->cus * 8), s);
  if (e == hipSuccess) e = batch_launch_gemm(b, 1, s);
  return e;
}

int batch_build(yyg_batch *b) {
  const int n = (int)b->grids.size();
  const bool lp = b->precision != YYG_FP64;
  const bool scaled = b->precision == YYG_FP16X2;
  b->rho.assign(n, nullptr);
  b->phi.assign(n, nullptr);
  b->part_gen.resize(n);
  for (int f = 0; f < n; ++f) b->part_gen[f] = b->grids[f]->part_gen;
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, b->device) == hipSuccess && cus > 0)
    b->cus = cus;
  if (hipEventCreateWithFlags(&b->done, hipEventDisableTiming) != hipSuccess) return YYG_ERR_DEVICE;
  if (hipStreamCreate(&b->stream) != hipSuccess) return YYG_ERR_DEVICE;
  for (int r = 0; r < 2; ++r) {
    if (lp) {
      if (hipHostMalloc(reinterpret_cast<void **>(&b->h_lp[r]), n * sizeof(yyg::GemmLpArgs), 0) != hipSuccess ||
          hipHostMalloc(reinterpret_cast<void **>(&b->h_split[r]), n * sizeof(yyg::SplitArgs), 0) != hipSuccess ||
          dev_malloc(reinterpret_cast<void **>(&b->d_lp[r]), n * sizeof(yyg::GemmLpArgs)) != hipSuccess ||
          dev_malloc(reinterpret_cast<void **>(&b->d_split[r]), n * sizeof(yyg::SplitArgs)) != hipSuccess) {
        (void)hipGetLastError();
        return YYG_ERR_OUT_OF_MEMORY;
      }
    } else {
      if (hipHostMalloc(reinterpret_cast<void **>(&b->h_f64[r]), n * sizeof(yyg::GemmF64Args), 0) != hipSuccess ||
          dev_malloc(reinterpret_cast<void **>(&b->d_f64[r]), n * sizeof(yyg::GemmF64Args)) != hipSuccess) {
        (void)hipGetLastError();
        return YYG_ERR_OUT_OF_MEMORY;
      }
    }
  }
  std::vector<yyg::ScanArgs> scan(n);
  std::vector<int4> scan_items;
  std::vector<int2> split_items[2];
  for (int f = 0; f < n; ++f) {
    yyg_grid *g = b->grids[f];
    const int Q = g->Q;
    const long M = (long)g->n_patch * g->n_r;
    if (!lp) {
      yyg::GemmF64Args &a = b->h_f64[0][f];
      a = yyg::GemmF64Args{(int)M, Q, (int)g->nang, nullptr, g->nang, g->d_Bt, g->ldb, g->d_part, Q, 0,
                           (int)(((g->nang + 15) / 16) * 16), 1};
      yyg::GemmF64Args &c = b->h_f64[1][f];
      c = yyg::GemmF64Args{(int)M, (int)g->nang, g->n_patch * Q, g->d_U, g->ldy, g->d_Y, g->ldy, nullptr, g->nang, 0,
                           (int)(((g->n_patch * Q + 15) / 16) * 16), 1};
    } else {
      auto &L = g->lp[b->precision - 1];
      const int bk = yyg::lp_stage_k(b->precision);
      b->h_split[0][f] = yyg::SplitArgs{nullptr, g->nang, (int)g->nang, scaled ? g->d_eA : nullptr, L.Ar, L.lda,
                                        M * L.lda};
      b->h_split[1][f] = yyg::SplitArgs{g->d_U, g->ldy, g->n_patch * Q, scaled ? g->d_eU : nullptr, L.Ur, L.ldu, M * L.ldu};
      b->h_lp[0][f] = yyg::GemmLpArgs{(int)M, Q, (int)g->nang, L.Ar, L.lda, M * L.lda, scaled ? g->d_eA : nullptr,
                                      L.Bt, L.ldb, (long)Q * L.ldb, L.eBt, g->d_part, Q, 0,
                                      (int)((g->nang + bk - 1) / bk * bk), 1};
      b->h_lp[1][f] = yyg::GemmLpArgs{(int)M, (int)g->nang, g->n_patch * Q, L.Ur, L.ldu, M * L.ldu,
                                      scaled ? g->d_eU : nullptr, L.Y, L.ldy, (long)g->nang * L.ldy, L.eY, nullptr,
                                      g->nang, 0, (int)((g->n_patch * Q + bk - 1) / bk * bk), 1};
      for (long r = 0; r < M; ++r) {
        split_items[0].push_back(int2{f, (int)r});
        split_items[1].push_back(int2{f, (int)r});
      }
    }
    scan[f] = yyg::ScanArgs{g->d_part, 1, M * Q, g->d_Ahat, g->d_coef, g->d_qdeg, g->n_r, Q, g->L, -g->G, g->d_U,
                            g->ldy, g->n_patch == 2 ? 1 : 0};
    for (int p = 0; p < g->n_patch; ++p)
      for (int cb = 0; cb < (Q + 15) / 16; ++cb) scan_items.push_back(int4{f, cb, p, 0});
  }
  int st = upload(&b->d_scan, scan);
  if (st == YYG_OK) st = upload(&b->d_scan_items, scan_items);
  b->n_scan_items = (int)scan_items.size();
  if (lp) {
    for (int r = 0; r < 2 && st == YYG_OK; ++r) {
      st = upload(&b->d_split_items[r], split_items[r]);
      b->n_split_items[r] = (int)split_items[r].size();
      if (st == YYG_OK &&
          hipMemcpy(b->d_split[r], b->h_split[r], n * sizeof(yyg::SplitArgs), hipMemcpyHostToDevice) != hipSuccess)
        st = YYG_ERR_DEVICE;
    }
  }
  // default tile variant 64 x 64 (index 3 of the FP64 list, 0 of the others)
  for (int role = 0; role < 2 && st == YYG_OK; ++role) st = batch_set_items(b, role, lp ? 0 : 3);
  return st;
}

// Work items of separable phase r over every plan for batch tile t, the
// longest contractions first so that the persistent blocks finish together:
// (plan, tile row, tile column, z), z the strided-batch index (phi phases)
// or the problem of the phase (theta phases, rotation).
// The number past the tiles: the sweeps of yyg_phi_quad.hip and
// yyg_theta.hip, where every plan can run them.
bool sep_batch_sweeps(const yyg_batch *b, int r) {
  for (int f = 0; f < (int)b->grids.size(); ++f) {
    const yyg_grid *g = b->grids[f];
    if (r == 0 || r == 4) {
      if (!b->sep_fold || !yyg::phi_group_fits(r == 0, b->h_quad[r == 0 ? 0 : 1][f])) return false;
    } else if ((r != 2 || g->n_patch == 2) && !g->sep.stream[r]) {
      return false;
    }
  }
  return true;
}

bool sep_batch_available(const yyg_batch *b, int r, int t) {
  return t < yyg::sep_batch_tile_count() || (t == yyg::sep_batch_tile_count() && sep_batch_sweeps(b, r));
}

// Work items of the sweeps, one a block, the longest first; a plan's phi
// blocks in runs per XCD (blocks go to the XCDs round-robin).  Theta blocks
// take 16 row tiles (their basis is staged once for them), rotation blocks
// 16 of a patch's.
int sep_batch_sweep_items(yyg_batch *b, int r) {
  std::vector<std::pair<long, int4>> work;
  const int n = (int)b->grids.size();
  b->smax[r] = 0;
  b->slds[r] = 0;
  for (int f = 0; f < n; ++f) {
    const yyg_grid *g = b->grids[f];
    const yyg::ThetaArgs &a = g->sep.theta;
    if (r == 0 || r == 4) {
      const yyg::PhiQuadArgs &q = b->h_quad[r == 0 ? 0 : 1][f];
      const int blocks = yyg::phi_group_blocks(r == 0, q), shape = yyg::phi_group_shape(r == 0, q);
      b->smax[r] = std::max(b->smax[r], shape);
      const int per = blocks / 8, rem = blocks % 8;
      for (int i = 0; i < blocks; ++i)
        work.push_back({(long)q.S * shape, int4{f, (i & 7) * per + std::min(i & 7, rem) + (i >> 3), shape, 0}});
      continue;
    }
    b->smax[r] = std::max(b->smax[r], g->L);
    if (r == 2) {
      if (g->n_patch != 2) continue;
      b->slds[r] = std::max(b->slds[r], 2 * yyg::rotation_doubles(g->L) * sizeof(double));
      const int tiles = (a.nR + 15) / 16, runs = (tiles + 15) / 16;
      for (int l = 0; l <= g->L; ++l)
        for (int u = 0; u < 3; ++u)
          for (int i = 0; i < runs; ++i)
            work.push_back({(long)(u == 0 ? 2 : 1) * l * (tiles / runs), int4{f, 3 * l + u, i, runs}});
    } else {
      const size_t lds = (r == 1 ? yyg::theta_ana_doubles(g->L, a.h) : yyg::theta_syn_doubles(g->L, a.h)) * sizeof(double);
      b->slds[r] = std::max(b->slds[r], lds);
      const int tiles = (a.Mr + 15) / 16, chunks = (tiles + 15) / 16;
      for (int mc = 0; mc < 2 * g->L + 1; ++mc)
        for (int i = 0; i < chunks; ++i)
          work.push_back({(long)a.h * (g->L + 2 - (mc + 1) / 2) * (tiles / chunks), int4{f, mc, i, chunks}});
    }
  }
  std::stable_sort(work.begin(), work.end(), [](const auto &x, const auto &y) { return x.first > y.first; });
  std::vector<int4> items(work.size());
  for (size_t i = 0; i < work.size(); ++i) items[i] = work[i].second;
  const int st = upload(&b->d_sitems[r], items);
  if (st != YYG_OK) return st;
  b->n_sitems[r] = (int)items.size();
  b->svar[r] = yyg::sep_batch_tile_count();
  return YYG_OK;
}

int sep_batch_set_items(yyg_batch *b, int r, int t) {
  if (t == yyg::sep_batch_tile_count()) return sep_batch_sweep_items(b, r);
  int bm, bn, threads;
  yyg::sep_batch_tile(t, &bm, &bn, &threads);
  std::vector<std::pair<long, int4>> work;
  const int n = (int)b->grids.size();
  auto tiles = [&](long M, long N, long K, int f, int z) {
    const int tm = (int)((M + bm - 1) / bm), tn = (int)((N + bn - 1) / bn);
    for (int j = 0; j < tn; ++j)
      for (int i = 0; i < tm; ++i) work.push_back({K, int4{f, i, j, z}});
  };
  for (int f = 0; f < n; ++f) {
    const yyg_grid *g = b->grids[f];
    const long Mr = (long)g->n_patch * g->n_r;
    const int L = g->L, nmc = 2 * L + 1;
    if (r == 0 || r == 4) {
      const yyg::GemmF64Args &a = b->h_phi[r == 0 ? 0 : 1][f];
      for (int z = 0; z < a.batch; ++z) tiles(a.M, a.N, a.K, f, z);
    } else if (r == 1) {
      for (int z = 0; z < nmc; ++z) tiles(Mr, L + 1 - (z + 1) / 2, g->n_t, f, z);
    } else if (r == 2) {
      if (g->n_patch == 2)
        for (int z = 0; z < 2 * (L + 1); ++z) tiles(g->n_r, 2 * (L - z / 2) + 1, 2 * (L - z / 2) + 1, f, z);
    } else {
      for (int z = 0; z < nmc; ++z) tiles(g->n_t, Mr, L + 1 - (z + 1) / 2, f, z);
    }
  }
  std::stable_sort(work.begin(), work.end(), [](const auto &x, const auto &y) { return x.first > y.first; });
  std::vector<int4> items(work.size());
  for (size_t i = 0; i < work.size(); ++i) items[i] = work[i].second;
  int st = upload(&b->d_sitems[r], items);
  if (st != YYG_OK) return st;
  b->n_sitems[r] = (int)items.size();
  b->svar[r] = t;
  // resident blocks: LDS-limited occupancy of the tile, four at most
  const long lds = 2L * (bm + bn) * 18 * 8;
  const int per_cu = (int)std::max(1L, std::min(4L, 160L * 1024 / lds));
  b->sblocks[r] = std::max(1, std::min(b->n_sitems[r], b->cus * per_cu));
  return YYG_OK;
}

int sep_batch_build(yyg_batch *b) {
  const int n = (int)b->grids.size();
  b->rho.assign(n, nullptr);
  b->phi.assign(n, nullptr);
  b->part_gen.resize(n);
  for (int f = 0; f < n; ++f) b->part_gen[f] = b->grids[f]->part_gen;
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, b->device) == hipSuccess && cus > 0)
    b->cus = cus;
  if (hipEventCreateWithFlags(&b->done, hipEventDisableTiming) != hipSuccess) return YYG_ERR_DEVICE;
  if (hipStreamCreate(&b->stream) != hipSuccess) return YYG_ERR_DEVICE;
  // folded phi transforms when every plan is mirror-symmetric (one launch
  // mode for all plans)
  b->sep_fold = true;
  for (int f = 0; f < n; ++f) b->sep_fold = b->sep_fold && b->grids[f]->sep.fold;
  const size_t pb = n * sizeof(yyg::GemmF64Args), qb = n * sizeof(yyg::PhiQuadArgs);
  b->args_bytes = 2 * (pb + qb);
  if (hipHostMalloc(reinterpret_cast<void **>(&b->h_args), b->args_bytes, 0) != hipSuccess ||
      dev_malloc(reinterpret_cast<void **>(&b->d_args), b->args_bytes) != hipSuccess) {
    (void)hipGetLastError();
    return YYG_ERR_OUT_OF_MEMORY;
  }
  for (int r = 0; r < 2; ++r) {
    b->h_phi[r] = reinterpret_cast<yyg::GemmF64Args *>(b->h_args + r * pb);
    b->d_phi[r] = reinterpret_cast<yyg::GemmF64Args *>(b->d_args + r * pb);
    b->h_quad[r] = reinterpret_cast<yyg::PhiQuadArgs *>(b->h_args + 2 * pb + r * qb);
    b->d_quad[r] = reinterpret_cast<yyg::PhiQuadArgs *>(b->d_args + 2 * pb + r * qb);
  }
  std::vector<yyg::SepPhaseArgs> sargs(n);
  std::vector<yyg::ThetaArgs> theta(n);
  std::vector<yyg::ScanQArgs> qscan(n);
  std::vector<int2> qitems;
  for (int f = 0; f < n; ++f) {
    yyg_grid *g = b->grids[f];
    auto &S = g->sep;
    b->h_phi[0][f] = b->sep_fold ? S.phi_ana_f : S.phi_ana;
    b->h_phi[1][f] = b->sep_fold ? S.phi_syn_f : S.phi_syn;
    b->h_quad[0][f] = S.quad_ana;
    b->h_quad[1][f] = S.quad_syn;
    theta[f] = S.theta;
    sargs[f] = S.args;
    const int chunk = ((g->n_r + 63) / 64) | 1;
    qscan[f] = yyg::ScanQArgs{g->n_patch == 2 ? S.At : g->d_Ahat, S.coefS, g->d_qdeg, g->n_r, g->L, chunk,
                              g->n_patch, -g->G, S.Ut};
    b->max_nr = std::max(b->max_nr, g->n_r);
  }
  // the longest columns first, two per block where several such blocks fit a CU
  b->scan_two = yyg::radial_scan_q_two(b->max_nr);
  std::vector<int> order(n);
  for (int f = 0; f < n; ++f) order[f] = f;
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return b->grids[x]->n_r > b->grids[y]->n_r; });
  for (int f : order)
    for (int l = 0; l <= b->grids[f]->L; ++l)
      for (int k = 0; k < 2 * l + 1; k += b->scan_two ? 2 : 1) qitems.push_back(int2{f, l * l + k});
  int st = upload(&b->d_sargs, sargs);
  if (st == YYG_OK) st = upload(&b->d_theta, theta);
  if (st == YYG_OK) st = upload(&b->d_qscan, qscan);
  if (st == YYG_OK) st = upload(&b->d_qitems, qitems);
  b->n_qitems = (int)qitems.size();
  // the sweeps where every plan can run them; else tiles: 64 x 80 for the phi analysis, 128 x 48 for the phi
  // synthesis, 32 x 32 for the theta phases and the rotation
  const int def[5] = {3, 0, 0, 0, 4};
  for (int r = 0; r < 5 && st == YYG_OK; ++r)
    st = sep_batch_set_items(b, r, sep_batch_sweeps(b, r) ? yyg::sep_batch_tile_count() : def[r]);
  return st;
}

// The batched separable solve on s; with ev (6 events) recorded before
// the argument copies and after each of the six launches.
hipError_t sep_batch_enqueue(yyg_batch *b, hipStream_t s, hipEvent_t *ev) {
  hipError_t e = hipSuccess;
  auto mark = [&](int i) {
    if (ev && e == hipSuccess) e = hipEventRecord(ev[i], s);
  };
  mark(0);
  e = hipMemcpyAsync(b->d_args, b->h_args, b->args_bytes, hipMemcpyHostToDevice, s);
  auto phase = [&](int r) {
    if (e != hipSuccess) return;
    const bool sweep = b->svar[r] == yyg::sep_batch_tile_count();
    if (sweep && (r == 0 || r == 4))
      e = yyg::launch_phi_group(r == 0, b->smax[r], b->d_quad[r == 0 ? 0 : 1], b->d_sitems[r], b->n_sitems[r], s);
    else if (sweep)
      e = yyg::launch_theta_group(r, b->smax[r], b->slds[r], b->d_theta, b->d_sitems[r], b->n_sitems[r], s);
    else
      e = yyg::launch_sep_batch_phase(b->svar[r], r, b->sep_fold, b->d_phi[r == 0 ? 0 : 1], b->d_sargs, b->d_sitems[r],
                                      b->n_sitems[r], b->sblocks[r], s);
  };
  phase(0);
  mark(1);
  phase(1);
  phase(2);
  mark(2);
  if (e == hipSuccess)
    e = yyg::launch_radial_scan_q_grouped(b->d_qscan, b->d_qitems, b->n_qitems, b->scan_two, b->max_nr, s);
  mark(3);
  phase(3);
  mark(4);
  phase(4);
  mark(5);
  return e;
}

}  // namespace

extern "C" {

int yyg_grid_create(const yyg_grid_desc *d, int device, yyg_grid **out) {
  if (!out) return YYG_ERR_INVALID_ARG;
  *out = nullptr;
  int st = yyg::validate_desc(d);
  if (st != YYG_OK) return st;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) {
    (void)hipGetLastError();
    return YYG_ERR_DEVICE;
  }
  if (device < 0 || device >= ndev) return YYG_ERR_INVALID_ARG;

  yyg_grid *g = new (std::nothrow) yyg_grid;
  if (!g) return YYG_ERR_OUT_OF_MEMORY;
  g->device = device;
  g->kind = d->kind;
  g->n_patch = d->kind == YYG_GRID_POLAR ? 1 : 2;
  g->n_r = d->n_r;
  g->n_t = d->n_theta;
  g->n_p = d->n_phi;
  g->L = d->lmax;
  g->Q = (d->lmax + 1) * (d->lmax + 1);
  g->G = d->G;
  g->nang = (long)g->n_t * g->n_p;
  g->ldb = round_up(g->nang, 16);
  g->ldy = round_up((long)g->n_patch * g->Q, 16);
  g->r_edges.assign(d->r_edges, d->r_edges + d->n_r + 1);
  g->geom = d->kind == YYG_GRID_POLAR ? yyg::make_polar_patch(g->n_t, g->n_p)
                                      : yyg::make_patch(g->n_t, g->n_p, d->delta_theta, d->delta_phi);
  const int L = g->L, Q = g->Q, n_r = g->n_r;
  const long M = (long)g->n_patch * n_r;
  {
    int bm, bn;
    yyg::gemm_f64_variant_tile(g->var_ana, &bm, &bn);
    g->nsplit = yyg::choose_split(((M + bm - 1) / bm) * ((Q + bn - 1) / bn), g->nang);
    g->part_cap = g->nsplit;
    if (fold_large(g) && !fold_wanted(g)) {
      low_degree_shape(g, &g->var_ana, &g->var_syn, &g->nsplit);
      g->part_cap = g->nsplit;
    }
    if (fold_wanted(g)) fold_shape(g, &g->fold.var_ana, &g->fold.var_syn, &g->fold.nsplit);
  }

  std::vector<double> Tt, CS, coef, P, Tr, Yx;
  std::vector<int> qdeg(Q);
  try {
    g->w_host.resize(g->nang);
    yyg::overlap_weights(g->geom, g->w_host.data());
    Tt.resize((size_t)g->n_t * Q);
    yyg::theta_table_normalised(g->geom, L, Tt.data());
    CS.resize((size_t)g->n_p * Q);
    yyg::phi_table(g->geom, L, CS.data());
    coef.resize((size_t)4 * n_r * (L + 1));
    yyg::radial_coefficients(n_r, g->r_edges.data(), L, coef.data());
    P.resize((size_t)g->n_t * Q);
    yyg::self_legendre_table(g->geom, L, P.data());
    Tr.resize((size_t)g->n_p * Q);
    yyg::self_trig_table(g->geom, L, Tr.data());
    if (g->n_patch == 2) {
      Yx.resize((size_t)g->nang * Q);
      yyg::cross_basis(g->geom, L, Yx.data());
    }
    auto cols = yyg::column_table(L);
    auto s = yyg::norm_sqrt(L);
    g->nrm_q.resize(Q);
    for (int q = 0; q < Q; ++q) {
      qdeg[q] = cols[q].l;
      g->nrm_q[q] = s[cols[q].l * (L + 1) + cols[q].m];
    }
  } catch (const std::bad_alloc &) {
    free_grid(g);
    return YYG_ERR_OUT_OF_MEMORY;
  }

  DeviceGuard dg(device);
  if (!dg.ok) {
    free_grid(g);
    return YYG_ERR_DEVICE;
  }
  {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && cus > 0)
      g->cus = cus;
  }
  double *d_w = nullptr, *d_Tt = nullptr, *d_CS = nullptr, *d_P = nullptr, *d_Tr = nullptr;
  auto cleanup_tmp = [&] {
    double *t[] = {d_w, d_Tt, d_CS, d_P, d_Tr};
    for (double *b : t)
      if (b) (void)dev_free(b);
  };
  st = YYG_OK;
  if (st == YYG_OK) st = dmalloc(&g->d_Bt, (size_t)Q * g->ldb);
  if (st == YYG_OK) st = dmalloc(&g->d_Y, (size_t)g->nang * g->ldy);
  if (st == YYG_OK) st = dmalloc(&g->d_coef, coef.size());
  if (st == YYG_OK) st = dmalloc(&g->d_qdeg, (size_t)Q);
  if (st == YYG_OK) st = dmalloc(&g->d_part, (size_t)g->part_cap * M * Q);
  if (st == YYG_OK) st = dmalloc(&g->d_Ahat, (size_t)M * Q);
  if (st == YYG_OK) st = dmalloc(&g->d_U, (size_t)M * g->ldy);
  if (st == YYG_OK) st = dmalloc(&d_w, (size_t)g->nang);
  if (st == YYG_OK) st = dmalloc(&d_Tt, Tt.size());
  if (st == YYG_OK) st = dmalloc(&d_CS, CS.size());
  if (st == YYG_OK) st = dmalloc(&d_P, P.size());
  if (st == YYG_OK) st = dmalloc(&d_Tr, Tr.size());
  if (st != YYG_OK) {
    cleanup_tmp();
    free_grid(g);
    return st;
  }
  hipError_t e = hipSuccess;
  auto chk = [&](hipError_t r) {
    if (e == hipSuccess && r != hipSuccess) e = r;
  };
  chk(hipMemcpy(g->d_coef, coef.data(), coef.size() * sizeof(double), hipMemcpyHostToDevice));
  chk(hipMemcpy(g->d_qdeg, qdeg.data(), qdeg.size() * sizeof(int), hipMemcpyHostToDevice));
  chk(hipMemcpy(d_w, g->w_host.data(), g->nang * sizeof(double), hipMemcpyHostToDevice));
  chk(hipMemcpy(d_Tt, Tt.data(), Tt.size() * sizeof(double), hipMemcpyHostToDevice));
  chk(hipMemcpy(d_CS, CS.data(), CS.size() * sizeof(double), hipMemcpyHostToDevice));
  chk(hipMemcpy(d_P, P.data(), P.size() * sizeof(double), hipMemcpyHostToDevice));
  chk(hipMemcpy(d_Tr, Tr.data(), Tr.size() * sizeof(double), hipMemcpyHostToDevice));
  chk(hipMemset(g->d_U, 0, (size_t)M * g->ldy * sizeof(double)));
  chk(hipMemset(g->d_Ahat, 0, (size_t)M * Q * sizeof(double)));
  if (e == hipSuccess) chk(yyg::launch_expand_analysis_basis(d_w, d_Tt, d_CS, g->n_t, g->n_p, Q, g->d_Bt, g->ldb, 0));
  if (e == hipSuccess) chk(yyg::launch_expand_self_basis(d_P, d_Tr, g->n_t, g->n_p, Q, g->d_Y, g->ldy, g->n_patch * Q, 0));
  // cross part: columns [Q, 2Q) of every row
  if (e == hipSuccess && g->n_patch == 2)
    chk(hipMemcpy2D(g->d_Y + Q, g->ldy * sizeof(double), Yx.data(), (size_t)Q * sizeof(double),
                    (size_t)Q * sizeof(double), g->nang, hipMemcpyHostToDevice));
  chk(hipDeviceSynchronize());
  cleanup_tmp();
  if (e != hipSuccess) {
    (void)hipGetLastError();
    free_grid(g);
    return YYG_ERR_DEVICE;
  }
  *out = g;
  return YYG_OK;
}

int yyg_grid_create_res(int n_r, const double *r_edges, double res_deg, int lmax, double G, int device,
                        yyg_grid **out) {
  if (!(res_deg > 0.0) || !std::isfinite(res_deg) || res_deg > 90.0) return YYG_ERR_INVALID_ARG;
  yyg_grid_desc d;
  std::memset(&d, 0, sizeof(d));
  d.kind = YYG_GRID_YINYANG;
  d.n_r = n_r;
  d.r_edges = r_edges;
  yyg::dims_from_resolution(res_deg, &d.n_theta, &d.n_phi, &d.delta_theta, &d.delta_phi);
  d.lmax = lmax;
  d.G = G;
  return yyg_grid_create(&d, device, out);
}

int yyg_grid_dims(const yyg_grid *g, int *n_r, int *n_theta, int *n_phi, int *Q) {
  if (!g) return YYG_ERR_INVALID_ARG;
  if (n_r) *n_r = g->n_r;
  if (n_theta) *n_theta = g->n_t;
  if (n_phi) *n_phi = g->n_p;
  if (Q) *Q = g->Q;
  return YYG_OK;
}

int yyg_grid_kind(const yyg_grid *g, int *kind, int *patches) {
  if (!g) return YYG_ERR_INVALID_ARG;
  if (kind) *kind = g->kind;
  if (patches) *patches = g->n_patch;
  return YYG_OK;
}

int yyg_prepare(yyg_grid *g, int precision) {
  if (!g) return YYG_ERR_INVALID_ARG;
  if (precision == YYG_FP64) {
    if (g->method == YYG_METHOD_DENSE) fold_try(g);
    return YYG_OK;
  }
  if (precision < 0 || precision > YYG_FP16X2) return YYG_ERR_INVALID_ARG;
  auto &L = g->lp[precision - 1];
  if (L.ready) return YYG_OK;
  DeviceGuard dg(g->device);
  if (!dg.ok) return YYG_ERR_DEVICE;
  const int Q = g->Q;
  const long M = (long)g->n_patch * g->n_r;
  const int parts = yyg::lp_parts(precision), eb = yyg::lp_elem_bytes(precision), bk = yyg::lp_stage_k(precision);
  L.ldb = round_up(g->nang, std::max(bk, 16));
  L.ldy = round_up((long)g->n_patch * Q, std::max(bk, 16));
  L.lda = L.ldb;
  L.ldu = L.ldy;
  const size_t bt_plane = (size_t)Q * L.ldb, y_plane = (size_t)g->nang * L.ldy;
  int st = YYG_OK;
  auto bmalloc = [&](void **ptr, size_t bytes) {
    if (st != YYG_OK) return;
    if (dev_malloc(ptr, bytes) != hipSuccess) {
      *ptr = nullptr;
      (void)hipGetLastError();
      st = YYG_ERR_OUT_OF_MEMORY;
    }
  };
  bmalloc(&L.Bt, bt_plane * parts * eb);
  bmalloc(reinterpret_cast<void **>(&L.eBt), (size_t)Q * sizeof(int));
  bmalloc(&L.Y, y_plane * parts * eb);
  bmalloc(reinterpret_cast<void **>(&L.eY), (size_t)g->nang * sizeof(int));
  bmalloc(&L.Ar, (size_t)M * L.lda * parts * eb);
  bmalloc(&L.Ur, (size_t)M * L.ldu * parts * eb);
  if (!g->d_eA) bmalloc(reinterpret_cast<void **>(&g->d_eA), (size_t)M * sizeof(int));
  if (!g->d_eU) bmalloc(reinterpret_cast<void **>(&g->d_eU), (size_t)M * sizeof(int));
  if (st != YYG_OK) {
    lp_release(L);
    return st;
  }
  hipError_t e = hipSuccess;
  auto chk = [&](hipError_t r) {
    if (e == hipSuccess && r != hipSuccess) e = r;
  };
  chk(yyg::launch_row_exponent(g->d_Bt, g->ldb, Q, (int)g->nang, L.eBt, 0));
  chk(yyg::launch_split_rows(precision, g->d_Bt, g->ldb, Q, (int)g->nang, L.eBt, L.Bt, L.ldb, (long)bt_plane, 0));
  chk(yyg::launch_row_exponent(g->d_Y, g->ldy, (int)g->nang, g->n_patch * Q, L.eY, 0));
  chk(yyg::launch_split_rows(precision, g->d_Y, g->ldy, (int)g->nang, g->n_patch * Q, L.eY, L.Y, L.ldy, (long)y_plane, 0));
  chk(hipDeviceSynchronize());
  if (e != hipSuccess) {
    (void)hipGetLastError();
    lp_release(L);
    return YYG_ERR_DEVICE;
  }
  int bm, bn;
  yyg::gemm_lp_variant_tile(0, &bm, &bn);
  L.var_ana = 0;
  L.var_syn = 0;
  L.nsplit = yyg::choose_split(((M + bm - 1) / bm) * ((Q + bn - 1) / bn), g->nang);
  if (L.nsplit > g->part_cap) {
    double *np = nullptr;
    if (dmalloc(&np, (size_t)L.nsplit * M * Q) != YYG_OK) {
      lp_release(L);
      return YYG_ERR_OUT_OF_MEMORY;
    }
    (void)dev_free(g->d_part);
    g->d_part = np;
    g->part_gen += 1;
    g->part_cap = L.nsplit;
  }
  L.ready = true;
  return YYG_OK;
}

int yyg_upload_rho(yyg_grid *g, const double *rho, int rho_is_device, void *stream) {
  if (!g || !rho) return YYG_ERR_INVALID_ARG;
  // the solve that follows cannot allocate
  if (g->method == YYG_METHOD_DENSE && !g->fold.tried && fold_wanted(g) && !capturing(as_stream(stream))) fold_try(g);
  if (rho_is_device) {
    g->rho = rho;
    return YYG_OK;
  }
  DeviceGuard dg(g->device);
  if (!dg.ok) return YYG_ERR_DEVICE;
  const size_t bytes = (size_t)g->n_patch * g->n_r * g->nang * sizeof(double);
  if (!g->d_rho_owned) {
    int st = dmalloc(&g->d_rho_owned, bytes / sizeof(double));
    if (st != YYG_OK) return st;
  }
  if (hipMemcpyAsync(g->d_rho_owned, rho, bytes, hipMemcpyHostToDevice, as_stream(stream)) != hipSuccess) {
    (void)hipGetLastError();
    return YYG_ERR_DEVICE;
  }
  g->rho = g->d_rho_owned;
  return YYG_OK;
}

int yyg_solve(yyg_grid *g, double *phi, int phi_is_device, int precision, void *stream) {
  if (!g || !phi) return YYG_ERR_INVALID_ARG;
  if (precision < 0 || precision > YYG_FP16X2) return YYG_ERR_INVALID_ARG;
  const bool sep_form = g->method == YYG_METHOD_SEPARABLE;
  // the separable form converts its operands in the kernels (nothing to
  // prepare); FP16's exponent range would need row scaling it does not do
  if (sep_form && precision == YYG_FP16X2) return YYG_ERR_UNSUPPORTED;
  if (!sep_form && precision != YYG_FP64 && !g->lp[precision - 1].ready) return YYG_ERR_NOT_READY;
  if (!g->rho) return YYG_ERR_NOT_READY;
  DeviceGuard dg(g->device);
  if (!dg.ok) return YYG_ERR_DEVICE;
  hipStream_t s = as_stream(stream);
  if (int st = check_rho(g, g->rho, s); st != YYG_OK) return st;
  const int Q = g->Q, n_r = g->n_r;
  const long M = (long)g->n_patch * n_r;
  double *out = phi;
  double *tmp = nullptr;
  if (!phi_is_device) {
    if (dmalloc(&tmp, (size_t)M * g->nang) != YYG_OK) return YYG_ERR_OUT_OF_MEMORY;
    out = tmp;
  }
  hipError_t e = hipSuccess;
  int t;
  const bool lp = precision != YYG_FP64;
  const bool scaled = precision == YYG_FP16X2;
  if (g->method == YYG_METHOD_SEPARABLE) {
    int st = sep_set_pointers(g, g->rho, out, s);
    if (st != YYG_OK) {
      if (tmp) (void)dev_free(tmp);
      return st;
    }
    e = sep_solve(g, s, precision);
    if (!phi_is_device) {
      if (e == hipSuccess)
        e = hipMemcpyAsync(phi, out, (size_t)M * g->nang * sizeof(double), hipMemcpyDeviceToHost, s);
      if (e == hipSuccess) e = hipStreamSynchronize(s);
      (void)dev_free(tmp);
      g->sep.phi_syn.C = nullptr;  // the temporary is gone
      g->sep.phi_syn_d.C = nullptr;
      g->sep.phi_syn_f.C = nullptr;
      g->sep.phi_syn_s.phi = nullptr;
      g->sep.quad_syn.C = nullptr;
      g->sep.phi_syn_l.C = nullptr;
    }
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return YYG_ERR_DEVICE;
    }
    return YYG_OK;
  }
  g->ahat_cols = false;
  FoldUse fold(lp ? nullptr : g, s);
  g->ahat_fold = (bool)fold;
  const int nsplit = lp ? g->lp[precision - 1].nsplit : fold ? g->fold.nsplit : g->nsplit;
  double *part = fold && nsplit > g->part_cap ? g->fold.part : g->d_part;
  if (lp) {
    // split the density into operand planes (rows scaled for FP16)
    const auto &L = g->lp[precision - 1];
    t = timing_begin(g, 3, s);
    if (scaled) e = yyg::launch_row_exponent(g->rho, g->nang, (int)M, (int)g->nang, g->d_eA, s);
    if (e == hipSuccess)
      e = yyg::launch_split_rows(precision, g->rho, g->nang, (int)M, (int)g->nang, scaled ? g->d_eA : nullptr, L.Ar,
                                 L.lda, M * L.lda, s);
    timing_end(g, t, s);
  }
  if (e == hipSuccess) {
    t = timing_begin(g, 0, s);
    if (fold) {
      e = yyg::launch_fold_rows(g->rho, g->fold.F, (int)M, g->n_t, g->n_p, s);
      if (e == hipSuccess) e = fold_analysis(g, g->fold.var_ana, nsplit, part, s);
    } else if (!lp) {
      e = yyg::launch_gemm_nt_f64(g->var_ana, 0, (int)M, Q, (int)g->nang, g->rho, g->nang, g->d_Bt, g->ldb,
                                  g->d_part, Q, nsplit, M * Q, s);
    } else {
      const auto &L = g->lp[precision - 1];
      e = yyg::launch_gemm_nt_lp(precision, L.var_ana, 0, (int)M, Q, (int)g->nang, L.Ar, L.lda, M * L.lda,
                                 scaled ? g->d_eA : nullptr, L.Bt, L.ldb, (long)Q * L.ldb, L.eBt, g->d_part, Q,
                                 nsplit, M * Q, s);
    }
    timing_end(g, t, s);
  }
  if (e == hipSuccess) {
    t = timing_begin(g, 1, s);
    e = yyg::launch_radial_scan(part, nsplit, M * Q, g->d_Ahat, g->d_coef, fold ? g->fold.d_deg : g->d_qdeg, n_r,
                                Q, g->L, -g->G, g->d_U, g->ldy, g->n_patch, s, fold ? g->fold.d_ucol : nullptr);
    timing_end(g, t, s);
  }
  if (e == hipSuccess && lp) {
    const auto &L = g->lp[precision - 1];
    t = timing_begin(g, 3, s);
    if (scaled) e = yyg::launch_row_exponent(g->d_U, g->ldy, (int)M, g->n_patch * Q, g->d_eU, s);
    if (e == hipSuccess)
      e = yyg::launch_split_rows(precision, g->d_U, g->ldy, (int)M, g->n_patch * Q, scaled ? g->d_eU : nullptr, L.Ur, L.ldu,
                                 M * L.ldu, s);
    timing_end(g, t, s);
  }
  if (e == hipSuccess) {
    t = timing_begin(g, 2, s);
    if (fold) {
      e = fold_synthesis(g, g->fold.var_syn, s);
      if (e == hipSuccess) e = yyg::launch_unfold_rows(g->fold.F, out, (int)M, g->n_t, g->n_p, s);
    } else if (!lp) {
      e = yyg::launch_gemm_nt_f64(g->var_syn, 1, (int)M, (int)g->nang, g->n_patch * Q, g->d_U, g->ldy, g->d_Y, g->ldy, out,
                                  g->nang, 1, 0, s);
    } else {
      const auto &L = g->lp[precision - 1];
      e = yyg::launch_gemm_nt_lp(precision, L.var_syn, 1, (int)M, (int)g->nang, g->n_patch * Q, L.Ur, L.ldu, M * L.ldu,
                                 scaled ? g->d_eU : nullptr, L.Y, L.ldy, (long)g->nang * L.ldy, L.eY, out, g->nang,
                                 1, 0, s);
    }
    timing_end(g, t, s);
  }
  if (!phi_is_device) {
    if (e == hipSuccess)
      e = hipMemcpyAsync(phi, out, (size_t)M * g->nang * sizeof(double), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)dev_free(tmp);
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return YYG_ERR_DEVICE;
  }
  return YYG_OK;
}

int yyg_solve_noalloc(yyg_grid *g, const double *rho, double *phi, void *stream) {
  if (!g || !rho || !phi) return YYG_ERR_INVALID_ARG;
  if (g->method != YYG_METHOD_SEPARABLE || !g->sep.ready) return YYG_ERR_NOT_READY;
  DeviceGuard dg(g->device);
  if (!dg.ok) return YYG_ERR_DEVICE;
  double *base = nullptr;
  size_t bytes = 0;
  if (yyg::scratch_region(g->device, &base, &bytes) != hipSuccess) {
    (void)hipGetLastError();
    return YYG_ERR_DEVICE;
  }
  if (sep_work_doubles(g) * sizeof(double) > bytes) return YYG_ERR_UNSUPPORTED;
  if (int st = check_rho(g, rho, as_stream(stream)); st != YYG_OK) return st;
  // carve the work buffers out of the scratch array; every one of them is
  // written in full by its phase before any later phase reads it, so none
  // needs clearing
  const long M = (long)g->n_patch * g->n_r, nmc = 2L * g->L + 1;
  auto r32 = [](long v) { return (v + 31) / 32 * 32; };
  SepWork w{};
  double *p = base;
  w.X2 = p, p += r32(nmc * g->n_t * M);
  w.V = p, p += r32(nmc * g->n_t * M);
  w.Ut = p, p += r32(nmc * (g->L + 1) * M);
  w.At = g->n_patch == 2 ? p : nullptr, p += g->n_patch == 2 ? r32(M * g->Q) : 0;
  w.Ahat = p;
  const SepWork own = sep_work(g);
  const bool timing = g->timing, cols = g->ahat_cols, folded = g->ahat_fold;
  g->timing = false;  // no events: nothing is created
  sep_bind_work(g, w);
  hipStream_t s = as_stream(stream);
  hipError_t e = hipSuccess;
  if (sep_set_pointers(g, rho, phi, s) != YYG_OK) e = hipErrorInvalidValue;
  if (e == hipSuccess) e = sep_solve(g, s);
  sep_bind_work(g, own);
  g->timing = timing;
  g->ahat_fold = folded;
  g->ahat_cols = cols;  // the plan's moments buffer still holds the last yyg_solve's
  sep_set_pointers(g, nullptr, nullptr, s);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return YYG_ERR_DEVICE;
  }
  return YYG_OK;
}

int yyg_set_check_finite(yyg_grid *g, int on) {
  if (!g) return YYG_ERR_INVALID_ARG;
  if (on && !g->d_flag) {
    DeviceGuard dg(g->device);
    if (!dg.ok) return YYG_ERR_DEVICE;
    if (int st = dmalloc(&g->d_flag, 1); st != YYG_OK) return st;
  }
  g->check_finite = on != 0;
  return YYG_OK;
}

int yyg_device_bytes(size_t *held) {
  if (!held) return YYG_ERR_INVALID_ARG;
  std::lock_guard<std::mutex> lock(g_mem_mu);
  *held = g_mem_held;
  return YYG_OK;
}

int yyg_get_moments(yyg_grid *g, double *A_host) {
  if (!g || !A_host) return YYG_ERR_INVALID_ARG;
  DeviceGuard dg(g->device);
  if (!dg.ok) return YYG_ERR_DEVICE;
  const long M = (long)g->n_patch * g->n_r;
  if (hipDeviceSynchronize() != hipSuccess ||
      hipMemcpy(A_host, g->d_Ahat, (size_t)M * g->Q * sizeof(double), hipMemcpyDeviceToHost) != hipSuccess) {
    (void)hipGetLastError();
    return YYG_ERR_DEVICE;
  }
  if (g->ahat_cols) {
    std::vector<double> t(A_host, A_host + M * g->Q);
    for (long r = 0; r < M; ++r)
      for (int q = 0; q < g->Q; ++q) A_host[r * g->Q + q] = t[q * M + r];
  } else if (g->ahat_fold) {
    std::vector<double> t(g->Q);
    for (long r = 0; r < M; ++r) {
      std::copy(A_host + r * g->Q, A_host + (r + 1) * g->Q, t.begin());
      for (int n = 0; n < g->Q; ++n) A_host[r * g->Q + g->fold.cols[n]] = t[n];
    }
  }
  for (long r = 0; r < M; ++r)
    for (int q = 0; q < g->Q; ++q) A_host[r * g->Q + q] /= g->nrm_q[q];
  return YYG_OK;
}

int yyg_get_weights(const yyg_grid *g, double *w_host) {
  if (!g || !w_host) return YYG_ERR_INVALID_ARG;
  std::memcpy(w_host, g->w_host.data(), g->w_host.size() * sizeof(double));
  return YYG_OK;
}

int yyg_grid_destroy(yyg_grid *g) {
  if (!g) return YYG_ERR_INVALID_ARG;
  DeviceGuard dg(g->device);
  (void)hipDeviceSynchronize();
  free_grid(g);
  return YYG_OK;
}

int yyg_set_timing(yyg_grid *g, int enable) {
  if (!g) return YYG_ERR_INVALID_ARG;
  DeviceGuard dg(g->device);
  (void)hipDeviceSynchronize();
  for (auto &t : g->launches) {
    (void)hipEventDestroy(t.start);
    (void)hipEventDestroy(t.stop);
  }
  g->launches.clear();
  g->timing = enable != 0;
  return YYG_OK;
}

int yyg_get_timing(yyg_grid *g, double *ms, long *counts, int n_slots) {
  if (!g || !ms || !counts || n_slots < 1 || n_slots > kSlots) return YYG_ERR_INVALID_ARG;
  DeviceGuard dg(g->device);
  for (int i = 0; i < n_slots; ++i) {
    ms[i] = 0.0;
    counts[i] = 0;
  }
  for (auto &t : g->launches) {
    if (hipEventSynchronize(t.stop) != hipSuccess) {
      (void)hipGetLastError();
      return YYG_ERR_DEVICE;
    }
    float v = 0.f;
    if (hipEventElapsedTime(&v, t.start, t.stop) != hipSuccess) {
      (void)hipGetLastError();
      return YYG_ERR_DEVICE;
    }
    if (t.slot < n_slots) {
      ms[t.slot] += v;
      counts[t.slot] += 1;
    }
  }
  return YYG_OK;
}

int yyg_set_method(yyg_grid *g, int method) {
  if (!g || (method != YYG_METHOD_DENSE && method != YYG_METHOD_SEPARABLE)) return YYG_ERR_INVALID_ARG;
  if (method == YYG_METHOD_SEPARABLE && !g->sep.ready) {
    DeviceGuard dg(g->device);
    if (!dg.ok) return YYG_ERR_DEVICE;
    if (hipDeviceSynchronize() != hipSuccess) {
      (void)hipGetLastError();
      return YYG_ERR_DEVICE;
    }
    int st = sep_build(g);
    if (st != YYG_OK) return st;
    fold_release(g, true);  // a plan that goes back to the dense form builds it again and keeps it
  }
  g->method = method;
  if (method == YYG_METHOD_DENSE && !g->fold.tried) fold_try(g);
  return YYG_OK;
}

int yyg_autotune(yyg_grid *g, int precision, void *stream) {
  if (!g) return YYG_ERR_INVALID_ARG;
  if (precision < 0 || precision > YYG_FP16X2) return YYG_ERR_INVALID_ARG;
  const bool lp = precision != YYG_FP64;
  const bool sep_form = g->method == YYG_METHOD_SEPARABLE;
  if (sep_form && precision == YYG_FP16X2) return YYG_ERR_UNSUPPORTED;
  if (lp && !sep_form && !g->lp[precision - 1].ready) return YYG_ERR_NOT_READY;
  DeviceGuard dg(g->device);
  if (!dg.ok) return YYG_ERR_DEVICE;
  hipStream_t s = as_stream(stream);
  if (lp && sep_form) {
    // the reduced-precision phi transforms of the separable form: each
    // tile shape timed inside whole solves, phi analysis then synthesis
    if (!g->sep.ready) return YYG_ERR_NOT_READY;
    const long Mt = (long)g->n_patch * g->n_r;
    double *phi_t = nullptr, *rho_t = nullptr;
    int st = dmalloc(&phi_t, (size_t)Mt * g->nang);
    if (st == YYG_OK && !g->rho) {
      st = dmalloc(&rho_t, (size_t)Mt * g->nang);
      if (st == YYG_OK) (void)hipMemsetAsync(rho_t, 0, (size_t)Mt * g->nang * sizeof(double), s);
    }
    if (st == YYG_OK) st = sep_set_pointers(g, g->rho ? g->rho : rho_t, phi_t, s);
    const bool timing = g->timing;
    g->timing = false;
    auto solve_ms = [&]() { return time_launch([&] { return sep_solve(g, s, precision); }, s, 5); };
    for (int r = 0; r < 2 && st == YYG_OK; ++r) {
      int &cur = g->sep.lpt[precision - 1][r];
      int best = cur;
      double bt = solve_ms() - 1e-4;
      const int t0 = cur;
      for (int t = 0; t < sep_lp_choices(g, precision, r); ++t) {
        if (t == t0 || !sep_lp_available(g, precision, r, t)) continue;
        cur = t;
        const double tm = solve_ms();
        if (tm < bt) {
          bt = tm;
          best = t;
        }
      }
      cur = best;
    }
    g->timing = timing;
    (void)hipStreamSynchronize(s);
    if (phi_t) (void)dev_free(phi_t);
    if (rho_t) (void)dev_free(rho_t);
    sep_set_pointers(g, nullptr, nullptr, s);
    return st;
  }
  const int Q = g->Q;
  const long M = (long)g->n_patch * g->n_r;
  const int nv = lp ? yyg::gemm_lp_variant_count() : yyg::gemm_f64_variant_count();
  auto tile = [&](int v, int *bm, int *bn) {
    if (lp)
      yyg::gemm_lp_variant_tile(v, bm, bn);
    else
      yyg::gemm_f64_variant_tile(v, bm, bn);
  };
  const char *cache_path = std::getenv("YYG_TUNE_CACHE");
  auto cache = read_tune_cache(cache_path);
  // a plan in the separable form tunes that form's phases only (FP64): the
  // dense contractions keep their configuration
  const bool sep_only = !lp && sep_form;
  if (!lp && !sep_only) fold_try(g);
  FoldUse fold(lp || sep_only ? nullptr : g, s);
  double *tmp_in = nullptr, *tmp_out = nullptr, *tmp_part = nullptr, *tmp_A = nullptr, *tmp_U = nullptr;
  const int smax = 32;
  long cells = 0;
  std::string ka, ks;
  int best_va = 0, best_sp = 1, best_vs = 0;
  bool have_a = sep_only, have_s = sep_only;
  for (int st = YYG_ERR_OUT_OF_MEMORY; st != YYG_OK;) {
    // the folded solve's four contractions over a quarter patch rank the
    // tiles differently than one contraction of the same sizes: roles of
    // their own
    cells = fold ? g->fold.hq : g->nang;
    ka = tune_key(precision, fold ? 2 : 0, M, Q, cells);
    ks = tune_key(precision, fold ? 3 : 1, M, cells, (long)g->n_patch * Q);
    best_va = lp ? g->lp[precision - 1].var_ana : fold ? g->fold.var_ana : g->var_ana;
    best_sp = lp ? g->lp[precision - 1].nsplit : fold ? g->fold.nsplit : g->nsplit;
    best_vs = lp ? g->lp[precision - 1].var_syn : fold ? g->fold.var_syn : g->var_syn;
    if (!sep_only && cache.count(ka)) {
      best_va = cache[ka].first;
      best_sp = cache[ka].second;
      have_a = best_va >= 0 && best_va < nv && best_sp >= 1 && best_sp <= 32;
    }
    if (!sep_only && cache.count(ks)) {
      best_vs = cache[ks].first;
      have_s = best_vs >= 0 && best_vs < nv;
    }
    if (have_a && have_s) break;
    // (the folded contractions run in the fold's own buffers)
    st = dmalloc(&tmp_part, (size_t)smax * M * Q);
    if (!fold && st == YYG_OK && !g->rho) st = dmalloc(&tmp_in, (size_t)M * g->nang);
    if (!fold && st == YYG_OK) st = dmalloc(&tmp_out, (size_t)M * g->nang);
    if (st == YYG_OK && tmp_in) (void)hipMemsetAsync(tmp_in, 0, (size_t)M * g->nang * sizeof(double), s);
    if (st == YYG_OK) {
      // the scan's outputs, where there is room (the plan's own hold the last
      // solve's)
      if (!lp && !have_a && dmalloc(&tmp_A, (size_t)M * Q) == YYG_OK && dmalloc(&tmp_U, (size_t)M * g->ldy) != YYG_OK) {
        (void)dev_free(tmp_A);
        tmp_A = nullptr;
      }
      break;
    }
    for (double **t : {&tmp_in, &tmp_out, &tmp_part}) {
      if (*t) (void)dev_free(*t);
      *t = nullptr;
    }
    if (!fold) return st;
    fold.end();
    fold_release(g, false);
    if (g->fold.ready) return st;  // in a recorded graph
    have_a = have_s = false;       // unfolded, with the fold's memory
  }
  const double *rho = g->rho ? g->rho : tmp_in;
  const bool scaled = precision == YYG_FP16X2;
  if (lp && (!have_a || !have_s)) {
    const auto &L = g->lp[precision - 1];
    if (scaled) {
      (void)yyg::launch_row_exponent(rho, g->nang, (int)M, (int)g->nang, g->d_eA, s);
      (void)yyg::launch_row_exponent(g->d_U, g->ldy, (int)M, g->n_patch * Q, g->d_eU, s);
    }
    (void)yyg::launch_split_rows(precision, rho, g->nang, (int)M, (int)g->nang, scaled ? g->d_eA : nullptr, L.Ar,
                                 L.lda, M * L.lda, s);
    (void)yyg::launch_split_rows(precision, g->d_U, g->ldy, (int)M, g->n_patch * Q, scaled ? g->d_eU : nullptr, L.Ur, L.ldu,
                                 M * L.ldu, s);
  }
  auto ana = [&](int v, int sp) -> hipError_t {
    if (fold) return fold_analysis(g, v, sp, tmp_part, s);
    if (!lp)
      return yyg::launch_gemm_nt_f64(v, 0, (int)M, Q, (int)g->nang, rho, g->nang, g->d_Bt, g->ldb, tmp_part, Q, sp,
                                     M * Q, s);
    const auto &L = g->lp[precision - 1];
    return yyg::launch_gemm_nt_lp(precision, v, 0, (int)M, Q, (int)g->nang, L.Ar, L.lda, M * L.lda,
                                  scaled ? g->d_eA : nullptr, L.Bt, L.ldb, (long)Q * L.ldb, L.eBt, tmp_part, Q, sp,
                                  M * Q, s);
  };
  auto syn = [&](int v) -> hipError_t {
    if (fold) return fold_synthesis(g, v, s);
    if (!lp)
      return yyg::launch_gemm_nt_f64(v, 1, (int)M, (int)g->nang, g->n_patch * Q, g->d_U, g->ldy, g->d_Y, g->ldy, tmp_out,
                                     g->nang, 1, 0, s);
    const auto &L = g->lp[precision - 1];
    return yyg::launch_gemm_nt_lp(precision, v, 1, (int)M, (int)g->nang, g->n_patch * Q, L.Ur, L.ldu, M * L.ldu,
                                  scaled ? g->d_eU : nullptr, L.Y, L.ldy, (long)g->nang * L.ldy, L.eY, tmp_out,
                                  g->nang, 1, 0, s);
  };
  // an analysis with the scan that reads its partial moments (one more split
  // can cost the scan more than it saves: polar 90 x 180, 400 shells, degree 5
  // as created 94 us, and 113 with the 32 splits chosen where the scan was
  // charged their bytes at the memory's rate)
  auto ana_scan = [&](int v, int sp) -> hipError_t {
    const hipError_t e = ana(v, sp);
    if (e != hipSuccess || !tmp_U) return e;
    return yyg::launch_radial_scan(tmp_part, sp, M * Q, tmp_A, g->d_coef, fold ? g->fold.d_deg : g->d_qdeg, g->n_r, Q,
                                   g->L, -g->G, tmp_U, g->ldy, g->n_patch, s, fold ? g->fold.d_ucol : nullptr);
  };
  if (!have_a) {
    double best = 1e30;
    for (int v = 0; v < nv; ++v) {
      int bm, bn;
      tile(v, &bm, &bn);
      long tiles = ((M + bm - 1) / bm) * ((Q + bn - 1) / bn);
      if (fold) tiles = fold_analysis_tiles(g, bm, bn);
      int base = yyg::choose_split(tiles, cells);
      int cands[] = {1, 2, 4, 8, 16, 32, base};
      for (int sp : cands) {
        if (sp > smax || (long)sp * 64 > cells + 64) continue;
        double t = time_launch([&] { return ana_scan(v, sp); }, s, 3);
        // else the partials' bytes at HBM speed
        if (!tmp_U) t += (double)sp * M * Q * 8.0 / 5.0e9;
        if (t < best) {
          best = t;
          best_va = v;
          best_sp = sp;
        }
      }
    }
  }
  if (!have_s) {
    double best = 1e30;
    for (int v = 0; v < nv; ++v) {
      double t = time_launch([&] { return syn(v); }, s, 3);
      if (t < best) {
        best = t;
        best_vs = v;
      }
    }
  }
  if (tmp_in) (void)dev_free(tmp_in);
  if (tmp_out) (void)dev_free(tmp_out);
  if (tmp_part) (void)dev_free(tmp_part);
  if (tmp_A) (void)dev_free(tmp_A);
  if (tmp_U) (void)dev_free(tmp_U);
  if (best_sp > std::max(g->part_cap, fold ? g->fold.splits : 0)) {
    double *np = nullptr;
    if (dmalloc(&np, (size_t)best_sp * M * Q) == YYG_OK) {
      (void)hipDeviceSynchronize();
      (void)dev_free(g->d_part);
      g->d_part = np;
      g->part_gen += 1;
      g->part_cap = best_sp;
    } else if (fold) {
      best_sp = g->fold.nsplit;
    } else {
      return YYG_ERR_OUT_OF_MEMORY;
    }
  }
  (lp ? g->lp[precision - 1].var_ana : fold ? g->fold.var_ana : g->var_ana) = best_va;
  (lp ? g->lp[precision - 1].nsplit : fold ? g->fold.nsplit : g->nsplit) = best_sp;
  (lp ? g->lp[precision - 1].var_syn : fold ? g->fold.var_syn : g->var_syn) = best_vs;
  // separable form (FP64): tile variant of each grouped phase
  if (sep_only && g->sep.ready) {
    double *phi_t = nullptr, *rho_t = nullptr;
    int st3 = dmalloc(&phi_t, (size_t)M * g->nang);
    if (st3 == YYG_OK && !g->rho) {
      st3 = dmalloc(&rho_t, (size_t)M * g->nang);
      if (st3 == YYG_OK) (void)hipMemsetAsync(rho_t, 0, (size_t)M * g->nang * sizeof(double), s);
    }
    if (st3 == YYG_OK) st3 = sep_set_pointers(g, g->rho ? g->rho : rho_t, phi_t, s);
    // Each phase in turn (the others at their current choice): every
    // variant is timed inside whole back-to-back solves, where the kernels
    // meet the caches and clocks they run under in use (timed alone, the
    // short phases rank differently); a variant replaces the current one only
    // when the solve gets faster by more than 0.5% (at least 0.3 us), so that
    // near-ties do not flip between runs.
    auto solve_ms = [&]() { return time_launch([&] { return sep_solve(g, s); }, s, 5); };
    const bool timing = g->timing;
    g->timing = false;  // no per-phase events while tuning
    for (int r = 0; r < 5 && st3 == YYG_OK; ++r) {
      if (r == 2 && g->n_patch != 2) continue;  // one patch: no rotation
      const int v0 = g->sep.var[r];
      const double t0 = solve_ms();
      double best = t0 - std::max(0.0003, 0.005 * t0);
      int bv = v0;
      for (int v = 0; v < sep_variant_count(r) && st3 == YYG_OK; ++v) {
        if (v == v0 || !sep_variant_available(g, r, v)) continue;
        st3 = sep_set_variant(g, r, v);
        if (st3 != YYG_OK) break;
        const double t = solve_ms();
        if (t < best) {
          best = t;
          bv = v;
        }
      }
      if (st3 == YYG_OK) st3 = sep_set_variant(g, r, bv);
    }
    g->timing = timing;
    (void)hipStreamSynchronize(s);
    if (phi_t) (void)dev_free(phi_t);
    if (rho_t) (void)dev_free(rho_t);
    g->sep.phi_ana.A = nullptr;  // the next solve writes its own pointers
    g->sep.phi_syn.C = nullptr;
    g->sep.phi_ana_d.X = nullptr;
    g->sep.phi_syn_d.C = nullptr;
    g->sep.phi_ana_f.A = nullptr;
    g->sep.phi_ana_s.rho = nullptr;
    g->sep.phi_ana_ab.A = nullptr;
    g->sep.phi_syn_f.C = nullptr;
    g->sep.phi_syn_s.phi = nullptr;
    g->sep.quad_ana.X = nullptr;
    g->sep.quad_syn.C = nullptr;
    g->sep.phi_syn_l.C = nullptr;
    if (st3 != YYG_OK) return st3;
  }
  if (cache_path && !sep_only && (!have_a || !have_s)) {
    if (std::FILE *f = std::fopen(cache_path, "a")) {
      if (!have_a) std::fprintf(f, "%s -> %d %d\n", ka.c_str(), best_va, best_sp);
      if (!have_s) std::fprintf(f, "%s -> %d %d\n", ks.c_str(), best_vs, 1);
      std::fclose(f);
    }
  }
  return YYG_OK;
}

int yyg_plan_config(yyg_grid *g, int precision, int var_ana, int split_ana, int var_syn) {
  if (!g || precision < 0 || precision > YYG_FP16X2) return YYG_ERR_INVALID_ARG;
  const bool lp = precision != YYG_FP64;
  if (lp && !g->lp[precision - 1].ready) return YYG_ERR_NOT_READY;
  const int nv = lp ? yyg::gemm_lp_variant_count() : yyg::gemm_f64_variant_count();
  if (var_ana < 0 || var_ana >= nv || var_syn < 0 || var_syn >= nv || split_ana < 1 || split_ana > 64)
    return YYG_ERR_INVALID_ARG;
  DeviceGuard dg(g->device);
  if (!dg.ok) return YYG_ERR_DEVICE;
  if (split_ana > g->part_cap) {
    const long M = (long)g->n_patch * g->n_r;
    double *np = nullptr;
    if (dmalloc(&np, (size_t)split_ana * M * g->Q) != YYG_OK) return YYG_ERR_OUT_OF_MEMORY;
    (void)hipDeviceSynchronize();
    (void)dev_free(g->d_part);
    g->d_part = np;
    g->part_gen += 1;
    g->part_cap = split_ana;
  }
  if (lp) {
    auto &L = g->lp[precision - 1];
    L.var_ana = var_ana;
    L.nsplit = split_ana;
    L.var_syn = var_syn;
  } else {
    g->var_ana = g->fold.var_ana = var_ana;
    g->nsplit = g->fold.nsplit = split_ana;
    g->var_syn = g->fold.var_syn = var_syn;
  }
  return YYG_OK;
}

int yyg_plan_info(const yyg_grid *g, int precision, int *info, int n) {
  if (!g || !info || n < 1 || precision < 0 || precision > YYG_FP16X2) return YYG_ERR_INVALID_ARG;
  const bool lp = precision != YYG_FP64;
  int va = g->var_ana, sp = g->nsplit, vs = g->var_syn;
  bool folded;
  {
    std::lock_guard<std::mutex> lock(g_fold_mu);
    folded = !lp && g->fold.ready;
    if (folded || (fold_wanted(g) && !g->fold.tried)) {  // or to be built
      va = g->fold.var_ana;
      sp = g->fold.nsplit;
      vs = g->fold.var_syn;
    }
  }
  if (lp) {
    va = g->lp[precision - 1].var_ana;
    sp = g->lp[precision - 1].nsplit;
    vs = g->lp[precision - 1].var_syn;
  }
  int ba, bn_a, bs, bn_s;
  if (lp) {
    yyg::gemm_lp_variant_tile(va, &ba, &bn_a);
    yyg::gemm_lp_variant_tile(vs, &bs, &bn_s);
  } else {
    yyg::gemm_f64_variant_tile(va, &ba, &bn_a);
    yyg::gemm_f64_variant_tile(vs, &bs, &bn_s);
  }
  const int vals[8] = {va, sp, vs, ba, bn_a, bs, bn_s, folded};
  for (int i = 0; i < n && i < 8; ++i) info[i] = vals[i];
  return YYG_OK;
}

int yyg_sep_config(yyg_grid *g, int phase, int variant) {
  if (!g || phase < 0 || phase > 4) return YYG_ERR_INVALID_ARG;
  if (!g->sep.ready) return YYG_ERR_NOT_READY;
  if (variant < 0 || variant >= sep_variant_count(phase)) return YYG_ERR_INVALID_ARG;
  DeviceGuard dg(g->device);
  if (!dg.ok) return YYG_ERR_DEVICE;
  if (hipDeviceSynchronize() != hipSuccess) {  // the work items may be in use
    (void)hipGetLastError();
    return YYG_ERR_DEVICE;
  }
  return sep_set_variant(g, phase, variant);
}

int yyg_sep_variant_count(int phase) {
  if (phase < 0 || phase > 4) return YYG_ERR_INVALID_ARG;
  return sep_variant_count(phase);
}

int yyg_sep_info(const yyg_grid *g, int *variants, int n) {
  if (!g || !variants || n < 1) return YYG_ERR_INVALID_ARG;
  for (int i = 0; i < n && i < 5; ++i)
    variants[i] = (!g->sep.ready || (i == 2 && g->n_patch != 2)) ? -1 : g->sep.var[i];
  if (n > 5) variants[5] = g->sep.ready && g->sep.fold ? g->sep.quad_syn.K : 0;
  return YYG_OK;
}

int yyg_sep_phase(yyg_grid *g, int phase, double *phi, void *stream) {
  if (!g || !phi || phase < 0 || phase > 4) return YYG_ERR_INVALID_ARG;
  if (g->method != YYG_METHOD_SEPARABLE || !g->sep.ready || !g->rho) return YYG_ERR_NOT_READY;
  DeviceGuard dg(g->device);
  if (!dg.ok) return YYG_ERR_DEVICE;
  hipStream_t s = as_stream(stream);
  const int st = sep_set_pointers(g, g->rho, phi, s);
  if (st != YYG_OK) return st;
  if (sep_launch_phase(g, phase, s) != hipSuccess) {
    (void)hipGetLastError();
    return YYG_ERR_DEVICE;
  }
  return YYG_OK;
}

int yyg_sep_kernel(const yyg_grid *g, int phase, char *name, size_t n) {
  if (!g || !name || n < 1 || phase < 0 || phase > 4) return YYG_ERR_INVALID_ARG;
  if (!g->sep.ready) return YYG_ERR_NOT_READY;
  if (phase == 2 && g->n_patch != 2) {
    name[0] = 0;
    return YYG_OK;
  }
  const int v = g->sep.var[phase], x0 = sep_x4_base(phase);
  const int quad = 2 * yyg::gemm_f64_variant_count() + yyg::phi_direct_variant_count();
  const int lean = quad + yyg::phi_quad_variant_count();
  const int r = phase == 4 && v >= sep_stream_base(4) ? yyg::phi_stream_kernel_name(v - sep_stream_base(4), name, n)
                : phase == 0 && v >= sep_xcol_base(0) ? yyg::fold_xcol_kernel_name(v - sep_xcol_base(0), name, n)
                : phase == 0 && v >= sep_stream_base(0)
                    ? yyg::phi_ana_stream_kernel_name(v - sep_stream_base(0), name, n)
                : v >= x0                    ? yyg::x4_kernel_name(v - x0, phase, g->sep.fold, name, n)
                : phase == 4 && v >= lean    ? yyg::phi_lean_kernel_name(v - lean, name, n)
                : sep_theta_variant(g, phase, v) >= 0
                    ? yyg::theta_stream_kernel_name(phase, sep_theta_variant(g, phase, v), g->sep.theta, name, n)
                : !sep_fold_variant(phase, v) ? yyg::sep_kernel_name(phase, v, g->sep.fold, name, n)
                                             : yyg::phi_quad_kernel_name(v - quad, phase == 0,
                                                                         phase == 0 ? g->sep.quad_ana : g->sep.quad_syn,
                                                                         name, n);
  return r == 0 ? YYG_OK : YYG_ERR_INVALID_ARG;
}

int yyg_sep_lp_config(yyg_grid *g, int precision, int phase, int tile) {
  if (!g || (phase != 0 && phase != 4)) return YYG_ERR_INVALID_ARG;
  if (precision != YYG_FP32 && precision != YYG_BF16X3) return YYG_ERR_INVALID_ARG;
  if (!g->sep.ready) return YYG_ERR_NOT_READY;
  const int side = phase == 0 ? 0 : 1;
  if (tile < 0 || tile >= yyg::sep_lp_tile_count() +
                              std::max(yyg::phi_stream32_variant_count(), yyg::phi_ana_stream32_variant_count()))
    return YYG_ERR_INVALID_ARG;
  if (!sep_lp_available(g, precision, side, tile)) return YYG_ERR_UNSUPPORTED;
  g->sep.lpt[precision - 1][side] = tile;
  return YYG_OK;
}

int yyg_sep_lp_kernel(const yyg_grid *g, int precision, int phase, char *name, size_t n) {
  if (!g || !name || n < 1 || (phase != 0 && phase != 4)) return YYG_ERR_INVALID_ARG;
  if (precision != YYG_FP32 && precision != YYG_BF16X3) return YYG_ERR_INVALID_ARG;
  if (!g->sep.ready) return YYG_ERR_NOT_READY;
  const int t = g->sep.lpt[precision - 1][phase == 0 ? 0 : 1], u = t - yyg::sep_lp_tile_count();
  const int r = u < 0        ? yyg::sep_lp_kernel_name(precision, t, phase, g->sep.fold, name, n)
                : phase == 4 ? yyg::phi_stream32_kernel_name(u, name, n)
                             : yyg::phi_ana_stream32_kernel_name(u, name, n);
  return r == 0 ? YYG_OK : YYG_ERR_INVALID_ARG;
}

int yyg_batch_create(yyg_grid *const *grids, int n, int precision, yyg_batch **out) {
  if (!out) return YYG_ERR_INVALID_ARG;
  *out = nullptr;
  if (!grids || n < 1 || precision < 0 || precision > YYG_FP16X2) return YYG_ERR_INVALID_ARG;
  // the separable form when every plan is in it (FP64), the dense form otherwise
  bool sep = precision == YYG_FP64;
  for (int f = 0; f < n; ++f) {
    if (!grids[f] || grids[f]->device != grids[0]->device) return YYG_ERR_INVALID_ARG;
    sep = sep && grids[f]->method == YYG_METHOD_SEPARABLE && grids[f]->sep.ready;
  }
  for (int f = 0; f < n; ++f) {
    if (!sep && grids[f]->n_r > 1024) return YYG_ERR_UNSUPPORTED;
    if (precision != YYG_FP64 && !grids[f]->lp[precision - 1].ready) return YYG_ERR_NOT_READY;
  }
  yyg_batch *b = new (std::nothrow) yyg_batch;
  if (!b) return YYG_ERR_OUT_OF_MEMORY;
  b->device = grids[0]->device;
  b->precision = precision;
  b->sep = sep;
  b->grids.assign(grids, grids + n);
  DeviceGuard dg(b->device);
  if (!dg.ok) {
    delete b;
    return YYG_ERR_DEVICE;
  }
  int st = sep ? sep_batch_build(b) : batch_build(b);
  if (st != YYG_OK) {
    batch_free(b);
    return st;
  }
  *out = b;
  return YYG_OK;
}

int yyg_batch_autotune(yyg_batch *b, void *stream) {
  if (!b) return YYG_ERR_INVALID_ARG;
  // the timed launches read the densities and write the potentials of the
  // last batched solve
  if (!b->launched) return YYG_ERR_NOT_READY;
  DeviceGuard dg(b->device);
  if (!dg.ok) return YYG_ERR_DEVICE;
  hipStream_t s = as_stream(stream);
  if (hipStreamSynchronize(b->stream) != hipSuccess || hipStreamSynchronize(s) != hipSuccess) {
    (void)hipGetLastError();
    return YYG_ERR_DEVICE;
  }
  if (b->sep) {
    // each phase in turn, the others at their current tile: whole eager
    // batched solves, the fastest of three per tile
    for (int r = 0; r < 5; ++r) {
      if (r == 2 && b->n_sitems[2] == 0) continue;  // no two-patch plan: nothing to rotate
      int best = b->svar[r];
      double bt = 1e30;
      for (int t = 0; t <= yyg::sep_batch_tile_count(); ++t) {
        if (!sep_batch_available(b, r, t)) continue;
        int st = sep_batch_set_items(b, r, t);
        if (st != YYG_OK) return st;
        const double tm = time_launch([&] { return sep_batch_enqueue(b, s, nullptr); }, s, 3);
        if (tm < bt) {
          bt = tm;
          best = t;
        }
      }
      int st = sep_batch_set_items(b, r, best);
      if (st != YYG_OK) return st;
    }
    batch_drop_graph(b);
    return YYG_OK;
  }
  const bool lp = b->precision != YYG_FP64;
  const int nv = lp ? yyg::gemm_lp_variant_count() : yyg::gemm_f64_variant_count();
  // time each phase's contraction per tile variant on the batch's own
  // problems (density pointers of the last solve, or whatever the plans
  // hold: timings do not depend on the values)
  int best[2] = {b->var[0], b->var[1]};
  for (int role = 0; role < 2; ++role) {
    double bt = 1e30;
    for (int v = 0; v < nv; ++v) {
      int st = batch_set_items(b, role, v);
      if (st != YYG_OK) return st;
      double t = time_launch([&] { return batch_launch_gemm(b, role, s); }, s, 3);
      if (t < bt) {
        bt = t;
        best[role] = v;
      }
    }
  }
  for (int role = 0; role < 2; ++role) {
    int st = batch_set_items(b, role, best[role]);
    if (st != YYG_OK) return st;
  }
  batch_drop_graph(b);
  return YYG_OK;
}

int yyg_batch_info(const yyg_batch *b, int *info, int n) {
  if (!b || !info || n < 1) return YYG_ERR_INVALID_ARG;
  if (b->sep) {
    const int vals[9] = {(int)b->grids.size(), b->precision, b->svar[0], b->svar[4], b->n_sitems[0], b->n_sitems[4],
                         b->svar[1], b->svar[2], b->svar[3]};
    for (int i = 0; i < n && i < 9; ++i) info[i] = vals[i];
    return YYG_OK;
  }
  const int vals[9] = {(int)b->grids.size(), b->precision, b->var[0], b->var[1], b->n_items[0], b->n_items[1],
                       -1, -1, -1};
  for (int i = 0; i < n && i < 9; ++i) info[i] = vals[i];
  return YYG_OK;
}

int yyg_batch_solve(yyg_batch *b, const double *const *d_rho, double *const *d_phi, void *stream) {
  if (!b || !d_rho || !d_phi) return YYG_ERR_INVALID_ARG;
  const int n = (int)b->grids.size();
  for (int f = 0; f < n; ++f)
    if (!d_rho[f] || !d_phi[f]) return YYG_ERR_INVALID_ARG;
  // a plan's work buffer moved (autotune / plan_config after the batch was
  // built): the recorded arguments are stale
  for (int f = 0; f < n; ++f)
    if (b->grids[f]->part_gen != b->part_gen[f]) return YYG_ERR_NOT_READY;
  DeviceGuard dg(b->device);
  if (!dg.ok) return YYG_ERR_DEVICE;
  // a graph cannot be recorded on the legacy default stream: use the
  // batch's own blocking stream, which that stream orders against
  hipStream_t s = stream ? as_stream(stream) : b->stream;
  for (int f = 0; f < n; ++f)
    if (int st = check_rho(b->grids[f], d_rho[f], s); st != YYG_OK) return st;
  for (int f = 0; f < n; ++f) b->grids[f]->ahat_fold = false;
  for (int f = 0; f < n; ++f) b->grids[f]->ahat_cols = b->sep;  // the moments' layout the batch leaves
  bool changed = false;
  for (int f = 0; f < n; ++f)
    if (b->rho[f] != d_rho[f] || b->phi[f] != d_phi[f]) changed = true;
  if (changed) {
    // the previous launch may still read the staged arguments
    if (b->launched && hipEventSynchronize(b->done) != hipSuccess) {
      (void)hipGetLastError();
      return YYG_ERR_DEVICE;
    }
    for (int f = 0; f < n; ++f) {
      b->rho[f] = d_rho[f];
      b->phi[f] = d_phi[f];
    }
    batch_patch_pointers(b);
  }
  hipError_t e = hipSuccess;
  if (!b->exec || b->exec_stream != s) {
    batch_drop_graph(b);
    // record the whole batched solve once, replay it afterwards
    e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
      hipError_t e2 = batch_enqueue(b, s);
      hipGraph_t graph = nullptr;
      e = hipStreamEndCapture(s, &graph);
      if (e == hipSuccess) e = e2;
      if (e == hipSuccess) e = hipGraphInstantiate(&b->exec, graph, nullptr, nullptr, 0);
      if (graph) (void)hipGraphDestroy(graph);
      if (e == hipSuccess) b->exec_stream = s;
    }
    if (e != hipSuccess) {
      (void)hipGetLastError();
      batch_drop_graph(b);
      return YYG_ERR_DEVICE;
    }
  }
  e = hipGraphLaunch(b->exec, s);
  if (e == hipSuccess) e = hipEventRecord(b->done, s);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return YYG_ERR_DEVICE;
  }
  b->launched = true;
  return YYG_OK;
}

int yyg_batch_profile(yyg_batch *b, void *stream, double *ms, int n) {
  if (!b || !ms || n < 1) return YYG_ERR_INVALID_ARG;
  if (!b->launched) return YYG_ERR_NOT_READY;
  DeviceGuard dg(b->device);
  if (!dg.ok) return YYG_ERR_DEVICE;
  hipStream_t s = stream ? as_stream(stream) : b->stream;
  hipEvent_t ev[6];
  for (auto &x : ev)
    if (hipEventCreate(&x) != hipSuccess) return YYG_ERR_DEVICE;
  if (b->sep) {
    // phases 0-2 (phi and theta analysis, rotation), the scans, phases 3-4
    hipError_t e = hipStreamSynchronize(s);
    if (e == hipSuccess) e = sep_batch_enqueue(b, s, ev);
    if (e == hipSuccess) e = hipEventSynchronize(ev[5]);
    float t[5] = {0, 0, 0, 0, 0};
    for (int i = 0; i < 5 && e == hipSuccess; ++i) e = hipEventElapsedTime(&t[i], ev[i], ev[i + 1]);
    for (auto &x : ev) (void)hipEventDestroy(x);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return YYG_ERR_DEVICE;
    }
    const double vals[4] = {(double)t[0] + t[1], t[2], (double)t[3] + t[4], 0.0};
    for (int i = 0; i < n && i < 4; ++i) ms[i] = vals[i];
    return YYG_OK;
  }
  const int nf = (int)b->grids.size();
  const bool lp = b->precision != YYG_FP64;
  hipError_t e = hipStreamSynchronize(s);
  // the same launches as the recorded graph, eagerly, with events between
  if (e == hipSuccess) {
    if (!lp) {
      e = hipMemcpyAsync(b->d_f64[0], b->h_f64[0], nf * sizeof(yyg::GemmF64Args), hipMemcpyHostToDevice, s);
      if (e == hipSuccess)
        e = hipMemcpyAsync(b->d_f64[1], b->h_f64[1], nf * sizeof(yyg::GemmF64Args), hipMemcpyHostToDevice, s);
    } else {
      e = hipMemcpyAsync(b->d_split[0], b->h_split[0], nf * sizeof(yyg::SplitArgs), hipMemcpyHostToDevice, s);
      if (e == hipSuccess)
        e = hipMemcpyAsync(b->d_lp[1], b->h_lp[1], nf * sizeof(yyg::GemmLpArgs), hipMemcpyHostToDevice, s);
    }
  }
  if (e == hipSuccess) e = hipEventRecord(ev[0], s);
  if (e == hipSuccess && lp)
    e = yyg::launch_split_rows_grouped(b->precision, b->d_split[0], b->d_split_items[0], b->n_split_items[0],
                                       std::min(b->n_split_items[0], b->cus * 8), s);
  if (e == hipSuccess) e = hipEventRecord(ev[1], s);
  if (e == hipSuccess) e = batch_launch_gemm(b, 0, s);
  if (e == hipSuccess) e = hipEventRecord(ev[2], s);
  if (e == hipSuccess)
    e = yyg::launch_radial_scan_grouped(b->d_scan, b->d_scan_items, b->n_scan_items,
                                        std::min(b->n_scan_items, b->cus * 2), s);
  if (e == hipSuccess) e = hipEventRecord(ev[3], s);
  if (e == hipSuccess && lp)
    e = yyg::launch_split_rows_grouped(b->precision, b->d_split[1], b->d_split_items[1], b->n_split_items[1],
                                       std::min(b->n_split_items[1], b->cus * 8), s);
  if (e == hipSuccess) e = hipEventRecord(ev[4], s);
  if (e == hipSuccess) e = batch_launch_gemm(b, 1, s);
  if (e == hipSuccess) e = hipEventRecord(ev[5], s);
  if (e == hipSuccess) e = hipEventSynchronize(ev[5]);
  float t[5] = {0, 0, 0, 0, 0};
  for (int i = 0; i < 5 && e == hipSuccess; ++i) e = hipEventElapsedTime(&t[i], ev[i], ev[i + 1]);
  for (auto &x : ev) (void)hipEventDestroy(x);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return YYG_ERR_DEVICE;
  }
  // slots as for plans: 0 analysis, 1 scan, 2 synthesis, 3 operand splits
  const double vals[4] = {t[1], t[2], t[4], (double)t[0] + t[3]};
  for (int i = 0; i < n && i < 4; ++i) ms[i] = vals[i];
  return YYG_OK;
}

int yyg_batch_destroy(yyg_batch *b) {
  if (!b) return YYG_ERR_INVALID_ARG;
  DeviceGuard dg(b->device);
  (void)hipDeviceSynchronize();
  batch_free(b);
  return YYG_OK;
}

}  // extern "C"
