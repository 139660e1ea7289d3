// gap.hip -- host side of libgap: parameter derivation, device state, the
// step sequence, re-sorting of the particle stores, diagnostics and the C ABI
// declared in include/gap.h.
#include "gap.h"
#include "gap_kernels.hpp"
#include "gap_merge.hpp"
#include "gap_adjoint.hpp"
#include "gap_diag.hpp"
#include "gap_qtab.hpp"
#include "gap_protons.hpp"
#include "gap_fused.hpp"
#include "gap_records.hpp"

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

using namespace gap;

namespace {

// ---------------------------------------------------------------- constants
// CGS values (CODATA); the unit system follows Sect. 2.2 of the paper:
// omega_p,co^2 = Omega omega_B, d = c / omega_p,co.
constexpr double kC = 2.99792458e10;
constexpr double kEoverMC = 1.75882001076e7;
constexpr double kLambdaC = 3.8615926796e-11;
constexpr double kBQ = 4.41400e13;
constexpr double kAlphaEM = 1.0 / 137.035999084;
constexpr double kPi = 3.14159265358979323846;
constexpr double kTwo24 = 16777216.0;

constexpr int kGrid = 2048;        // workgroups of the particle passes (multiple of 8)
constexpr int kDiagGrid = 1024;    // workgroups of the diagnostics' passes (multiple of 8)

// ---------------------------------------------------------------- spectrum table
// Cumulative classical synchrotron photon-number spectrum C(xi) =
// (3/(5 pi)) int_0^xi dxi' int_xi'^inf K_{5/3}.  From the integral
// representation of K_nu, 1 - C(xi) = (3/(5 pi)) int_0^inf exp(-xi cosh s)
// cosh(5s/3) / cosh^2 s ds, evaluated here with Simpson's rule.
struct SyncQuad {
  std::vector<double> wg, ch;
  SyncQuad() {
    const double h = 1.0 / 32.0;
    const int n = 48 * 32;  // s in [0, 48], n even
    wg.resize(n + 1);
    ch.resize(n + 1);
    for (int i = 0; i <= n; ++i) {
      const double s = i * h;
      const double c = std::cosh(s);
      const double simpson = (i == 0 || i == n) ? 1.0 : (i % 2 ? 4.0 : 2.0);
      ch[i] = c;
      wg[i] = simpson * h / 3.0 * std::cosh(5.0 * s / 3.0) / (c * c) * 3.0 / (5.0 * kPi);
    }
  }
  // tail = 1 - C(xi); dens = -d tail / d xi = dC/dxi
  void eval(double xi, double* tail, double* dens) const {
    double t = 0.0, d = 0.0;
    for (size_t i = 0; i < wg.size(); ++i) {
      const double a = xi * ch[i];
      if (a > 700.0) break;
      const double e = std::exp(-a) * wg[i];
      t += e;
      d += e * ch[i];
    }
    *tail = t;
    *dens = d;
  }
};

// Solve tail(xi) = target (target in (0,1)) for log(xi), Newton with a bracket.
double solve_tail(const SyncQuad& q, double target, bool use_cdf) {
  double lo = -110.0, hi = 6.0;
  double y = use_cdf ? 3.0 * std::log(std::max(1.0 - target, 1e-300) / 1.2316) : std::log(std::max(-std::log(target), 1e-3));
  if (!(y > lo && y < hi)) y = 0.5 * (lo + hi);
  for (int it = 0; it < 300; ++it) {
    double t, d;
    const double xi = std::exp(y);
    q.eval(xi, &t, &d);
    // g(y) = log tail - log target, decreasing in y
    double g, dg;
    if (use_cdf) {           // for small C compare C = 1 - tail directly
      g = (1.0 - target) - (1.0 - t);   // C_target - C(xi): decreasing in y
      dg = -d * xi;
    } else {
      g = std::log(t) - std::log(target);
      dg = -d * xi / t;
    }
    if (g > 0) lo = y; else hi = y;
    double yn = y - g / dg;
    if (!(yn > lo && yn < hi) || !std::isfinite(yn)) yn = 0.5 * (lo + hi);
    if (std::fabs(yn - y) < 1e-13 || hi - lo < 1e-13) return std::exp(yn);
    y = yn;
  }
  return std::exp(y);
}

const std::vector<float>& sync_table() {
  static std::vector<float> tab;
  static std::once_flag once;
  std::call_once(once, [] {
    SyncQuad q;
    tab.assign(2 * (NTAB + 1), 0.0f);
    for (int i = 1; i <= NTAB; ++i) {
      const double r = 0.5 * i / NTAB;                         // C(xi) = r
      tab[i] = (float)std::cbrt(solve_tail(q, 1.0 - r, true));
    }
    for (int i = 0; i <= NTAB; ++i) {
      const double y = TAB_YLO + (double)i * (TAB_YHI - TAB_YLO) / NTAB;   // tail = e^-y
      tab[NTAB + 1 + i] = (float)solve_tail(q, std::exp(-y), false);
    }
  });
  return tab;
}

// host copy of the device sampler (same table, same interpolation)
float sync_sample_host(float r, const float* tab) {
  if (r <= 0.5f) {
    float t = r * (2.0f * NTAB);
    int i = std::min((int)t, NTAB - 1);
    float f = t - (float)i;
    float v = tab[i] + f * (tab[i + 1] - tab[i]);
    return v * v * v;
  }
  float y = -std::log(1.0f - r);
  float t = (y - TAB_YLO) * ((float)NTAB / (TAB_YHI - TAB_YLO));
  t = std::fmin(std::fmax(t, 0.0f), (float)NTAB - 1e-3f);
  int i = (int)t;
  float f = t - (float)i;
  const float* h = tab + NTAB + 1;
  return h[i] + f * (h[i + 1] - h[i]);
}

const qtab::Tables& quantum_tables() {
  return qtab::tables(QS_COLS, QS_ROW, QS_NR, QS_CHI_LO, QS_PER_DEC, QS_ALO, QS_AHI, QS_YLO, QS_YHI, QB_COLS, QB_NR,
                      QB_CHI_LO, QB_PER_DEC);
}

// ---------------------------------------------------------------- static workspace
// Workspace of the allocation-free spectrum entry point: the two ping-pong
// buffers of the largest FFT it accepts (2^18 points, 8 MiB per device, held
// until the process ends).  In host code the name below is not a device
// address: the address on each device comes from hipGetSymbolAddress, taken
// once per device (scratch_on_device) and kept.
constexpr int kScratchMaxM = 1 << 18;
static __device__ __align__(256) double2 scratch[2 * kScratchMaxM];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double2* g_scratch_dev[kMaxDevices] = {};

// Address of `scratch` on the current device `dev` (nullptr if it cannot be had).
double2* scratch_on_device(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
    g_scratch_dev[dev] = (double2*)p;
  }
  return g_scratch_dev[dev];
}

// ---------------------------------------------------------------- state
struct Store {
  Ctl* ctl = nullptr;
  int cur = 0;
  uint32_t* pos[2] = {nullptr, nullptr};
  float* a[2] = {nullptr, nullptr};      // u (leptons) or x (photons)
  float* w[2] = {nullptr, nullptr};
  int32_t* n0[2] = {nullptr, nullptr};   // photons only
  uint64_t* id[2] = {nullptr, nullptr};
  int32_t* tt = nullptr;
  int32_t* chunk[2] = {nullptr, nullptr};
  int32_t* tcount = nullptr;
  int nclass = 1;                 // placement classes within a tile at a re-sort
  int32_t* ccount = nullptr;      // [nclass - 1][n_tiles]: particles of the leading classes per tile
  int32_t* ccur = nullptr;        // [nclass][n_tiles]: placement cursors
  int32_t* wh = nullptr;          // [kGrid][window][nclass]: window counts of the re-sort's count workgroups
  uint8_t* cls = nullptr;         // class of each slot, decided by the count kernel
  uint16_t* chot = nullptr;       // photons: hot slots at the start of each sorted chunk
  long long* tchunk = nullptr;
  int64_t capacity = 0, limit = 0, cap_live = 0;
  LepBuf lep(int b) const { return LepBuf{pos[b], a[b], w[b], id[b]}; }
  PhoBuf pho(int b) const { return PhoBuf{pos[b], a[b], w[b], n0[b], id[b]}; }
};

struct Derived { double d_cm, lam, rc, dt, H, w0, s_co; int N; };

// Saved state at the start of a window segment (stores re-sorted, tail empty).
struct WinCkpt {
  long long nl = 0, np = 0, nch_l = 0, nch_p = 0;
  uint32_t* lpos = nullptr; float* lu = nullptr; float* lw = nullptr; uint64_t* lid = nullptr; int32_t* lchunk = nullptr;
  uint32_t* ppos = nullptr; float* px = nullptr; float* pw = nullptr; int32_t* pn0 = nullptr; uint64_t* pid = nullptr;
  int32_t* pchunk = nullptr;
  Ctl lctl{}, pctl{};
  Tube* tubes = nullptr;
  float* ebar = nullptr;
  float* E = nullptr;
  long long* shard = nullptr;
  int64_t host_step = 0;
};

// A window of steps run by gap_window_forward, kept for gap_backward.
struct WinState {
  bool valid = false;
  int64_t W = 0, K = 0, nseg = 0, step_end = 0;
  long long max_used = 0;
  std::vector<WinCkpt> ck;
  std::vector<void*> mem;       // allocations of this window
  double* loss_acc = nullptr;
  // reverse-pass buffers
  long long M = 0;              // tape stride (slots)
  uint32_t* tpos = nullptr; float* tu = nullptr; TapeMeta* meta = nullptr;
  float* teb = nullptr; float* tE = nullptr; float* wlast = nullptr;
  float* lam[2][3] = {{nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr}};
  double* lamE = nullptr; double* suf = nullptr; double* lamEb[2] = {nullptr, nullptr};
  unsigned long long* frec = nullptr;   // records of the reverse field scan
  AdjTube* at = nullptr;
  uint32_t* hvals = nullptr; uint64_t hmask = 0;
};

}  // namespace

struct gap_t {
  int n_tubes = 0;
  hipStream_t s = nullptr;
  // second stream: the photon side of each step (prologue, sorted photon
  // pass, pairs) runs on it beside the lepton side.  ev_l: the
  // caller's stream up to the start of a step; ev_pre: the prologue done;
  // ev_p: the photon side of the last enqueued step done.
  hipStream_t s2 = nullptr;
  hipEvent_t ev_l = nullptr, ev_pre = nullptr, ev_p = nullptr;
  hipEvent_t ev_f = nullptr, ev_j = nullptr;   // fork and join of the two stores' re-sort or merge
  bool ev_l_bound = false;   // ev_l is already the completion of the last field kernel on the caller's stream
  bool s2_pending = false;  // photon-side work not yet joined into the caller's stream
  bool capturing = false;   // graph capture: everything stays on the caller's stream
  gap_allocator al{};
  bool custom_alloc = false;
  std::vector<void*> owned;
  std::vector<gap_params> P;
  std::vector<Derived> D;
  std::vector<Tube> th;
  std::vector<Tile> tiles_h;
  std::vector<LTile> ltiles_h;
  std::vector<PTile> ptiles_h;
  std::vector<FBlk> fb_h;
  Tube* tubes = nullptr;
  Tile* tiles = nullptr;
  LTile* ltiles = nullptr;
  PTile* ptiles = nullptr;
  int n_tiles = 0;
  long long total_nodes = 0, total_cells = 0;
  int max_cells = 1;   // largest tube
  long long* rho = nullptr;
  long long* rho_last = nullptr;
  float* E = nullptr;
  float* ebar = nullptr;
  FBlk* fb = nullptr;
  int n_fb = 0;
  long long* part = nullptr;
  long long* part2 = nullptr;
  unsigned long long* fscan = nullptr;   // single-pass field: 4 words per block, then an epoch per tube
  // device words the host reads back at every synchronising call: the sticky
  // error bits, and each store's chunk count + 1 as its last re-sort left it
  struct Status { int err, pad; long long chunks[2]; };
  Status* status = nullptr;
  uint32_t* stage = nullptr;       // device staging of the small reads (the conversion queue, which only a step
  size_t stage_bytes = 0;          // uses), its size, and their host side
  std::vector<char> stage_h;
  // what the last such call found (chunks -1: not known), and the re-sorts
  // enqueued since, by steps or within replayed graphs
  int64_t seen_l = -1, seen_p = -1;
  int rb_seen = 0;
  float* tab = nullptr;
  float* qs = nullptr;     // quantum photon-spectrum table (tubes with GAP_QUANTUM)
  float* qb = nullptr;     // quantum pair-split table
  int* err = nullptr;
  long long* live = nullptr;     // live leptons, then photons, per tube
  long long* counts = nullptr;   // one tube's counters, gathered for the host
  long long* shard = nullptr;   // [tube][NSHARD][C_N] event counters
  Store lep, pho;
  // per-kernel event timing (eager steps only), and, for one that the caller
  // asked for, the particle passes in launches of their own whatever the form
  bool timing = false;
  bool apart = false;
  std::vector<hipEvent_t> ev_pool;
  size_t ev_used = 0;
  std::vector<std::pair<int, std::pair<hipEvent_t, hipEvent_t>>> ev_marks;   // (kernel id, start, stop)
  int R = 64;
  int64_t since_rb = 0;
  int64_t host_step = 0;        // steps enqueued (all tubes advance together)
  bool merge_on = false;
  int merge_every = 64;
  SortBuf sort_l{}, sort_p{};
  double* thresh_l = nullptr;
  double* thresh_p = nullptr;
  double tmin_l = 0.0, tmin_p = 0.0;   // smallest tube threshold of each store
  // conversion queue of the sorted photon pass (one entry per photon slot at
  // most), and per workgroup of the pass the entries' number and start
  uint4* pq = nullptr;
  // discharge diagnostics: return spectra [n_tubes][RET_N]; profile sums and
  // results for the largest tube at one cell per bin
  double* ret = nullptr;
  double* ret_thr = nullptr;           // [RET_NB]: lower bin edges in u^2
  double* prof_acc = nullptr;
  double* prof_out = nullptr;
  int prof_bin = 64;                   // cells per profile bin
  // waterfall of E^2 (off while wf_every == 0): ring of records per tube
  int wf_every = 0, wf_B = 64, wf_cap = 0, wf_nbmax = 0;
  double* wf_ring = nullptr;
  long long* wf_steps = nullptr;
  std::vector<void*> wf_mem;
  double* spec_thr = nullptr;   // squares of the momentum-spectrum edges
  double* spec_acc = nullptr;   // [3][SPEC_NB]
  double* phase_acc = nullptr;  // [3][nb][PHASE_NP], allocated on first use
  size_t phase_cap = 0;
  double2* fft_buf = nullptr;   // 2 M complex values of the largest tube, allocated on first use
  double* fft_pow = nullptr;
  int* pq_count = nullptr;
  long long* pq_start = nullptr;
  uint4* bq = nullptr;                 // birth queue of the sorted lepton pass: entries, and per
  int* bq_count = nullptr;             // workgroup of the pass their number and first entry
  long long* bq_start = nullptr;
  int pq_groups = 0;                   // entries of pq_count (bounds the photon grid)
  bool grid_lep_set = false;   // grid_lep was set or tuned
  int grid_lep = 2048, grid_pho = 2048, grid_tail = 1024;   // workgroups of the particle passes
  int round_lep = 2048, round_pho = 2048, cus = 256;        // one resident round of each pass; CUs
  int rmax = 64;                                            // longest re-sort interval the tile margin allows
  bool any_periodic = false;
  bool any_filter = false;
  bool any_quantum = false;
  bool any_protons = false;   // a tube with an atmosphere or the proton initial state
  bool any_atm = false;       // a tube with a thermal atmosphere
  ProBuf pr[2]{};             // protons (double buffer for the compaction at re-sorts)
  int pr_cur = 0;
  long long* pr_n = nullptr;  // device: proton slots in use
  int64_t pr_cap = 0;
  double* E0 = nullptr;   // filtered tubes: reference field; Du: E_u - E0 of the step
  double* Du = nullptr;
  int sticky = 0;
  double2* scratch = nullptr;   // this device's address of the allocation-free spectrum's workspace
  // graph: replay is valid from the recorded start state and leaves the end state
  WinState win;
  hipGraphExec_t gexec = nullptr;
  int64_t gsteps = -1;
  bool graph_fused = false;   // the captured steps take the fused form
  int graph_rb = 0;           // re-sorts among them
  int graph_form = 0;         // their form, as GAP_DIAG_FORM gives it
  int form = 0;               // the last enqueued step's
  int gs_l = -1, gs_p = -1, ge_l = -1, ge_p = -1, gs_r = -1, ge_r = -1;
  int64_t gs_since = -1, ge_since = -1, gs_step = -1;
};

namespace {

int from_hip(hipError_t e) { return e == hipSuccess ? GAP_OK : GAP_EDEVICE; }
#define HIPCHK(x) do { hipError_t _e = (x); if (_e != hipSuccess) return GAP_EDEVICE; } while (0)

size_t up256(size_t bytes) { return (bytes + 255) & ~(size_t)255; }

void* dalloc(gap_t* g, size_t bytes) {
  bytes = (bytes + 255) & ~(size_t)255;
  if (bytes == 0) bytes = 256;
  g->owned.push_back(nullptr);   // (its place first: no block is lost to a failed host allocation)
  void* p = nullptr;
  if (g->custom_alloc) p = g->al.alloc(bytes, g->al.ctx);
  else if (hipMalloc(&p, bytes) != hipSuccess) p = nullptr;
  if (p) {
    g->owned.back() = p;
    (void)hipMemsetAsync(p, 0, bytes, g->s);
  } else {
    g->owned.pop_back();
  }
  return p;
}

// The quantum samplers of the particle passes on given (chi, Philox word)
// pairs: kind 0 the photon energy fraction, kind 1 the pair's electron
// fraction.
__global__ void k_qed_sample(int kind, const float* chi, const uint32_t* w, int64_t n, const float* qs,
                             const float* qb, float* out) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = kind == 0 ? qsyn_fraction(chi[i], w[i], qs) : qbw_fraction(chi[i], w[i], qb);
}

// Device copies of the quantum tables (built once per process on the host).
int upload_quantum_tables(gap_t* g) {
  if (g->qs) return GAP_OK;
  const qtab::Tables& t = quantum_tables();
  g->qs = (float*)dalloc(g, sizeof(float) * t.syn.size());
  g->qb = (float*)dalloc(g, sizeof(float) * t.bw.size());
  if (!g->qs || !g->qb) return GAP_ENOMEM;
  HIPCHK(hipMemcpyAsync(g->qs, t.syn.data(), sizeof(float) * t.syn.size(), hipMemcpyHostToDevice, g->s));
  HIPCHK(hipMemcpyAsync(g->qb, t.bw.data(), sizeof(float) * t.bw.size(), hipMemcpyHostToDevice, g->s));
  HIPCHK(hipStreamSynchronize(g->s));
  return GAP_OK;
}

// Returns one allocation of dalloc (the caller has waited for work using it).
void dfree(gap_t* g, void* p) {
  if (!p) return;
  auto it = std::find(g->owned.begin(), g->owned.end(), p);
  if (it == g->owned.end()) return;
  g->owned.erase(it);
  if (g->custom_alloc) g->al.free(p, g->al.ctx);
  else (void)hipFree(p);
}

void win_release(gap_t* g);

// Frees the waterfall ring (the caller has waited for queued work).
void wf_release(gap_t* g) {
  for (void* p : g->wf_mem) {
    if (g->custom_alloc) g->al.free(p, g->al.ctx);
    else (void)hipFree(p);
  }
  g->wf_mem.clear();
  g->wf_ring = nullptr;
  g->wf_steps = nullptr;
  g->wf_every = 0;
  g->wf_cap = 0;
}

// A graph exec may only be destroyed once no launch of it is in flight: wait
// for both streams of the handle first.
void drop_graph(gap_t* g) {
  if (!g->gexec) return;
  if (g->s2) (void)hipStreamSynchronize(g->s2);
  (void)hipStreamSynchronize(g->s);
  (void)hipGraphExecDestroy(g->gexec);
  g->gexec = nullptr;
  g->gsteps = -1;
}

void release(gap_t* g) {
  drop_graph(g);
  (void)hipStreamSynchronize(g->s);   // (also the default stream: an allocator may reuse a block at once)
  if (g->s2) { (void)hipStreamSynchronize(g->s2); (void)hipStreamDestroy(g->s2); g->s2 = nullptr; }
  for (hipEvent_t* e : {&g->ev_l, &g->ev_pre, &g->ev_p, &g->ev_f, &g->ev_j})
    if (*e) { (void)hipEventDestroy(*e); *e = nullptr; }
  win_release(g);
  wf_release(g);
  for (hipEvent_t e : g->ev_pool) (void)hipEventDestroy(e);
  g->ev_pool.clear();
  for (void* p : g->owned) {
    if (g->custom_alloc) g->al.free(p, g->al.ctx);
    else (void)hipFree(p);
  }
  g->owned.clear();
}

int validate(const gap_params& p) {
  if (p.n_cells < 2 || p.n_cells > (1 << 26)) return GAP_EINVAL;
  if ((p.flags & GAP_FILTER) && p.n_cells < 2 * FLT_PASSES) return GAP_EINVAL;
  if (!(p.dx > 0) || !(p.cfl > 0 && p.cfl < 1.0)) return GAP_EINVAL;
  if (p.ppc_ref < 1 || p.ppc_init < 0) return GAP_EINVAL;
  if (!(p.b > 0) || !(p.r_curv_cm > 0) || !(p.period_s > 0)) return GAP_EINVAL;
  if (!(p.lambda_c_scale > 0) || !(p.r_curv_scale > 0)) return GAP_EINVAL;
  if (!(p.h_gap_frac >= 0)) return GAP_EINVAL;
  if (p.init_kind < 0 || p.init_kind > GAP_INIT_ATMOSPHERE) return GAP_EINVAL;
  if (p.atm_ppc < 0 || p.atm_ppc > (1 << 20)) return GAP_EINVAL;
  if (p.atm_ppc > 0 && (!(p.atm_temp > 0) || !std::isfinite(p.atm_temp))) return GAP_EINVAL;
  if ((p.atm_ppc > 0 || p.init_kind == GAP_INIT_ATMOSPHERE) && (p.flags & GAP_PERIODIC)) return GAP_EINVAL;
  if (!(p.inj_rate >= 0) || !(p.inj_weight > 0) || p.inj_weight >= 65536.0) return GAP_EINVAL;
  if (p.cap_leptons < 1 || p.cap_photons < 1) return GAP_EINVAL;
  if (p.nsub_max < 1 || p.nsub_max > 64) return GAP_EINVAL;
  if (p.rebucket_every < 0) return GAP_EINVAL;
  if (!(p.merge_frac > 0)) return GAP_EINVAL;
  return GAP_OK;
}

Derived derive(const gap_params& p) {
  Derived d{};
  const double omega = 2.0 * kPi / p.period_s;
  const double omega_b = kEoverMC * p.b * kBQ;
  d.d_cm = kC / std::sqrt(omega * omega_b);
  d.lam = kLambdaC / d.d_cm * p.lambda_c_scale;
  d.rc = p.r_curv_cm / d.d_cm * p.r_curv_scale;
  d.dt = p.cfl * p.dx;
  d.H = p.h_gap_frac * p.n_cells * p.dx;
  d.w0 = p.dx / p.ppc_ref;
  d.s_co = (p.flags & GAP_ANTI_ALIGNED) ? 1.0 : -1.0;
  d.N = p.n_cells;
  return d;
}

int64_t init_k_lo(const gap_params& p, const Derived& d) {
  if (p.init_kind == GAP_INIT_GAP) return (int64_t)std::ceil(d.H / p.dx - 1e-9);
  return 0;
}

int64_t init_count(const gap_params& p, const Derived& d) {
  const int64_t ncell = std::max<int64_t>(0, p.n_cells - init_k_lo(p, d));
  switch (p.init_kind) {
    case GAP_INIT_GAP: return ncell * p.ppc_init;
    case GAP_INIT_UNIFORM: return 2 * ncell * p.ppc_init;
    case GAP_INIT_ELECTRON: return ncell * p.ppc_init;
    case GAP_INIT_ATMOSPHERE: return ncell * p.ppc_init;
    default: return 0;
  }
}

// Initial protons of a tube (proton initial state): ppc_init per cell below H.
int64_t init_protons(const gap_params& p, const Derived& d) {
  if (p.init_kind != GAP_INIT_ATMOSPHERE) return 0;
  const int64_t k_h = std::min<int64_t>(p.n_cells, (int64_t)std::ceil(d.H / p.dx - 1e-9));
  return std::max<int64_t>(0, k_h) * p.ppc_init;
}

// The atmosphere's counts of the previous push: as if it had left the
// reservoir full (no refill before the next push); the other parity clear.
void atm_reset(Tube& T) {
  const int prev = (int)((T.step - 1) & 1);
  for (int sp = 0; sp < 2; ++sp) {
    T.atm_cnt[2 * sp + prev] = T.atm_ppc;
    T.atm_cnt[2 * sp + (prev ^ 1)] = 0;
  }
}

// Workgroups of the sorted lepton pass: those set or tuned, else one resident
// round, or two for a store of at least eight chunks per workgroup of it, as
// last seen (a pass is then long enough that a second, later-starting round
// evens out its end.  A step with two rounds and with one: 26 chunks per
// workgroup, 64 tubes, 221 and 228 us; 13, 108 and 111; 10, 82.0 and 83.3; 6,
// 62.9 and 61.4; the production gap at 5.5, 99.1 and 97.9).
int lepton_grid(const gap_t* g) {
  return g->grid_lep_set || g->seen_l < 8LL * g->round_lep ? g->grid_lep : 2 * g->round_lep;
}

Ctx make_ctx(gap_t* g) {
  Ctx c;
  c.tubes = g->tubes;
  c.tiles = g->tiles;
  c.ltiles = g->ltiles;
  c.ptiles = g->ptiles;
  c.L = g->lep.lep(g->lep.cur);
  c.lc = g->lep.ctl;
  c.lchunk = g->lep.chunk[g->lep.cur];
  c.ltt = g->lep.tt;
  c.P = g->pho.pho(g->pho.cur);
  c.pc = g->pho.ctl;
  c.pchunk = g->pho.chunk[g->pho.cur];
  c.pchot = g->pho.chot;
  c.ptt = g->pho.tt;
  c.rho = g->rho;
  c.ebar = g->ebar;
  c.tab = g->tab;
  c.qs = g->qs;
  c.qb = g->qb;
  c.R = g->pr[g->pr_cur];
  c.pr_n = g->pr_n;
  c.pr_cap = g->pr_cap;
  c.err = g->err;
  c.shard = g->shard;
  c.pq = g->pq;
  c.pq_count = g->pq_count;
  c.pq_start = g->pq_start;
  c.pq_groups = g->grid_pho;
  c.bq = g->bq;
  c.bq_count = g->bq_count;
  c.bq_start = g->bq_start;
  c.bq_groups = lepton_grid(g);
  c.ret = g->ret;
  c.ret_thr = g->ret_thr;
  return c;
}

hipEvent_t next_event(gap_t* g) {
  if (g->ev_used == g->ev_pool.size()) {
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    g->ev_pool.push_back(e);
  }
  return g->ev_pool[g->ev_used++];
}

// kernel ids of the timing diagnostic
enum { KT_LEPTONS = 0, KT_PHOTONS = 1, KT_FIELD = 2, KT_RESORT = 3, KT_PRE = 4, KT_TAILS = 5, KT_MERGE = 6,
       KT_CONV = 7, KT_N = 8 };

struct Timer {
  gap_t* g; int id; hipStream_t st; hipEvent_t a = nullptr, b = nullptr;
  Timer(gap_t* gg, int i, hipStream_t stream) : g(gg), id(i), st(stream) {
    // eager steps only: an event recorded into a captured graph is not a
    // timestamp the host can read
    if (g->timing && !g->capturing && g->ev_pool.size() < 200000) {
      a = next_event(g); b = next_event(g);
      if (a) (void)hipEventRecord(a, st);
    }
  }
  Timer(gap_t* gg, int i) : Timer(gg, i, gg->s) {}
  ~Timer() {
    if (a && b) { (void)hipEventRecord(b, st); g->ev_marks.push_back({id, {a, b}}); }
  }
};

FieldCtx make_fctx(gap_t* g, int mode) {
  FieldCtx f;
  f.tubes = g->tubes;
  f.fb = g->fb;
  f.rho = g->rho;
  f.rho_last = g->rho_last;
  f.E = g->E;
  f.ebar = g->ebar;
  f.part = g->part;
  f.part2 = g->part2;
  f.err = g->err;
  f.pc = g->pho.ctl;
  f.loss = nullptr;
  f.fs = g->fscan;
  f.E0 = g->E0;
  f.Du = g->Du;
  f.mode = mode;
  return f;
}

__global__ void k_cold_off(Ctl* c) { c->cold_steps = -1; }
// A tube's counters as GAP_DIAG_COUNTS gives them: its own and its shards', live
// particles and steps (the error code is the host's).  One wave.
__global__ void k_counts(const Tube* tubes, int tube, int n_tubes, const long long* shard, const long long* live,
                         long long* out) {
  __shared__ long long s_o[C_N];
  const int i = (int)threadIdx.x;
  if (i < C_N) {
    long long v = tubes[tube].cnt[i];
    for (int k = 0; k < NSHARD; ++k) v += shard[((long long)tube * NSHARD + k) * C_N + i];
    s_o[i] = v;
  }
  __syncthreads();
  if (i >= C_N) return;
  long long v = s_o[i];
  // totals include the tail passes (the *_TAIL slots hold that part)
  if (i == C_LEP_STEPS) v += s_o[C_LEP_STEPS_TAIL];
  if (i == C_EMIT_EVAL) v += s_o[C_EMIT_EVAL_TAIL];
  if (i == C_PHO_STEPS) v += s_o[C_PHO_STEPS_TAIL];
  if (i == C_CONV_EVAL) v += s_o[C_CONV_EVAL_TAIL];
  if (i == C_LEPTONS) v = live[tube];
  if (i == C_PHOTONS) v = live[n_tubes + tube];
  if (i == C_STEP) v = tubes[tube].step;
  out[i] = v;
}
__global__ void k_raise(int* err, int bits) { atomicOr(err, bits); }

__global__ void k_fill_i32(int32_t* p, long long n, int32_t v) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) p[i] = v;
}
__global__ void k_fill_i64(long long* p, long long n, long long v) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) p[i] = v;
}

template <class B>
void rebucket_t(gap_t* g, Store& st, B src, B dst, hipStream_t s) {
  RbCtx<B> cx;
  cx.tubes = g->tubes;
  cx.tiles = g->tiles;
  cx.src = src;
  cx.dst = dst;
  cx.ctl = st.ctl;
  cx.chunk_old = st.chunk[st.cur];
  cx.chunk_new = st.chunk[st.cur ^ 1];
  cx.tt = st.tt;
  cx.tcount = st.tcount;
  cx.ccount = st.ccount;
  cx.ccur = st.ccur;
  cx.cls = st.cls;
  cx.chot = st.chot;
  cx.window = g->R;
  cx.tchunk = st.tchunk;
  cx.wh = st.wh;
  cx.chunks_seen = &g->status->chunks[std::is_same<B, PhoBuf>::value ? 1 : 0];
  cx.n_tiles = g->n_tiles;
  // (the tile and class counts were cleared by rebucket_clear)
  k_rb_count<B><<<kGrid, TPB, 0, s>>>(cx);
  k_rb_scan<B><<<1, RB_SCAN_T, 0, s>>>(cx);
  k_rb_chunks<B><<<kGrid, 256, 0, s>>>(cx);
  k_rb_scatter<B><<<kGrid, TPB, 0, s>>>(cx);
  k_rb_pad<B><<<std::max(1, std::min(g->n_tiles, kGrid)), TPB, 0, s>>>(cx);
  k_rb_finish<B><<<1, 1, 0, s>>>(cx);
  st.cur ^= 1;
}

// Clears a store's tile and class counts for its re-sort.  Both stores' are
// cleared on the caller's stream before the photon store's re-sort is forked
// onto the second one: a small kernel issued beside the other store's full
// count grid waited for a free CU for a quarter of a millisecond.
void rebucket_clear(gap_t* g, Store& st) {
  const int fgrid = std::max(1, std::min(1024, (g->n_tiles + 255) / 256));
  k_fill_i32<<<fgrid, 256, 0, g->s>>>(st.tcount, g->n_tiles, 0);
  k_fill_i32<<<fgrid, 256, 0, g->s>>>(st.ccount, (long long)(st.nclass - 1) * g->n_tiles, 0);
}

__global__ void k_count_resort(Tube* tubes, int n_tubes) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n_tubes) tubes[t].cnt[C_REBUCKETS] += 1;
}

void join_photon_side(gap_t* g);

// Work on the two stores side by side: outside graph capture, the photon
// store's part is forked onto the second stream once the caller's stream has
// reached this point, and the caller's stream waits for it at the end.  The
// re-sort and the merge of one store touch only that store and its own
// buffers (the tubes and tiles they read do not change meanwhile).
hipStream_t fork_stores(gap_t* g) {
  join_photon_side(g);
  if (g->capturing) return g->s;
  (void)hipEventRecord(g->ev_f, g->s);
  (void)hipStreamWaitEvent(g->s2, g->ev_f, 0);
  return g->s2;
}
void join_stores(gap_t* g, hipStream_t ps) {
  if (ps == g->s) return;
  (void)hipEventRecord(g->ev_j, ps);
  (void)hipStreamWaitEvent(g->s, g->ev_j, 0);
}

// (the count stops far above the few that matter)
void count_resorts(gap_t* g, int n) { g->rb_seen = std::min(g->rb_seen + n, 1 << 20); }

void rebucket_all(gap_t* g) {
  join_photon_side(g);
  rebucket_clear(g, g->pho);
  rebucket_clear(g, g->lep);
  hipStream_t ps = fork_stores(g);
  rebucket_t<PhoBuf>(g, g->pho, g->pho.pho(g->pho.cur), g->pho.pho(g->pho.cur ^ 1), ps);
  rebucket_t<LepBuf>(g, g->lep, g->lep.lep(g->lep.cur), g->lep.lep(g->lep.cur ^ 1), g->s);
  k_count_resort<<<(g->n_tubes + 255) / 256, 256, 0, g->s>>>(g->tubes, g->n_tubes);
  if (g->any_protons) {
    k_pro_compact<<<1, PRO_COMPACT_THREADS, 0, g->s>>>(g->pr[g->pr_cur], g->pr[g->pr_cur ^ 1], g->pr_n, g->pr_cap);
    g->pr_cur ^= 1;
  }
  join_stores(g, ps);
  count_resorts(g, 1);
}

// With `done`, the single-pass kernel's own completion is recorded into that
// event (no separate marker on the stream); returns whether it was.
bool field_pass(gap_t* g, const FieldCtx& f, hipEvent_t done = nullptr) {
  const bool filt = g->any_filter && f.mode == 0;
  if (filt) done = nullptr;   // the step's field is complete only after k_filter
  bool bound = false;
  if (!g->any_periodic) {
    if (done) hipExtLaunchKernelGGL(k_field_1p, dim3(g->n_fb), dim3(FB_THREADS), 0, g->s, nullptr, done, 0, f);
    else k_field_1p<<<g->n_fb, FB_THREADS, 0, g->s>>>(f);
    bound = done != nullptr;
  } else {
    // a periodic tube subtracts the mean field, which needs the whole tube's
    // sums before any output: two passes
    k_field_a<<<g->n_fb, FB_THREADS, 0, g->s>>>(f);
    k_field_b<<<g->n_fb, FB_THREADS, 0, g->s>>>(f);
  }
  if (filt) k_filter<<<dim3((g->max_cells + FLT_CELLS - 1) / FLT_CELLS, g->n_tubes), FLT_CELLS, 0, g->s>>>(f);
  return bound;
}
// Node charge and field from the current particles and E_s (no drive).
void rebuild_field(gap_t* g) {
  const int grid = std::max(1, (int)std::min<long long>(1024, (g->total_nodes + 255) / 256));
  k_fill_i64<<<grid, 256, 0, g->s>>>(g->rho, g->total_nodes, 0);
  k_deposit_all<<<kGrid, TPB, 0, g->s>>>(make_ctx(g));
  if (g->any_protons) k_deposit_protons<<<kGrid, TPB, 0, g->s>>>(make_ctx(g));
  field_pass(g, make_fctx(g, 1));
}

template <class B>
void merge_store(gap_t* g, Store& st, B buf, SortBuf& sb, const double* thresh, double thresh_min, hipStream_t s) {
  const int t1 = (g->n_tubes + 255) / 256;
  k_merge_gate<<<1, 64, 0, s>>>(st.ctl, thresh_min, sb.gate);
  k_fill_i64<<<std::max(1, t1), 256, 0, s>>>(sb.live, g->n_tubes, 0);
  k_count_live<B><<<kGrid, TPB, 0, s>>>(buf, st.ctl, st.chunk[st.cur], st.tt, g->tiles, sb.live, g->n_tubes,
                                           sb.gate);
  // (one-wave workgroups: they start beside the other store's kernels)
  k_merge_flags<<<(g->n_tubes + WAVE - 1) / WAVE, WAVE, 0, s>>>(sb.live, thresh, sb.flags, g->n_tubes, sb.gate);
  k_fill_i64<<<1, 64, 0, s>>>(sb.n, 1, 0);
  k_merge_keys<B><<<kGrid, TPB, 0, s>>>(buf, st.ctl, st.chunk[st.cur], st.tt, g->tiles, g->tubes, sb);
  int src = 0;
  for (int pass = 0; pass < 12; ++pass) {
    k_rs_hist<<<kGrid, RS_TPB, 0, s>>>(sb, src, pass);
    k_rs_scan<<<RS_SCAN_WG, RS_SCAN_T, 0, s>>>(sb);
    k_rs_scatter<<<kGrid, RS_TPB, 0, s>>>(sb, src, pass);
    src ^= 1;
  }
  k_merge_bounds<<<kGrid, 256, 0, s>>>(sb, src, sb.start);
  k_mx_reduce<<<kGrid, RS_TPB, 0, s>>>(sb, sb.start, sb.bmax);
  k_mx_carry<<<1, 1024, 0, s>>>(sb, sb.bmax);
  k_mx_apply<<<kGrid, RS_TPB, 0, s>>>(sb, sb.start, sb.bmax);
  k_merge_pairs<B><<<kGrid, 256, 0, s>>>(buf, sb, src, sb.start, g->tubes, g->tiles, st.chunk[st.cur], st.tt,
                                            st.ctl, g->shard);
}

void merge_all(gap_t* g) {
  hipStream_t ps = fork_stores(g);
  merge_store<PhoBuf>(g, g->pho, g->pho.pho(g->pho.cur), g->sort_p, g->thresh_p, g->tmin_p, ps);
  merge_store<LepBuf>(g, g->lep, g->lep.lep(g->lep.cur), g->sort_l, g->thresh_l, g->tmin_l, g->s);
  join_stores(g, ps);
  // merged-away records are dead slots until the next scheduled re-sort
}

// ------------------------------------------------------------------ window
int sync_and_err(gap_t* g);
Ctl read_ctl(const Store& st);

void* walloc(gap_t* g, size_t bytes) {
  bytes = (bytes + 255) & ~(size_t)255;
  if (bytes == 0) bytes = 256;
  g->win.mem.push_back(nullptr);
  void* p = nullptr;
  if (g->custom_alloc) p = g->al.alloc(bytes, g->al.ctx);
  else if (hipMalloc(&p, bytes) != hipSuccess) p = nullptr;
  if (p) {
    g->win.mem.back() = p;
    (void)hipMemsetAsync(p, 0, bytes, g->s);
  } else {
    g->win.mem.pop_back();
  }
  return p;
}

void win_release(gap_t* g) {
  if (!g->win.mem.empty()) (void)hipStreamSynchronize(g->s);
  for (void* p : g->win.mem) {
    if (g->custom_alloc) g->al.free(p, g->al.ctx);
    else (void)hipFree(p);
  }
  g->win = WinState{};
}

// Workgroups of the fused tail launch: each role takes the tail workgroup
// count rounded up to a multiple of eight (the roles alternate in eights).
// threads of the prologue: a wave per 64 tubes, up to PRE_THREADS
int pre_threads(const gap_t* g) { return std::min(PRE_THREADS, (g->n_tubes + WAVE - 1) / WAVE * WAVE); }
int tails_grid(const gap_t* g) { return 2 * ((g->grid_tail + 7) / 8 * 8); }
// workgroups of the tail launch that write the sorted lepton pass's queued
// photon births: one per CU
int births_wg(const gap_t* g) { return std::max(16, g->cus); }
// workgroups that write the pairs of the converted photons (segs: workgroups
// of the photon pass, each with a queue segment)
int pairs_wg(const gap_t* g, int segs) { return std::min(std::max(16, g->cus), segs); }

// The particle kernels with the quantum branches only for handles that have
// quantum tubes.
void launch_leptons(gap_t* g, const Ctx& cx, hipStream_t s) {
  if (g->any_quantum) {
    if (g->any_atm) k_leptons<true, true><<<cx.bq_groups, TPB, 0, s>>>(cx);
    else k_leptons<true, false><<<cx.bq_groups, TPB, 0, s>>>(cx);
  } else {
    if (g->any_atm) k_leptons<false, true><<<cx.bq_groups, TPB, 0, s>>>(cx);
    else k_leptons<false, false><<<cx.bq_groups, TPB, 0, s>>>(cx);
  }
}
// The pairs of the converted photons.
void launch_conversions(gap_t* g, const Ctx& cx, hipStream_t s) {
  if (g->any_quantum) k_conversions<true><<<pairs_wg(g, cx.pq_groups), TPB, 0, s>>>(cx);
  else k_conversions<false><<<pairs_wg(g, cx.pq_groups), TPB, 0, s>>>(cx);
}
void launch_tails(gap_t* g, const Ctx& cx, hipStream_t s) {
  if (g->any_quantum) {
    if (g->any_atm) k_tails<true, true><<<tails_grid(g) + births_wg(g), TPB, 0, s>>>(cx, births_wg(g));
    else k_tails<true, false><<<tails_grid(g) + births_wg(g), TPB, 0, s>>>(cx, births_wg(g));
  } else {
    if (g->any_atm) k_tails<false, true><<<tails_grid(g) + births_wg(g), TPB, 0, s>>>(cx, births_wg(g));
    else k_tails<false, false><<<tails_grid(g) + births_wg(g), TPB, 0, s>>>(cx, births_wg(g));
  }
}

void join_photon_side(gap_t* g);

// The photon side of a window step (photon pass, pairs), forked
// onto the second stream once the caller's stream has done the prologue; the
// caller joins it at the end of the step (join_photon_side), before the next
// prologue takes the pairs it made.  The two sides touch disjoint data, as in
// enqueue_step.  Under graph capture everything stays on the caller's stream.
void fork_photon_side(gap_t* g, const Ctx& cx) {
  if (g->capturing) {
    k_photons<<<cx.pq_groups, TPB, 0, g->s>>>(cx);
    launch_conversions(g, cx, g->s);
    return;
  }
  (void)hipEventRecord(g->ev_pre, g->s);
  (void)hipStreamWaitEvent(g->s2, g->ev_pre, 0);
  k_photons<<<cx.pq_groups, TPB, 0, g->s2>>>(cx);
  launch_conversions(g, cx, g->s2);
  (void)hipEventRecord(g->ev_p, g->s2);
  g->s2_pending = true;
}

bool fused_form(const gap_t* g);
void enqueue_fused(gap_t* g, Ctx cx, bool pre);

// The particle passes of a window step whose prologue has run.
void window_passes(gap_t* g, const Ctx& cx) {
  if (fused_form(g)) {
    enqueue_fused(g, cx, false);
    return;
  }
  g->form = 0;
  fork_photon_side(g, cx);
  launch_leptons(g, cx, g->s);
  launch_tails(g, cx, g->s);
}

// One step of a window: no merge, no re-sort (slots stay put).  loss: per
// field block, accumulates the sum of E^2 after the step.
void enqueue_window_step(gap_t* g, double* loss) {
  const Ctx cx = make_ctx(g);
  if (fused_form(g)) {
    enqueue_fused(g, cx, true);
  } else {
    k_pre<<<1, pre_threads(g), 0, g->s>>>(cx, g->n_tubes);
    window_passes(g, cx);
  }
  FieldCtx f = make_fctx(g, 0);
  f.loss = loss;
  field_pass(g, f);
  join_photon_side(g);
  ++g->host_step;
}

#define D2D(dst, src, bytes) HIPCHK(hipMemcpyAsync((dst), (src), (bytes), hipMemcpyDeviceToDevice, g->s))

int save_ckpt(gap_t* g, WinCkpt& c) {
  HIPCHK(hipStreamSynchronize(g->s));
  c.lctl = read_ctl(g->lep);
  c.pctl = read_ctl(g->pho);
  if (c.lctl.tail != 0 || c.pctl.tail != 0) return GAP_ESTATE;
  c.nch_l = c.lctl.n_sorted_chunks;
  c.nch_p = c.pctl.n_sorted_chunks;
  g->seen_l = c.nch_l;
  g->seen_p = c.nch_p;
  g->rb_seen = 0;
  c.nl = c.nch_l * CHUNK;
  c.np = c.nch_p * CHUNK;
  const size_t nl = (size_t)c.nl, np = (size_t)c.np;
  c.lpos = (uint32_t*)walloc(g, nl * 4); c.lu = (float*)walloc(g, nl * 4); c.lw = (float*)walloc(g, nl * 4);
  c.lid = (uint64_t*)walloc(g, nl * 8); c.lchunk = (int32_t*)walloc(g, (size_t)c.nch_l * 4 + 4);
  c.ppos = (uint32_t*)walloc(g, np * 4); c.px = (float*)walloc(g, np * 4); c.pw = (float*)walloc(g, np * 4);
  c.pn0 = (int32_t*)walloc(g, np * 4); c.pid = (uint64_t*)walloc(g, np * 8);
  c.pchunk = (int32_t*)walloc(g, (size_t)c.nch_p * 4 + 4);
  c.tubes = (Tube*)walloc(g, sizeof(Tube) * g->n_tubes);
  c.ebar = (float*)walloc(g, sizeof(float) * g->total_nodes);
  c.E = (float*)walloc(g, sizeof(float) * g->total_cells);
  c.shard = (long long*)walloc(g, sizeof(long long) * g->n_tubes * NSHARD * C_N);
  if (!c.lpos || !c.lu || !c.lw || !c.lid || !c.lchunk || !c.ppos || !c.px || !c.pw || !c.pn0 || !c.pid ||
      !c.pchunk || !c.tubes || !c.ebar || !c.E || !c.shard)
    return GAP_ENOMEM;
  const Store& L = g->lep;
  const Store& P = g->pho;
  const int bl = L.cur, bp = P.cur;
  if (nl) {
    D2D(c.lpos, L.pos[bl], nl * 4); D2D(c.lu, L.a[bl], nl * 4); D2D(c.lw, L.w[bl], nl * 4);
    D2D(c.lid, L.id[bl], nl * 8); D2D(c.lchunk, L.chunk[bl], (size_t)c.nch_l * 4);
  }
  if (np) {
    D2D(c.ppos, P.pos[bp], np * 4); D2D(c.px, P.a[bp], np * 4); D2D(c.pw, P.w[bp], np * 4);
    D2D(c.pn0, P.n0[bp], np * 4); D2D(c.pid, P.id[bp], np * 8); D2D(c.pchunk, P.chunk[bp], (size_t)c.nch_p * 4);
  }
  D2D(c.tubes, g->tubes, sizeof(Tube) * g->n_tubes);
  D2D(c.ebar, g->ebar, sizeof(float) * g->total_nodes);
  D2D(c.E, g->E, sizeof(float) * g->total_cells);
  D2D(c.shard, g->shard, sizeof(long long) * g->n_tubes * NSHARD * C_N);
  c.host_step = g->host_step;
  return GAP_OK;
}

int restore_ckpt(gap_t* g, const WinCkpt& c) {
  Store& L = g->lep;
  Store& P = g->pho;
  const int bl = L.cur, bp = P.cur;
  const size_t nl = (size_t)c.nl, np = (size_t)c.np;
  if (nl) {
    D2D(L.pos[bl], c.lpos, nl * 4); D2D(L.a[bl], c.lu, nl * 4); D2D(L.w[bl], c.lw, nl * 4);
    D2D(L.id[bl], c.lid, nl * 8); D2D(L.chunk[bl], c.lchunk, (size_t)c.nch_l * 4);
  }
  if (np) {
    D2D(P.pos[bp], c.ppos, np * 4); D2D(P.a[bp], c.px, np * 4); D2D(P.w[bp], c.pw, np * 4);
    D2D(P.n0[bp], c.pn0, np * 4); D2D(P.id[bp], c.pid, np * 8); D2D(P.chunk[bp], c.pchunk, (size_t)c.nch_p * 4);
  }
  // the saved layout's hot prefixes are not kept: no cold guarantee until
  // the next re-sort
  Ctl lc = c.lctl, pc = c.pctl;
  lc.cold_steps = pc.cold_steps = -1;
  HIPCHK(hipMemcpyAsync(L.ctl, &lc, sizeof(Ctl), hipMemcpyHostToDevice, g->s));
  HIPCHK(hipMemcpyAsync(P.ctl, &pc, sizeof(Ctl), hipMemcpyHostToDevice, g->s));
  D2D(g->tubes, c.tubes, sizeof(Tube) * g->n_tubes);
  D2D(g->ebar, c.ebar, sizeof(float) * g->total_nodes);
  D2D(g->E, c.E, sizeof(float) * g->total_cells);
  D2D(g->shard, c.shard, sizeof(long long) * g->n_tubes * NSHARD * C_N);
  HIPCHK(hipStreamSynchronize(g->s));
  g->host_step = c.host_step;
  g->since_rb = 0;
  g->seen_l = c.nch_l;
  g->seen_p = c.nch_p;
  g->rb_seen = 0;
  return GAP_OK;
}

int window_forward(gap_t* g, int64_t W, int64_t K, double* loss) {
  if (g->any_protons) return GAP_EINVAL;   // the differentiated map has leptons only
  for (int t = 0; t < g->n_tubes; ++t) {
    const gap_params& q = g->P[t];
    if (q.flags & (GAP_PERIODIC | GAP_FIELD_FROZEN)) return GAP_EINVAL;
    const int64_t rmax = std::max(1, (int)std::floor((MARGIN - 2) / q.cfl) - 1);
    if (K > rmax) return GAP_EINVAL;
  }
  win_release(g);
  WinState& w = g->win;
  w.W = W;
  w.K = K;
  w.nseg = (W + K - 1) / K;
  w.ck.resize((size_t)w.nseg + 1);
  w.loss_acc = (double*)walloc(g, sizeof(double) * g->n_fb);
  if (!w.loss_acc) return GAP_ENOMEM;
  int e;
  for (int64_t sg = 0; sg < w.nseg; ++sg) {
    rebucket_all(g);
    g->since_rb = 0;
    if ((e = save_ckpt(g, w.ck[sg]))) return e;
    const int64_t Ks = std::min(K, W - sg * K);
    for (int64_t j = 0; j < Ks; ++j) enqueue_window_step(g, w.loss_acc);
    HIPCHK(hipStreamSynchronize(g->s));
    const Ctl c = read_ctl(g->lep);
    w.max_used = std::max<long long>(w.max_used, c.n_sorted_chunks * CHUNK + c.tail);
  }
  rebucket_all(g);
  g->since_rb = 0;
  if ((e = save_ckpt(g, w.ck[(size_t)w.nseg]))) return e;
  if ((e = sync_and_err(g))) return e;
  std::vector<double> acc(g->n_fb), sum(g->n_tubes, 0.0);
  HIPCHK(hipMemcpy(acc.data(), w.loss_acc, sizeof(double) * g->n_fb, hipMemcpyDeviceToHost));
  for (int b = 0; b < g->n_fb; ++b) sum[g->fb_h[b].tube] += acc[b];
  for (int t = 0; t < g->n_tubes; ++t) loss[t] = sum[t] / ((double)W * g->P[t].n_cells);
  w.step_end = g->host_step;
  w.valid = true;
  return GAP_OK;
}

int backward_alloc(gap_t* g) {
  WinState& w = g->win;
  if (w.tpos) return GAP_OK;
  w.M = (w.max_used + CHUNK - 1) / CHUNK * CHUNK + CHUNK;
  const size_t M = (size_t)w.M, K = (size_t)w.K;
  w.tpos = (uint32_t*)walloc(g, (K + 1) * M * 4);
  w.tu = (float*)walloc(g, (K + 1) * M * 4);
  w.meta = (TapeMeta*)walloc(g, (K + 1) * sizeof(TapeMeta));
  w.teb = (float*)walloc(g, (K + 1) * (size_t)g->total_nodes * 4);
  w.tE = (float*)walloc(g, (K + 1) * (size_t)g->total_cells * 4);
  w.wlast = (float*)walloc(g, M * 4);
  for (int b = 0; b < 2; ++b)
    for (int k = 0; k < 3; ++k) w.lam[b][k] = (float*)walloc(g, M * 4);
  w.lamE = (double*)walloc(g, (size_t)g->total_cells * 8);
  w.suf = (double*)walloc(g, (size_t)g->total_nodes * 8);
  for (int b = 0; b < 2; ++b) w.lamEb[b] = (double*)walloc(g, (size_t)g->total_nodes * 8);
  w.frec = (unsigned long long*)walloc(g, sizeof(unsigned long long) * (4 * (size_t)g->n_fb + g->n_tubes));
  w.at = (AdjTube*)walloc(g, sizeof(AdjTube) * g->n_tubes);
  uint64_t hs = 1024;
  while (hs < 2 * (uint64_t)M) hs <<= 1;
  w.hmask = hs - 1;
  w.hvals = (uint32_t*)walloc(g, hs * 4);
  if (!w.tpos || !w.tu || !w.meta || !w.teb || !w.tE || !w.wlast || !w.lamE || !w.suf || !w.lamEb[0] ||
      !w.lamEb[1] || !w.frec || !w.at || !w.hvals)
    return GAP_ENOMEM;
  for (int b = 0; b < 2; ++b)
    for (int k = 0; k < 3; ++k)
      if (!w.lam[b][k]) return GAP_ENOMEM;
  return GAP_OK;
}

int backward(gap_t* g, double* dalpha, double* dninj) {
  WinState& w = g->win;
  if (!w.valid || g->host_step != w.step_end) return GAP_ESTATE;
  int e;
  if ((e = backward_alloc(g))) return e;
  {
    std::vector<AdjTube> at(g->n_tubes);
    for (int t = 0; t < g->n_tubes; ++t) {
      AdjTube& a = at[t];
      std::memset(&a, 0, sizeof(a));
      a.w0 = g->D[t].w0;
      a.s_co = g->D[t].s_co;
      a.dt = g->D[t].dt;
      a.cfl = g->P[t].cfl;
      a.lossw = 2.0 / ((double)w.W * g->P[t].n_cells);
      a.N = g->P[t].n_cells;
      a.cell_off = g->th[t].cell_off;
      a.node_off = g->th[t].node_off;
    }
    HIPCHK(hipStreamSynchronize(g->s));
    HIPCHK(hipMemcpy(w.at, at.data(), sizeof(AdjTube) * g->n_tubes, hipMemcpyHostToDevice));
  }
  const size_t M = (size_t)w.M, nn = (size_t)g->total_nodes, nc = (size_t)g->total_cells;
  const int fgrid = (int)std::min<long long>(4096, (w.M + 255) / 256);
  int cur = 0;
  // node-field adjoints of the step being reversed and of the one before it
  int nb = 0;
  for (int b = 0; b < 2; ++b)
    k_fill_i64<<<std::max(1, (int)std::min<size_t>(1024, (nn + 255) / 256)), 256, 0, g->s>>>((long long*)w.lamEb[b],
                                                                                             (long long)nn, 0);
  // the reverse field pass: of the window's last field, or (step) of the one
  // before a step whose leptons have been reversed
  auto adj_field = [&](const float* E, bool step) {
    AdjFieldCtx f{g->fb, w.frec, w.lamE, w.suf, step ? w.lamEb[nb] : nullptr, w.lamEb[nb ^ 1], E, w.at, g->err};
    k_adj_field<<<g->n_fb, FB_THREADS, 0, g->s>>>(f);
    if (step) nb ^= 1;
  };
  for (int64_t sg = w.nseg - 1; sg >= 0; --sg) {
    if ((e = restore_ckpt(g, w.ck[(size_t)sg]))) return e;
    const int64_t Ks = std::min(w.K, w.W - sg * w.K);
    D2D(w.tE, g->E, sizeof(float) * nc);
    D2D(w.teb, g->ebar, sizeof(float) * nn);
    // recompute the segment, taping the lepton store before each step and the
    // fields as they are made (the handle's own are restored at the end)
    for (int64_t j = 0; j < Ks; ++j) {
      Ctx cx = make_ctx(g);
      cx.ebar = w.teb + j * nn;
      k_pre<<<1, pre_threads(g), 0, g->s>>>(cx, g->n_tubes);
      k_tape<<<fgrid, 256, 0, g->s>>>(cx.L, g->lep.ctl, w.tpos + j * M, w.tu + j * M, w.wlast, w.meta + j,
                                      w.M, 0, g->err);
      window_passes(g, cx);          // (the tape of the leptons is taken; photons are not taped)
      FieldCtx f = make_fctx(g, 0);
      f.E = w.tE + (j + 1) * nc;
      f.ebar = w.teb + (j + 1) * nn;
      field_pass(g, f);
      ++g->host_step;
      join_photon_side(g);
    }
    {
      Ctx cx = make_ctx(g);
      k_tape<<<fgrid, 256, 0, g->s>>>(cx.L, g->lep.ctl, w.tpos + Ks * M, w.tu + Ks * M, w.wlast, w.meta + Ks,
                                      w.M, 1, g->err);
    }
    // adjoint of the state after the segment, in this recomputed layout
    if (sg == w.nseg - 1) {
      for (int k = 0; k < 3; ++k) k_fill_i32<<<fgrid, 256, 0, g->s>>>((int32_t*)w.lam[cur][k], w.M, 0);
      adj_field(w.tE + Ks * nc, false);
    } else {
      const WinCkpt& nx = w.ck[(size_t)sg + 1];
      const int hgrid = (int)std::min<uint64_t>(4096, (w.hmask + 256) / 256);
      k_hash_clear<<<hgrid, 256, 0, g->s>>>(w.hvals, (long long)w.hmask + 1);
      k_hash_insert<<<fgrid, 256, 0, g->s>>>(nx.lid, nx.lw, nx.lchunk, g->tiles, nx.nl, w.hvals, w.hmask);
      const int nw = cur ^ 1;
      k_lam_map<<<fgrid, 256, 0, g->s>>>(g->lep.lep(g->lep.cur), g->lep.ctl, g->lep.chunk[g->lep.cur], g->lep.tt,
                                         g->tiles, nx.lid, nx.lchunk, w.hvals, w.hmask,
                                         w.lam[cur][0], w.lam[cur][1], w.lam[cur][2], w.lam[nw][0], w.lam[nw][1],
                                         w.lam[nw][2], w.M, g->err);
      cur = nw;
    }
    // reverse steps
    AdjCtx ac;
    ac.tiles = g->tiles;
    ac.chunk = g->lep.chunk[g->lep.cur];
    ac.tt = g->lep.tt;
    ac.wlast = w.wlast;
    ac.lxi = w.lam[cur][0];
    ac.lu = w.lam[cur][1];
    ac.lw = w.lam[cur][2];
    ac.lamE = w.lamE;
    ac.suf = w.suf;
    ac.at = w.at;
    for (int64_t j = Ks - 1; j >= 0; --j) {
      ac.pos0 = w.tpos + j * M;
      ac.u0 = w.tu + j * M;
      ac.pos1 = w.tpos + (j + 1) * M;
      ac.u1 = w.tu + (j + 1) * M;
      ac.meta0 = w.meta + j;
      ac.eb0 = w.teb + j * nn;
      ac.lamEb = w.lamEb[nb];
      k_adj_leptons<<<ADJ_GRID, TPB, 0, g->s>>>(ac);
      if (sg > 0 || j > 0) adj_field(w.tE + j * nc, true);   // (the window's start field is not in the loss)
    }
  }
  if ((e = sync_and_err(g))) return e;
  std::vector<AdjTube> at(g->n_tubes);
  HIPCHK(hipMemcpy(at.data(), w.at, sizeof(AdjTube) * g->n_tubes, hipMemcpyDeviceToHost));
  for (int t = 0; t < g->n_tubes; ++t) {
    dalpha[t] = at[t].dalpha;
    const double rate = g->P[t].inj_rate;
    dninj[t] = rate > 0 ? at[t].dinjw / rate : 0.0;
  }
  if ((e = restore_ckpt(g, w.ck[(size_t)w.nseg]))) return e;
  return sync_and_err(g);
}

#undef D2D

// The caller's stream waits for the photon side of the steps enqueued so far.
void join_photon_side(gap_t* g) {
  if (!g->s2_pending) return;
  (void)hipStreamWaitEvent(g->s, g->ev_p, 0);
  g->s2_pending = false;
}

// The particle passes of a step in their general form: on two streams, or
// (two == false) on the caller's.
void enqueue_passes(gap_t* g, bool two, bool merged) {
  g->form = 0;
  Ctx cx = make_ctx(g);
  hipStream_t ps = g->s;
  if (two) {
    ps = g->s2;
    // the previous step's field kernel carries ev_l when nothing came after it
    if (merged || !g->ev_l_bound) (void)hipEventRecord(g->ev_l, g->s);
    (void)hipStreamWaitEvent(g->s2, g->ev_l, 0);
  }
  g->ev_l_bound = false;
  {
    Timer t(g, KT_PRE, ps);
    if (two) hipExtLaunchKernelGGL(k_pre, dim3(1), dim3(pre_threads(g)), 0, ps, nullptr, g->ev_pre, 0, cx, g->n_tubes);
    else k_pre<<<1, pre_threads(g), 0, ps>>>(cx, g->n_tubes);
  }
  { Timer t(g, KT_PHOTONS, ps); k_photons<<<cx.pq_groups, TPB, 0, ps>>>(cx); }
  { Timer t(g, KT_CONV, ps); launch_conversions(g, cx, ps); }
  if (two) {
    (void)hipEventRecord(g->ev_p, g->s2);
    g->s2_pending = true;
  }
  { Timer t(g, KT_LEPTONS); launch_leptons(g, cx, g->s); }
  if (two) (void)hipStreamWaitEvent(g->s, g->ev_pre, 0);
  { Timer t(g, KT_TAILS); launch_tails(g, cx, g->s); }
  if (g->any_protons) {
    Timer t(g, KT_TAILS);
    k_protons<<<std::max(8, g->grid_tail), TPB, 0, g->s>>>(cx);
  }
}

// The fused form of the particle passes (gap_fused.hpp) is for photon stores
// of at most this many chunks (1024 slots each): where the forms cross depends
// on the leptons too, and the line lies between.  A step in it and in the
// general form: the production gap with 225 photon chunks 28 and 49 us, 3900
// 45 and 57, 7000 (and 2600 of leptons) 65 and 67, 8200 73 and 70, 10400 88
// and 79; the paper's setup with 6200 69 and 82, 16700 130 and 124; 8
// QED-active tubes with 4300 lepton chunks 63 and 63 at no photons, 73 and 70
// at 1400, 87 and 79 at 3700.
constexpr int64_t FUSED_PHO_CHUNKS = 4096;

// Whether the next step takes the fused form.  A store's chunk count, read
// back at every synchronising call, holds until the next re-sort, and is
// taken as a sign of its size for three periods after that; a longer run
// without such a call may have grown the store, and goes over to the general
// form.  (No result depends on it.  With one period after it the tiny gap's
// 500-step cascade takes 14.4 to 14.8 ms instead of 11.7.)
bool fused_form(const gap_t* g) {
  return !g->apart && g->seen_l >= 0 && g->seen_p >= 0 && g->seen_p <= FUSED_PHO_CHUNKS && g->rb_seen <= 3;
}

template <bool Q, bool A, int V>
void launch_fused(gap_t* g, const Ctx& cx, bool pre, int gp, int gl, const RestGrid& n) {
  k_sorted<Q, A, V><<<FUSED_PRE + gp + gl, TPB, 0, g->s>>>(cx, pre ? g->n_tubes : -1, gp, gl);
  k_rest<Q, A><<<n.births + n.conv + n.tails + n.protons, TPB, 0, g->s>>>(cx, n);
}

// The particle passes of one step on the caller's stream (pre: the prologue
// with them).
void enqueue_fused(gap_t* g, Ctx cx, bool pre) {
  // A workgroup per chunk up to the usual grids, and a store of fewer chunks
  // than CUs in pieces of a quarter chunk.  After a re-sort the counts are a
  // sign only, and the grids twice what they say and at least some per tile:
  // a store may have grown since.  In a graph, which will be replayed on other
  // counts, one resident round.  (With one round also after a re-sort the tiny
  // gap's 500-step cascade takes 12.4 ms instead of 11.7, 200 steps of the
  // production gap's start 6.37 instead of 5.89; with pieces up to a resident
  // round of them the latter takes 6.28.  No result depends on it.)
  const bool exact = g->rb_seen == 0;
  const bool pieces = !g->capturing && g->seen_l < g->cus && g->seen_p < g->cus;
  g->form = pieces ? 2 : 1;
  auto grid = [&](int64_t chunks, int most) {
    if (g->capturing) return most;
    const int64_t n = (pieces ? PPC : 1) * (exact ? chunks : 2 * std::max<int64_t>(chunks, 16 + g->n_tiles / 8));
    return (int)std::max<int64_t>(8, std::min<int64_t>((n + 7) / 8 * 8, most));
  };
  const int gl = grid(g->seen_l, lepton_grid(g)), gp = grid(g->seen_p, std::min(g->grid_pho, g->round_pho));
  cx.bq_groups = gl;
  cx.pq_groups = gp;
  RestGrid n;
  n.births = std::min(births_wg(g), gl);
  n.conv = pairs_wg(g, gp);
  n.tails = tails_grid(g);
  n.protons = g->any_protons ? std::max(8, g->grid_tail) : 0;
  const int form = (g->any_quantum ? 4 : 0) | (g->any_atm ? 2 : 0) | (pieces ? 1 : 0);
  switch (form) {
    case 0: launch_fused<false, false, VEC>(g, cx, pre, gp, gl, n); break;
    case 1: launch_fused<false, false, 1>(g, cx, pre, gp, gl, n); break;
    case 2: launch_fused<false, true, VEC>(g, cx, pre, gp, gl, n); break;
    case 3: launch_fused<false, true, 1>(g, cx, pre, gp, gl, n); break;
    case 4: launch_fused<true, false, VEC>(g, cx, pre, gp, gl, n); break;
    case 5: launch_fused<true, false, 1>(g, cx, pre, gp, gl, n); break;
    case 6: launch_fused<true, true, VEC>(g, cx, pre, gp, gl, n); break;
    default: launch_fused<true, true, 1>(g, cx, pre, gp, gl, n); break;
  }
}

// One step.  Photon side (second stream): prologue (injection, lepton tail
// snapshot, step index), sorted photon pass, pairs.  Lepton side
// (caller's stream): sorted lepton pass, then, once the prologue is done,
// the lepton and photon tail passes, the field update (which also takes the
// photon tail snapshot of the next step) and the re-sort when due.  The
// re-sort and the merge check join the photon side and then run the two
// stores side by side (fork_stores).
//
// The sides touch disjoint data: each pass reads its own store up to its
// tail snapshot, births go past the snapshots, only leptons deposit charge,
// and the prologue changes the surface charge only atomically.  The photon
// side of a step starts when the caller's stream has finished the previous
// step (its field update counts the step and snapshots the photon tail);
// the lepton side needs the photon side only for its tail passes (the
// prologue's snapshot) and for the re-sort and merging (everything).  So the
// sorted lepton pass of a step starts without waiting, and one step costs
// one wait on each stream.  Captured graphs keep every kernel on the
// caller's stream, in an order that respects the same dependencies.
void enqueue_step(gap_t* g, bool more) {
  const bool two = !g->capturing;
  const bool merge = g->merge_on && g->host_step % g->merge_every == 0;
  if (merge) {
    if (two) join_photon_side(g);
    Timer t(g, KT_MERGE);
    merge_all(g);
  }
  const bool fused = g->capturing ? g->graph_fused : fused_form(g);
  if (fused) {
    if (two) join_photon_side(g);
    g->ev_l_bound = false;
    enqueue_fused(g, make_ctx(g), true);
  } else {
    enqueue_passes(g, two, merge);
  }
  {
    // another step follows at once, with no re-sort or merge in between:
    // its photon side can wait on the field kernel itself
    const bool bind = two && !fused && more && g->since_rb + 1 < g->R &&
                      !(g->merge_on && (g->host_step + 1) % g->merge_every == 0);
    Timer t(g, KT_FIELD);
    g->ev_l_bound = field_pass(g, make_fctx(g, 0), bind ? g->ev_l : nullptr);
  }
  if (g->wf_every > 0) {
    WfCtx w{g->tubes, g->E, g->wf_ring, g->wf_steps, g->wf_every, g->wf_B, g->wf_cap, g->wf_nbmax};
    k_waterfall<<<dim3((g->wf_nbmax + TPB / WAVE - 1) / (TPB / WAVE), g->n_tubes), TPB, 0, g->s>>>(w);
  }
  if (++g->since_rb >= g->R) {
    if (two) join_photon_side(g);
    Timer t(g, KT_RESORT);
    rebucket_all(g);
    g->since_rb = 0;
  }
  ++g->host_step;
}

int take_status(gap_t* g, const gap_t::Status& st) {
  const int e = st.err;
  g->seen_l = st.chunks[0] - 1;
  g->seen_p = st.chunks[1] - 1;
  g->rb_seen = 0;
  if (e & E_TILE) g->sticky = GAP_ETILE;
  else if (e & E_NAN) g->sticky = GAP_ENAN;
  else if (e & E_SCAN) g->sticky = GAP_EDEVICE;
  else if (e & E_CAP) g->sticky = GAP_ECAP;
  return g->sticky;
}

int read_err(gap_t* g) {
  gap_t::Status st{};
  if (hipMemcpy(&st, g->status, sizeof(st), hipMemcpyDeviceToHost) != hipSuccess) return GAP_EDEVICE;
  return take_status(g, st);
}

int sync_and_err(gap_t* g) {
  if (hipStreamSynchronize(g->s) != hipSuccess) return GAP_EDEVICE;
  if (hipGetLastError() != hipSuccess) return GAP_EDEVICE;
  return read_err(g);
}

// Reads `bytes` device bytes into host memory behind all queued work, together
// with the status words: one kernel gathers both, so that one copy and one
// wait do (the copies of a few bytes cost what a wait does: a step of the tiny
// gap with a read of its field and its charge took 87 us with two waits and
// two copies per read).  Results past the staging buffer, for which the
// conversion queue serves (every call joins the photon side before it
// returns), take their own copy.
constexpr size_t kStageBytes = 4 << 20;
constexpr size_t kStageHead = 64;
static_assert(sizeof(gap_t::Status) <= kStageHead, "");

__global__ void k_gather(const uint32_t* status, const uint32_t* src, long long words, uint32_t* out) {
  const long long i0 = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i0 < (long long)(sizeof(gap_t::Status) / 4)) out[i0] = status[i0];
  for (long long i = i0; i < words; i += (long long)gridDim.x * blockDim.x) out[kStageHead / 4 + i] = src[i];
}

int read_back(gap_t* g, const void* src, size_t bytes, void* host) {
  if (bytes + kStageHead > g->stage_bytes || bytes % 4 != 0) {
    const int e = sync_and_err(g);
    if (e == GAP_EDEVICE) return e;
    HIPCHK(hipMemcpy(host, src, bytes, hipMemcpyDeviceToHost));
    return GAP_OK;
  }
  const long long words = (long long)(bytes / 4);
  g->stage_h.resize(kStageHead + bytes);
  k_gather<<<std::max(1, (int)std::min<long long>(256, (words + 255) / 256)), 256, 0, g->s>>>(
      (const uint32_t*)g->status, (const uint32_t*)src, words, g->stage);
  HIPCHK(hipMemcpyAsync(g->stage_h.data(), g->stage, kStageHead + bytes, hipMemcpyDeviceToHost, g->s));
  HIPCHK(hipStreamSynchronize(g->s));
  if (hipGetLastError() != hipSuccess) return GAP_EDEVICE;
  gap_t::Status st;
  std::memcpy(&st, g->stage_h.data(), sizeof(st));
  if (take_status(g, st) == GAP_EDEVICE) return GAP_EDEVICE;
  std::memcpy(host, g->stage_h.data() + kStageHead, bytes);
  return GAP_OK;
}

Ctl read_ctl(const Store& st) {
  Ctl c{};
  (void)hipMemcpy(&c, st.ctl, sizeof(Ctl), hipMemcpyDeviceToHost);
  return c;
}

int alloc_store(gap_t* g, Store& st, int64_t cap, bool photon) {
  st.cap_live = cap;
  st.capacity = cap + 2LL * g->n_tiles * CHUNK + CHUNK;
  st.limit = st.capacity - (int64_t)g->n_tiles * CHUNK;
  const size_t n = (size_t)st.capacity;
  for (int b = 0; b < 2; ++b) {
    st.pos[b] = (uint32_t*)dalloc(g, n * 4);
    st.a[b] = (float*)dalloc(g, n * 4);
    st.w[b] = (float*)dalloc(g, n * 4);
    st.id[b] = (uint64_t*)dalloc(g, n * 8);
    if (photon) st.n0[b] = (int32_t*)dalloc(g, n * 4);
    st.chunk[b] = (int32_t*)dalloc(g, (n / CHUNK + 1) * 4);
    if (!st.pos[b] || !st.a[b] || !st.w[b] || !st.id[b] || (photon && !st.n0[b]) || !st.chunk[b]) return GAP_ENOMEM;
  }
  st.tt = (int32_t*)dalloc(g, n * 4);
  st.tcount = (int32_t*)dalloc(g, (size_t)g->n_tiles * 4);
  st.nclass = photon ? RbClasses<PhoBuf>::N : RbClasses<LepBuf>::N;
  st.ccount = (int32_t*)dalloc(g, (size_t)(st.nclass - 1) * g->n_tiles * 4);
  st.ccur = (int32_t*)dalloc(g, (size_t)st.nclass * g->n_tiles * 4);
  st.wh = (int32_t*)dalloc(g, (size_t)kGrid * rb_window(g->n_tiles) * st.nclass * 4);
  st.cls = (uint8_t*)dalloc(g, (size_t)st.capacity);
  if (!st.ccount || !st.ccur || !st.cls || !st.wh) return GAP_ENOMEM;
  if (photon) {
    st.chot = (uint16_t*)dalloc(g, (n / CHUNK + 1) * 2);
    if (!st.chot) return GAP_ENOMEM;
  }
  st.tchunk = (long long*)dalloc(g, ((size_t)g->n_tiles + 1) * 8);
  st.ctl = (Ctl*)dalloc(g, sizeof(Ctl));
  if (!st.tt || !st.tcount || !st.tchunk || !st.ctl) return GAP_ENOMEM;
  Ctl c{};
  c.capacity = st.capacity;
  c.limit = st.limit;
  c.cap_live = cap;
  c.cold_steps = -1;
  if (hipMemcpyAsync(st.ctl, &c, sizeof(Ctl), hipMemcpyHostToDevice, g->s) != hipSuccess) return GAP_EDEVICE;
  return GAP_OK;
}

int upload_tubes(gap_t* g) {
  return from_hip(hipMemcpy(g->tubes, g->th.data(), sizeof(Tube) * g->n_tubes, hipMemcpyHostToDevice));
}
int download_tubes(gap_t* g) {
  return from_hip(hipMemcpy(g->th.data(), g->tubes, sizeof(Tube) * g->n_tubes, hipMemcpyDeviceToHost));
}

// The sorted lepton pass's constants of one tile.
LTile lepton_tile(const Tube& T, const Tile& tl, double xc_floor) {
  LTile k{};
  k.tube = tl.tube;
  k.base = tl.base;
  k.N = T.N;
  k.node_off = T.node_off;
  k.flags = (uint32_t)T.flags;
  const bool per = (T.flags & GAP_PERIODIC) != 0;
  const int64_t b0 = (int64_t)tl.base * (1 << FRAC), last = 0xFFFFFFFFll;
  k.xlo = per || tl.base >= 0 ? 0u : (uint32_t)(-b0);
  k.xtop = (uint32_t)(per ? last : std::min(((int64_t)T.N << FRAC) - b0 - 1, last));
  const int64_t z = T.hfix - b0 - 1;      // last offset inside the QED zone
  k.zone = per || z >= 0;
  k.ztop = (uint32_t)(per ? last : std::max(std::min(z, last), (int64_t)0));
  k.dt = T.dt;
  k.cfl24 = T.cfl24;
  k.lr = T.lr;
  k.emit_k = T.emit_k;
  k.xc_floor = T.xc_floor;
  k.x_thr = T.x_thr;
  // x_c = 1.5 gamma^3 lambda~/R~ reaches the floor at this gamma; one per
  // cent under its momentum x_c is at least 0.5 % under the floor (from
  // gamma = 1.1 on), far beyond the rounding of the passes' FP32 x_c
  const double gf = std::cbrt(xc_floor / (1.5 * (double)T.lr));
  k.u_skip = gf > 1.1 ? (float)(0.99 * std::sqrt(gf * gf - 1.0)) : 0.0f;
  k.nsub_max = T.nsub_max;
  k.hfix = T.hfix;
  k.seed = T.seed;
  return k;
}

// The sorted photon pass's constants of one tile.
PTile photon_tile(const Tube& T, const Tile& tl) {
  PTile k{};
  k.tube = tl.tube;
  k.base = tl.base;
  k.N = T.N;
  k.dpho = T.dpho;
  k.flags = (uint32_t)T.flags;
  const bool per = (T.flags & GAP_PERIODIC) != 0;
  const int64_t b0 = (int64_t)tl.base * (1 << FRAC), last = 0xFFFFFFFFll;
  // a photon stays while it is in [0, L) and below H
  const int64_t top = std::min(T.hfix, (int64_t)T.N << FRAC) - b0 - 1;
  k.xlo = per || tl.base >= 0 ? 0u : (uint32_t)(-b0);
  k.xtop = (uint32_t)(per ? last : std::max(std::min(top, last), (int64_t)0));
  if (!per && top < 0) {                       // every position is above it
    k.xlo = 1;
    k.xtop = 0;
  }
  k.dt = T.dt;
  k.inv_rc = T.inv_rc;
  k.b = T.b;
  k.conv_k = T.conv_k;
  k.chi_skip = T.chi_skip;
  k.hfix = T.hfix;
  k.seed = T.seed;
  return k;
}

int build(gap_t* g, const gap_params* p, int n_tubes) {
  g->n_tubes = n_tubes;
  g->P.assign(p, p + n_tubes);
  g->D.resize(n_tubes);
  g->th.assign(n_tubes, Tube{});
  int64_t cap_l = 0, cap_p = 0;
  int rmin = 1 << 30;
  for (int t = 0; t < n_tubes; ++t) {
    const gap_params& q = g->P[t];
    const Derived d = derive(q);
    g->D[t] = d;
    Tube& T = g->th[t];
    std::memset(&T, 0, sizeof(Tube));
    T.N = q.n_cells;
    T.node_off = (int32_t)g->total_nodes;
    T.cell_off = (int32_t)g->total_cells;
    T.tile_first = g->n_tiles;
    T.n_tiles = (q.n_cells + TILE - 1) / TILE;
    T.flags = q.flags;
    T.nsub_max = q.nsub_max;
    T.dt = (float)d.dt;
    T.cfl24 = (float)(q.cfl * kTwo24);
    T.lr = (float)(d.lam / d.rc);
    T.inv_rc = (float)(1.0 / d.rc);
    T.b = (float)q.b;
    T.b_over_lam = (float)(q.b / d.lam);
    T.xc_floor = (float)q.xc_floor;
    T.x_thr = (float)q.x_thr;
    T.emit_k = (float)(kAlphaEM * d.dt / d.rc);
    T.conv_k = (float)(kAlphaEM * d.dt * q.b / d.lam);
    {
      // p <= conv_k 0.23 exp(-8/(3 chi)) <= 2^-27 for chi <= chi_skip
      const double a = 0.23 * (double)T.conv_k * 134217728.0;
      T.chi_skip = a > 1.0 ? (float)(8.0 / (3.0 * std::log(a))) : 3.0e38f;
    }
    T.dpho = (int32_t)std::llrint(q.cfl * kTwo24);
    T.dtd = d.dt;
    T.scale = d.w0 / kTwo24;
    T.drive = q.alpha * d.s_co * d.dt;
    T.inj_per_step = q.inj_rate * q.ppc_ref / ((q.flags & GAP_INJ_FIXED) ? 1.0 : q.inj_weight);
    T.inv_len_scale = d.w0 / ((double)q.n_cells * kTwo24 * kTwo24);
    T.bg_unit = (q.flags & GAP_ETA_CO_OFF) ? 0 : (int64_t)std::llrint(-d.s_co) * q.ppc_ref * (int64_t)kTwo24;
    T.hfix = (int64_t)std::ceil(q.h_gap_frac * q.n_cells * kTwo24);
    T.inj_w = (float)q.inj_weight;
    T.inj_T = std::llrint((double)T.inj_w * kTwo24);
    T.seed = q.seed;
    T.atm_ppc = q.atm_ppc;
    T.atm_theta_e = q.atm_temp;
    T.atm_theta_p = q.atm_temp / (double)MASS_P;
    atm_reset(T);
    T.cnt[C_PROTONS] = init_protons(q, d);
    if (q.atm_ppc > 0) g->any_atm = true;
    if (q.atm_ppc > 0 || q.init_kind == GAP_INIT_ATMOSPHERE) {
      g->any_protons = true;
      g->pr_cap += q.cap_leptons;
    }
    for (int j = 0; j < T.n_tiles; ++j) {
      Tile tl;
      tl.tube = t;
      tl.first = j * TILE;
      tl.base = tl.first - MARGIN;
      tl.ncell = std::min(TILE, q.n_cells - tl.first);
      g->tiles_h.push_back(tl);
      g->ltiles_h.push_back(lepton_tile(T, tl, q.xc_floor));
      g->ptiles_h.push_back(photon_tile(T, tl));
    }
    const int nb = (q.n_cells + FB_NODES - 1) / FB_NODES;
    const int first = (int)g->fb_h.size();
    for (int j = 0; j < nb; ++j) g->fb_h.push_back(FBlk{t, j * FB_NODES, first, nb, T.N, T.node_off, T.cell_off, T.flags, T.scale, T.bg_unit});
    g->n_tiles += T.n_tiles;
    g->total_nodes += q.n_cells + 1;
    g->total_cells += q.n_cells;
    cap_l += q.cap_leptons;
    cap_p += q.cap_photons;
    if (q.flags & GAP_PERIODIC) g->any_periodic = true;
    if (q.flags & GAP_FILTER) g->any_filter = true;
    if (q.flags & GAP_QUANTUM) g->any_quantum = true;
    g->max_cells = std::max(g->max_cells, q.n_cells);
    const int rmax = std::max(1, (int)std::floor((MARGIN - 2) / q.cfl) - 1);
    rmin = std::min(rmin, q.rebucket_every > 0 ? std::min(q.rebucket_every, rmax) : rmax);
  }
  g->R = rmin;
  g->rmax = 1 << 30;
  for (int t = 0; t < n_tubes; ++t)
    g->rmax = std::min(g->rmax, std::max(1, (int)std::floor((MARGIN - 2) / g->P[t].cfl) - 1));
  g->n_fb = (int)g->fb_h.size();
  {
    // one resident round of workgroups for the persistent-range passes
    int dev = 0, cus = 0, nl = 0, np = 0;
    HIPCHK(hipGetDevice(&dev));
    HIPCHK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    HIPCHK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&nl, k_leptons<false, false>, TPB, 0));
    HIPCHK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&np, k_photons, TPB, 0));
    // defaults measured on the production gap (2e7 particles): one resident
    // round for the lepton pass, four for the photon pass (short ranges keep
    // its conversion queue segments small), two workgroups per CU for each
    // role of the fused tail launch; gap_autotune or GAP_STATE_LAUNCH can
    // change them
    g->round_lep = std::max(8, (cus * std::max(nl, 1)) / 8 * 8);
    g->round_pho = std::max(8, (cus * std::max(np, 1)) / 8 * 8);
    g->grid_lep = g->round_lep;
    g->grid_pho = 4 * g->round_pho;
    g->grid_tail = std::max(8, cus * 2);
    g->cus = cus;
  }
  if (g->total_nodes > (1LL << 30)) return GAP_EINVAL;

  g->tubes = (Tube*)dalloc(g, sizeof(Tube) * n_tubes);
  // the tiles, both passes' constants of them and the edges of the spectra's
  // bins: one allocation, one copy
  const size_t part_bytes[5] = {sizeof(Tile) * (size_t)g->n_tiles, sizeof(LTile) * (size_t)g->n_tiles,
                                sizeof(PTile) * (size_t)g->n_tiles, sizeof(double) * RET_NB, sizeof(double) * SPEC_EDGES};
  size_t part_at[6] = {0};
  for (int i = 0; i < 5; ++i) part_at[i + 1] = part_at[i] + up256(part_bytes[i]);
  char* tiles_d = (char*)dalloc(g, part_at[5]);
  if (!tiles_d) return GAP_ENOMEM;
  g->tiles = (Tile*)tiles_d;
  g->ltiles = (LTile*)(tiles_d + part_at[1]);
  g->ptiles = (PTile*)(tiles_d + part_at[2]);
  g->ret_thr = (double*)(tiles_d + part_at[3]);
  g->spec_thr = (double*)(tiles_d + part_at[4]);
  g->rho = (long long*)dalloc(g, sizeof(long long) * g->total_nodes);
  g->rho_last = (long long*)dalloc(g, sizeof(long long) * g->total_nodes);
  g->E = (float*)dalloc(g, sizeof(float) * g->total_cells);
  g->ebar = (float*)dalloc(g, sizeof(float) * g->total_nodes);
  g->fb = (FBlk*)dalloc(g, sizeof(FBlk) * g->n_fb);
  g->part = (long long*)dalloc(g, sizeof(long long) * g->n_fb);
  g->part2 = (long long*)dalloc(g, sizeof(long long) * g->n_fb);
  g->fscan = (unsigned long long*)dalloc(g, sizeof(unsigned long long) * (4 * (size_t)g->n_fb + g->n_tubes));
  if (g->any_filter) {
    g->E0 = (double*)dalloc(g, sizeof(double) * g->total_cells);
    g->Du = (double*)dalloc(g, sizeof(double) * g->total_cells);
    if (!g->E0 || !g->Du) return GAP_ENOMEM;
  }
  g->tab = (float*)dalloc(g, sizeof(float) * 2 * (NTAB + 1));
  char* read_d = (char*)dalloc(g, up256(sizeof(gap_t::Status)) + sizeof(long long) * C_N);
  if (!read_d) return GAP_ENOMEM;
  g->status = (gap_t::Status*)read_d;
  g->err = &g->status->err;
  g->counts = (long long*)(read_d + up256(sizeof(gap_t::Status)));
  g->live = (long long*)dalloc(g, sizeof(long long) * 2 * n_tubes);
  g->shard = (long long*)dalloc(g, sizeof(long long) * n_tubes * NSHARD * C_N);
  if (!g->shard) return GAP_ENOMEM;
  if (!g->tubes || !g->tiles || !g->rho || !g->rho_last || !g->E || !g->ebar || !g->fb || !g->part || !g->part2 || !g->fscan ||
      !g->tab || !g->err || !g->live)
    return GAP_ENOMEM;
  int e;
  if ((e = alloc_store(g, g->lep, cap_l, false))) return e;
  if ((e = alloc_store(g, g->pho, cap_p, true))) return e;
  g->pq_groups = 8 * g->round_pho + 64;   // the autotuner tries grids up to 4 resident rounds
  g->pq = (uint4*)dalloc(g, (size_t)g->pho.capacity * sizeof(uint4));
  g->pq_start = (long long*)dalloc(g, (size_t)g->pq_groups * (sizeof(long long) + sizeof(int)));
  if (!g->pq || !g->pq_start) return GAP_ENOMEM;
  g->pq_count = (int*)(g->pq_start + g->pq_groups);
  g->stage = (uint32_t*)g->pq;
  g->stage_bytes = std::min(kStageBytes, (size_t)g->pho.capacity * sizeof(uint4));
  // at most one entry per slot of the sorted lepton region; a count and a
  // start per workgroup of the largest lepton grid the launch settings allow
  // (4 rounds)
  g->bq = (uint4*)dalloc(g, (size_t)g->lep.capacity * sizeof(uint4));
  g->bq_count = (int*)dalloc(g, (size_t)(4 * g->round_lep + 64) * sizeof(int));
  g->bq_start = (long long*)dalloc(g, (size_t)(4 * g->round_lep + 64) * sizeof(long long));
  if (!g->bq || !g->bq_count || !g->bq_start) return GAP_ENOMEM;
  if (g->any_protons) {
    const size_t n = (size_t)g->pr_cap;
    for (int b = 0; b < 2; ++b) {
      ProBuf& r = g->pr[b];
      r.cell = (int32_t*)dalloc(g, n * 4);
      r.frac = (uint32_t*)dalloc(g, n * 4);
      r.u = (float*)dalloc(g, n * 4);
      r.w = (float*)dalloc(g, n * 4);
      r.id = (uint64_t*)dalloc(g, n * 8);
      r.tube = (int32_t*)dalloc(g, n * 4);
      if (!r.cell || !r.frac || !r.u || !r.w || !r.id || !r.tube) return GAP_ENOMEM;
    }
    g->pr_n = (long long*)dalloc(g, sizeof(long long));
    if (!g->pr_n) return GAP_ENOMEM;
  }
  int max_n = 1;
  for (int t = 0; t < n_tubes; ++t) max_n = std::max(max_n, p[t].n_cells);
  g->ret = (double*)dalloc(g, sizeof(double) * RET_N * (size_t)n_tubes);
  g->spec_acc = (double*)dalloc(g, sizeof(double) * 3 * SPEC_NB);
  if (!g->spec_acc) return GAP_ENOMEM;
  g->prof_acc = (double*)dalloc(g, sizeof(double) * PROF_G * PROF_M * (size_t)max_n);
  g->prof_out = (double*)dalloc(g, sizeof(double) * PROF_G * 3 * (size_t)max_n);
  if (!g->ret || !g->prof_acc || !g->prof_out) return GAP_ENOMEM;
  for (int t = 0; t < n_tubes; ++t) if (g->P[t].flags & GAP_MERGE_ON) g->merge_on = true;
  if (g->merge_on) {
    g->merge_every = std::max(1, g->P[0].merge_every);
    for (int sp = 0; sp < 2; ++sp) {
      SortBuf& sb = sp ? g->sort_p : g->sort_l;
      const size_t n = (size_t)(sp ? g->pho.capacity : g->lep.capacity);
      sb.max_blocks = (int)(n / RS_ITEMS + 1);
      for (int b = 0; b < 2; ++b) {
        sb.major[b] = (uint32_t*)dalloc(g, n * 4);
        sb.id[b] = (uint64_t*)dalloc(g, n * 8);
        sb.val[b] = (uint32_t*)dalloc(g, n * 4);
        if (!sb.major[b] || !sb.id[b] || !sb.val[b]) return GAP_ENOMEM;
      }
      sb.bhist = (uint32_t*)dalloc(g, (size_t)256 * sb.max_blocks * 4);
      sb.dtot = (uint32_t*)dalloc(g, 256 * 4);
      sb.live = (long long*)dalloc(g, sizeof(long long) * n_tubes);
      sb.start = (uint32_t*)dalloc(g, n * 4);
      sb.bmax = (uint32_t*)dalloc(g, (n / MX_ITEMS + 2) * 4);
      sb.flags = (uint32_t*)dalloc(g, (size_t)n_tubes * 4);
      sb.gate = (uint32_t*)dalloc(g, 8);
      sb.n = (long long*)dalloc(g, 8);
      if (!sb.bhist || !sb.dtot || !sb.live || !sb.start || !sb.bmax || !sb.flags || !sb.gate || !sb.n) return GAP_ENOMEM;
    }
    g->thresh_l = (double*)dalloc(g, sizeof(double) * n_tubes);
    g->thresh_p = (double*)dalloc(g, sizeof(double) * n_tubes);
    if (!g->thresh_l || !g->thresh_p) return GAP_ENOMEM;
    std::vector<double> tl(n_tubes), tp(n_tubes);
    for (int t = 0; t < n_tubes; ++t) {
      const bool on = (g->P[t].flags & GAP_MERGE_ON) != 0;
      tl[t] = on ? g->P[t].merge_frac * (double)g->P[t].cap_leptons : 1e300;
      tp[t] = on ? g->P[t].merge_frac * (double)g->P[t].cap_photons : 1e300;
    }
    g->tmin_l = *std::min_element(tl.begin(), tl.end());
    g->tmin_p = *std::min_element(tp.begin(), tp.end());
    HIPCHK(hipStreamSynchronize(g->s));
    HIPCHK(hipMemcpy(g->thresh_l, tl.data(), sizeof(double) * n_tubes, hipMemcpyHostToDevice));
    HIPCHK(hipMemcpy(g->thresh_p, tp.data(), sizeof(double) * n_tubes, hipMemcpyHostToDevice));
  }
  // (every buffer is cleared by a fill on the caller's stream, which a plain
  // copy does not wait for when that stream is a non-blocking one)
  HIPCHK(hipStreamSynchronize(g->s));
  if ((e = upload_tubes(g))) return e;
  {
    // return spectrum, bin b: gamma in [10^(b/8), 10^((b+1)/8)), i.e. u^2 = gamma^2 - 1 from 10^(b/4) - 1;
    // momentum spectra, edge b at 10^(-2 + b/8) in |u| or |x|, compared as squares
    double ret_thr[RET_NB], spec_thr[SPEC_EDGES];
    for (int b = 0; b < RET_NB; ++b) ret_thr[b] = std::pow(10.0, b / 4.0) - 1.0;
    for (int b = 0; b < SPEC_EDGES; ++b) spec_thr[b] = std::pow(10.0, 2.0 * (-2.0 + b / 8.0));
    const void* const part[5] = {g->tiles_h.data(), g->ltiles_h.data(), g->ptiles_h.data(), ret_thr, spec_thr};
    std::vector<char> all(part_at[5]);
    for (int i = 0; i < 5; ++i) std::memcpy(all.data() + part_at[i], part[i], part_bytes[i]);
    HIPCHK(hipMemcpy(g->tiles, all.data(), all.size(), hipMemcpyHostToDevice));
  }
  HIPCHK(hipMemcpy(g->fb, g->fb_h.data(), sizeof(FBlk) * g->n_fb, hipMemcpyHostToDevice));
  const std::vector<float>& tab = sync_table();
  HIPCHK(hipMemcpy(g->tab, tab.data(), sizeof(float) * tab.size(), hipMemcpyHostToDevice));
  if (g->any_quantum && (e = upload_quantum_tables(g))) return e;

  // initial particles into the lepton tail, then sort and solve the field
  std::vector<long long> off(n_tubes + 1, 0);
  std::vector<int32_t> kind(n_tubes), ppc(n_tubes), klo(n_tubes);
  std::vector<float> u0(n_tubes);
  for (int t = 0; t < n_tubes; ++t) {
    off[t + 1] = off[t] + init_count(g->P[t], g->D[t]);
    kind[t] = g->P[t].init_kind;
    ppc[t] = std::max(1, g->P[t].ppc_init);
    klo[t] = (int32_t)init_k_lo(g->P[t], g->D[t]);
    u0[t] = (float)g->P[t].u_init;
    if (init_count(g->P[t], g->D[t]) > g->P[t].cap_leptons) return GAP_ECAP;
  }
  const long long total = off[n_tubes];
  if (total > g->lep.limit) return GAP_ECAP;
  if (total > 0) {
    long long* d_off = (long long*)dalloc(g, sizeof(long long) * (n_tubes + 1));
    int32_t* d_kind = (int32_t*)dalloc(g, 4 * n_tubes);
    int32_t* d_ppc = (int32_t*)dalloc(g, 4 * n_tubes);
    int32_t* d_klo = (int32_t*)dalloc(g, 4 * n_tubes);
    float* d_u0 = (float*)dalloc(g, 4 * n_tubes);
    if (!d_off || !d_kind || !d_ppc || !d_klo || !d_u0) return GAP_ENOMEM;
    HIPCHK(hipStreamSynchronize(g->s));
    HIPCHK(hipMemcpy(d_off, off.data(), sizeof(long long) * (n_tubes + 1), hipMemcpyHostToDevice));
    HIPCHK(hipMemcpy(d_kind, kind.data(), 4 * n_tubes, hipMemcpyHostToDevice));
    HIPCHK(hipMemcpy(d_ppc, ppc.data(), 4 * n_tubes, hipMemcpyHostToDevice));
    HIPCHK(hipMemcpy(d_klo, klo.data(), 4 * n_tubes, hipMemcpyHostToDevice));
    HIPCHK(hipMemcpy(d_u0, u0.data(), 4 * n_tubes, hipMemcpyHostToDevice));
    InitCtx ic;
    ic.tubes = g->tubes;
    ic.tiles = g->tiles;
    ic.L = g->lep.lep(g->lep.cur);
    ic.ltt = g->lep.tt;
    ic.base_slot = 0;
    ic.tube_off = d_off;
    ic.kind = d_kind;
    ic.ppc = d_ppc;
    ic.k_lo = d_klo;
    ic.u0 = d_u0;
    ic.n_tubes = n_tubes;
    k_init_particles<<<kGrid, 256, 0, g->s>>>(ic);
    Ctl c{};
    c.capacity = g->lep.capacity;
    c.limit = g->lep.limit;
    c.cap_live = g->lep.cap_live;
    c.tail = total;
    c.cold_steps = -1;
    HIPCHK(hipMemcpyAsync(g->lep.ctl, &c, sizeof(Ctl), hipMemcpyHostToDevice, g->s));
  }
  if (g->any_protons) {
    // initial protons: ids after each tube's initial electrons
    std::vector<long long> poff(n_tubes + 1, 0);
    std::vector<int32_t> pppc(n_tubes);
    std::vector<int64_t> id0(n_tubes);
    for (int t = 0; t < n_tubes; ++t) {
      poff[t + 1] = poff[t] + init_protons(g->P[t], g->D[t]);
      pppc[t] = std::max(1, g->P[t].ppc_init);
      id0[t] = init_count(g->P[t], g->D[t]) + 1;
    }
    const long long np = poff[n_tubes];
    if (np > g->pr_cap) return GAP_ECAP;
    if (np > 0) {
      long long* d_off = (long long*)dalloc(g, sizeof(long long) * (n_tubes + 1));
      int32_t* d_ppc = (int32_t*)dalloc(g, 4 * n_tubes);
      int64_t* d_id0 = (int64_t*)dalloc(g, 8 * n_tubes);
      if (!d_off || !d_ppc || !d_id0) return GAP_ENOMEM;
      HIPCHK(hipStreamSynchronize(g->s));
      HIPCHK(hipMemcpy(d_off, poff.data(), sizeof(long long) * (n_tubes + 1), hipMemcpyHostToDevice));
      HIPCHK(hipMemcpy(d_ppc, pppc.data(), 4 * n_tubes, hipMemcpyHostToDevice));
      HIPCHK(hipMemcpy(d_id0, id0.data(), 8 * n_tubes, hipMemcpyHostToDevice));
      ProInit pi{g->tubes, g->pr[g->pr_cur], d_off, d_ppc, d_id0, n_tubes};
      k_init_protons<<<kGrid, 256, 0, g->s>>>(pi);
    }
    HIPCHK(hipMemcpyAsync(g->pr_n, &np, sizeof(long long), hipMemcpyHostToDevice, g->s));
    HIPCHK(hipStreamSynchronize(g->s));
  }
  rebucket_all(g);
  rebuild_field(g);
  return sync_and_err(g);
}

// Transform of E zero-padded to M cells; x and y hold M values each, the
// returned one the result.
double2* fft(gap_t* g, const float* E, int N, int M, double2* x, double2* y) {
  const int grid = std::max(1, std::min(1024, (M + 255) / 256));
  k_fft_load<<<grid, 256, 0, g->s>>>(E, N, M, x);
  int Ns = 1;
  for (; 4 * Ns <= M; Ns *= 4) {
    k_fft_stage4<<<grid, 256, 0, g->s>>>(x, y, M, Ns);
    std::swap(x, y);
  }
  if (Ns < M) {                      // M is an odd power of two
    k_fft_stage<<<grid, 256, 0, g->s>>>(x, y, M, Ns);
    std::swap(x, y);
  }
  return x;
}

// The live records of tube `tube` into host_buf in slot order (*need: their
// bytes; nothing is copied when they do not fit).  The pieces are packed in
// the birth queue, which only a step uses, and the blocks' record counts (8 B
// per 1024 slots) stand in the store's classes (1 B per slot), which only a
// re-sort uses: a read allocates nothing.
int export_store(gap_t* g, bool photon, int tube, void* host_buf, size_t buf_bytes, size_t* need) {
  RecCtx r;
  r.cx = make_ctx(g);
  r.tube = tube;
  r.n_tiles = g->n_tiles;
  r.lep = photon ? 0 : 1;
  r.count = (int64_t*)(photon ? g->pho : g->lep).cls;
  r.total = g->counts;
  k_rec_count<<<kGrid, TPB, 0, g->s>>>(r);
  k_rec_scan<<<1, REC_SCAN_T, 0, g->s>>>(r);
  long long n = 0;
  int e = read_back(g, g->counts, sizeof(n), &n);
  if (e) return e;
  const size_t rs = photon ? REC_PHO : REC_LEP;
  *need = rs * (size_t)n;
  if (*need > buf_bytes) return GAP_OK;
  const long long piece = (long long)(g->lep.capacity * sizeof(uint4) / REC_PHO);
  for (long long lo = 0; lo < n; lo += piece) {
    const long long hi = std::min(n, lo + piece);
    k_rec_pack<<<kGrid, TPB, 0, g->s>>>(r, lo, hi, (uint2*)g->bq);
    HIPCHK(hipMemcpyAsync((char*)host_buf + rs * (size_t)lo, g->bq, rs * (size_t)(hi - lo), hipMemcpyDeviceToHost, g->s));
  }
  HIPCHK(hipStreamSynchronize(g->s));
  return hipGetLastError() == hipSuccess ? GAP_OK : GAP_EDEVICE;
}

int graph_capture(gap_t* g, int64_t n) {
  drop_graph(g);
  g->graph_fused = fused_form(g);
  g->gs_l = g->lep.cur; g->gs_p = g->pho.cur; g->gs_r = g->pr_cur; g->gs_since = g->since_rb; g->gs_step = g->host_step;
  const int rb_seen = g->rb_seen;
  hipGraph_t graph = nullptr;
  HIPCHK(hipStreamBeginCapture(g->s, hipStreamCaptureModeThreadLocal));
  g->rb_seen = 0;
  g->capturing = true;
  for (int64_t i = 0; i < n; ++i) enqueue_step(g, i + 1 < n);
  g->capturing = false;
  hipError_t e = hipStreamEndCapture(g->s, &graph);
  g->ge_l = g->lep.cur; g->ge_p = g->pho.cur; g->ge_r = g->pr_cur; g->ge_since = g->since_rb;
  g->graph_rb = g->rb_seen;
  g->graph_form = g->form;
  // nothing ran yet: back to the start state
  g->lep.cur = g->gs_l; g->pho.cur = g->gs_p; g->pr_cur = g->gs_r; g->since_rb = g->gs_since; g->host_step = g->gs_step;
  g->rb_seen = rb_seen;
  if (e != hipSuccess) return GAP_EDEVICE;
  e = hipGraphInstantiate(&g->gexec, graph, nullptr, nullptr, 0);
  (void)hipGraphDestroy(graph);
  if (e != hipSuccess) { g->gexec = nullptr; return GAP_EDEVICE; }
  g->gsteps = n;
  return GAP_OK;
}

// ------------------------------------------------------------------ autotuner
// Launch shapes and the re-sort interval change no result (the deposit is in
// integers and every particle's arithmetic is independent of the grid and of
// its slot), so candidates are timed on real steps of the simulation, in the
// form that the handle's steps take.
int timed_steps(gap_t* g, int64_t n, double* kt, double* wall_ms) {
  g->ev_marks.clear();
  g->ev_used = 0;
  hipEvent_t a = next_event(g), b = next_event(g);
  if (!a || !b) return GAP_EDEVICE;
  HIPCHK(hipEventRecord(a, g->s));
  for (int64_t i = 0; i < n; ++i) enqueue_step(g, i + 1 < n);
  join_photon_side(g);
  HIPCHK(hipEventRecord(b, g->s));
  HIPCHK(hipEventSynchronize(b));
  float ms = 0.0f;
  HIPCHK(hipEventElapsedTime(&ms, a, b));
  *wall_ms = ms;
  for (int i = 0; i < KT_N; ++i) kt[i] = 0.0;
  for (auto& m : g->ev_marks) {
    float t = 0.0f;
    HIPCHK(hipEventElapsedTime(&t, m.second.first, m.second.second));
    kt[m.first] += t;
  }
  g->ev_marks.clear();
  g->ev_used = 0;
  return read_err(g);
}

int autotune(gap_t* g, int trial, int32_t* chosen) {
  struct Timing {                     // (kernel timing as it was, however the search ends)
    gap_t* g;
    const bool was = g->timing;
    ~Timing() { g->timing = was; }
  } timing{g};
  g->timing = true;
  g->grid_lep_set = true;
  drop_graph(g);
  double kt[KT_N], wall;
  int e;
  auto cands = [](int round, int lo) {
    std::vector<int> v;
    for (int m : {1, 2, 4, 8}) v.push_back(std::max(lo, (round * m / 2) / 8 * 8));
    return v;
  };
  struct Knob { int* grid; std::vector<int> c; };
  Knob knobs[3] = {{&g->grid_lep, cands(g->round_lep, 8)},
                   {&g->grid_pho, cands(g->round_pho, 8)},
                   {&g->grid_tail, {g->cus * 2, g->cus * 4, g->cus * 8, g->cus * 16}}};
  if ((e = timed_steps(g, trial, kt, &wall))) return e;   // warm-up
  for (Knob& k : knobs) {
    double best = 1e300;
    int arg = *k.grid;
    // the passes of the two species overlap on two streams: the measure is
    // the steps' wall time, less the re-sorts that fall into the trial, the
    // better of two rounds over the candidates
    std::vector<double> tbest(k.c.size(), 1e300);
    for (int round = 0; round < 2; ++round) {
      for (size_t ci = 0; ci < k.c.size(); ++ci) {
        *k.grid = k.c[ci];
        if ((e = timed_steps(g, trial, kt, &wall))) return e;
        tbest[ci] = std::min(tbest[ci], wall - kt[KT_RESORT]);
      }
    }
    for (size_t ci = 0; ci < k.c.size(); ++ci)
      if (tbest[ci] < best) { best = tbest[ci]; arg = k.c[ci]; }
    *k.grid = arg;
  }
  // re-sort interval: whole steps, each candidate over at least two re-sorts
  {
    std::vector<int> rc;
    for (int r : {g->R / 4, g->R / 2, g->R, g->rmax}) {
      r = std::max(4, std::min(r, g->rmax));
      if (std::find(rc.begin(), rc.end(), r) == rc.end()) rc.push_back(r);
    }
    double best = 1e300;
    int arg = g->R;
    for (int r : rc) {
      // the count of steps since the last re-sort carries over (a shorter
      // interval re-sorts at once): the drift bound of the tile margin holds
      // only for steps actually counted since a re-sort
      g->R = r;
      const int64_t n = std::max<int64_t>(trial, 2 * (int64_t)r);
      if ((e = timed_steps(g, n, kt, &wall))) return e;
      const double per = wall / (double)n;
      if (per < best) { best = per; arg = r; }
    }
    g->R = arg;
  }
  chosen[0] = g->grid_lep;
  chosen[1] = g->grid_pho;
  chosen[2] = g->grid_tail;
  chosen[3] = g->R;
  return g->sticky;
}

}  // namespace

// ====================================================================== C ABI
// Host allocations (staging, tables, records) may fail: no exception crosses
// the ABI.
#define GAP_NO_THROW catch (...) { return GAP_ENOMEM; }

extern "C" {

int gap_init(const gap_params* p, int32_t n_tubes, void* stream, const gap_allocator* alloc, gap_t** out) {
  if (!p || !out || n_tubes < 1) return GAP_EINVAL;
  *out = nullptr;
  for (int t = 0; t < n_tubes; ++t) {
    int e = validate(p[t]);
    if (e) return e;
  }
  if (alloc && (!alloc->alloc || !alloc->free)) return GAP_EINVAL;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) return GAP_EDEVICE;
  gap_t* g = new (std::nothrow) gap_t();
  if (!g) return GAP_ENOMEM;
  g->s = (hipStream_t)stream;
  {
    // this device's address of the static workspace, taken once per device
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || !(g->scratch = scratch_on_device(dev))) {
      delete g;
      return GAP_EDEVICE;
    }
  }
  // default priority, like every stream of the library; the events order the two
  // streams on this device only, so they need no system-scope fence
  constexpr unsigned kSyncEvent = hipEventDisableTiming | hipEventDisableSystemFence;
  if (hipStreamCreateWithFlags(&g->s2, hipStreamNonBlocking) != hipSuccess ||
      hipEventCreateWithFlags(&g->ev_l, kSyncEvent) != hipSuccess ||
      hipEventCreateWithFlags(&g->ev_pre, kSyncEvent) != hipSuccess ||
      hipEventCreateWithFlags(&g->ev_p, kSyncEvent) != hipSuccess ||
      hipEventCreateWithFlags(&g->ev_f, kSyncEvent) != hipSuccess ||
      hipEventCreateWithFlags(&g->ev_j, kSyncEvent) != hipSuccess) {
    release(g);
    delete g;
    return GAP_EDEVICE;
  }
  if (alloc) { g->al = *alloc; g->custom_alloc = true; }
  int e;
  try { e = build(g, p, n_tubes); } catch (...) { e = GAP_ENOMEM; }
  if (e) {
    release(g);
    delete g;
    return e;
  }
  *out = g;
  return GAP_OK;
}

int gap_step(gap_t* g, int64_t n_steps) try {
  if (!g || n_steps < 0) return GAP_EINVAL;
  if (g->sticky) return g->sticky;   // a reported error stops the run
  for (int64_t i = 0; i < n_steps; ++i) enqueue_step(g, i + 1 < n_steps);
  join_photon_side(g);   // the caller's stream holds all the work again
  if (hipGetLastError() != hipSuccess) return GAP_EDEVICE;
  return g->sticky;
} GAP_NO_THROW

int gap_step_graph(gap_t* g, int64_t n_steps) try {
  if (!g || n_steps < 0) return GAP_EINVAL;
  if (n_steps == 0 || g->sticky) return g->sticky;
  if (g->s == nullptr) return GAP_ESTATE;   // stream capture needs a non-default stream
  join_photon_side(g);
  const bool valid = g->gexec && g->gsteps == n_steps && g->lep.cur == g->gs_l && g->pho.cur == g->gs_p &&
                     g->pr_cur == g->gs_r &&
                     g->since_rb == g->gs_since &&
                     !(g->graph_fused && g->seen_p > FUSED_PHO_CHUNKS) &&
                     (!g->merge_on || (g->host_step - g->gs_step) % g->merge_every == 0);
  if (!valid) {
    int e = graph_capture(g, n_steps);
    if (e) return e;
  }
  HIPCHK(hipGraphLaunch(g->gexec, g->s));
  g->lep.cur = g->ge_l; g->pho.cur = g->ge_p; g->pr_cur = g->ge_r; g->since_rb = g->ge_since;
  g->host_step += n_steps;
  count_resorts(g, g->graph_rb);
  g->form = g->graph_form;
  return g->sticky;
} GAP_NO_THROW

int gap_sync(gap_t* g) {
  if (!g) return GAP_EINVAL;
  return sync_and_err(g);
}

int gap_diag(gap_t* g, int32_t kind, int32_t tube, void* host_buf, size_t buf_bytes, size_t* bytes_written) try {
  if (!g || tube < 0 || tube >= g->n_tubes || (!host_buf && buf_bytes)) return GAP_EINVAL;
  int e = GAP_OK;
  // (the other kinds wait where they read)
  if (kind == GAP_DIAG_LEPTONS || kind == GAP_DIAG_PHOTONS || kind == GAP_DIAG_PROTONS || kind == GAP_DIAG_RETURN ||
      kind == GAP_DIAG_WATERFALL || kind == GAP_DIAG_TIMING || kind == GAP_DIAG_LAUNCH ||
      kind == GAP_DIAG_FORM || kind == GAP_DIAG_DERIVED) {
    e = sync_and_err(g);
    if (e == GAP_EDEVICE) return e;
  }
  const Tube& Th = g->th[tube];
  const int N = g->P[tube].n_cells;
  size_t need = 0;
  auto fits = [&](size_t n) {
    need = n;
    if (bytes_written) *bytes_written = n;
    return n <= buf_bytes;
  };
  // a read that is refused waits and takes notice of errors like any other
  auto refused = [&]() { return sync_and_err(g) == GAP_EDEVICE ? GAP_EDEVICE : GAP_EINVAL; };
  switch (kind) {
    case GAP_DIAG_COUNTS: {
      if (!fits(sizeof(int64_t) * 32)) return refused();
      k_fill_i64<<<1, 256, 0, g->s>>>(g->live, 2 * g->n_tubes, 0);
      k_count_live<LepBuf><<<kGrid, TPB, 0, g->s>>>(g->lep.lep(g->lep.cur), g->lep.ctl, g->lep.chunk[g->lep.cur], g->lep.tt,
                                                  g->tiles, g->live, g->n_tubes);
      k_count_live<PhoBuf><<<kGrid, TPB, 0, g->s>>>(g->pho.pho(g->pho.cur), g->pho.ctl, g->pho.chunk[g->pho.cur], g->pho.tt,
                                                  g->tiles, g->live + g->n_tubes, g->n_tubes);
      k_counts<<<1, 64, 0, g->s>>>(g->tubes, tube, g->n_tubes, g->shard, g->live, g->counts);
      if ((e = read_back(g, g->counts, sizeof(int64_t) * 32, host_buf))) return e;
      int64_t* o = (int64_t*)host_buf;
      o[GAP_C_ERR] = g->sticky;
      return GAP_OK;
    }
    case GAP_DIAG_FIELD:
      if (!fits(sizeof(float) * N)) return refused();
      return read_back(g, g->E + Th.cell_off, sizeof(float) * N, host_buf);
    case GAP_DIAG_NODE_E:
      if (!fits(sizeof(float) * (N + 1))) return refused();
      return read_back(g, g->ebar + Th.node_off, sizeof(float) * (N + 1), host_buf);
    case GAP_DIAG_RHO:
      if (!fits(sizeof(int64_t) * (N + 1))) return refused();
      return read_back(g, g->rho_last + Th.node_off, sizeof(int64_t) * (N + 1), host_buf);
    case GAP_DIAG_ES:
      if (!fits(sizeof(double))) return refused();
      return read_back(g, &g->tubes[tube].Es, sizeof(double), host_buf);
    case GAP_DIAG_PROFILE:
    case GAP_DIAG_PEAK: {
      const int B = g->prof_bin;
      const int nb = (N + B - 1) / B;
      if (kind == GAP_DIAG_PROFILE ? !fits(sizeof(double) * 3 * PROF_G * (size_t)nb) : !fits(sizeof(double) * 6))
        return refused();
      const long long nacc = (long long)nb * PROF_G * PROF_M;
      k_fill_i64<<<std::max(1, (int)std::min<long long>(1024, (nacc + 255) / 256)), 256, 0, g->s>>>(
          (long long*)g->prof_acc, nacc, 0);
      k_profile<<<kDiagGrid, TPB, 0, g->s>>>(make_ctx(g), tube, B, nb, g->prof_acc);
      const double bppc = (double)B * (double)g->P[tube].ppc_ref;
      if (kind == GAP_DIAG_PROFILE) {
        k_profile_finish<<<std::max(1, std::min(1024, (nb * PROF_G + 255) / 256)), 256, 0, g->s>>>(g->prof_acc, nb,
                                                                                                 bppc, g->prof_out);
        if ((e = read_back(g, g->prof_out, sizeof(double) * 3 * PROF_G * (size_t)nb, host_buf))) return e;
      } else {
        k_profile_peak<<<1, PEAK_T, 0, g->s>>>(g->prof_acc, nb, B, g->P[tube].dx, g->D[tube].H, bppc,
                                            g->E + Th.cell_off, N, g->prof_out);
        if ((e = read_back(g, g->prof_out, sizeof(double) * 6, host_buf))) return e;
      }
      return g->sticky;
    }
    case GAP_DIAG_RETURN: {
      // double[RET_N]; reading resets the tube's record
      if (!fits(sizeof(double) * RET_N)) return GAP_EINVAL;
      double* r = g->ret + (size_t)tube * RET_N;
      HIPCHK(hipMemcpy(host_buf, r, sizeof(double) * RET_N, hipMemcpyDeviceToHost));
      k_fill_i64<<<1, 256, 0, g->s>>>((long long*)r, RET_N, 0);
      return sync_and_err(g);
    }
    case GAP_DIAG_WATERFALL: {
      // int64 n, int64 nb, n step indices (ascending), n x nb doubles;
      // reading empties the tube's ring
      if (g->wf_every <= 0) return GAP_ESTATE;
      const int nb = (N + g->wf_B - 1) / g->wf_B;
      std::vector<long long> st((size_t)g->wf_cap);
      HIPCHK(hipMemcpy(st.data(), g->wf_steps + (size_t)tube * g->wf_cap, sizeof(long long) * st.size(),
                       hipMemcpyDeviceToHost));
      std::vector<int> order;
      for (int i = 0; i < g->wf_cap; ++i) if (st[i] >= 0) order.push_back(i);
      std::sort(order.begin(), order.end(), [&](int a, int b) { return st[a] < st[b]; });
      const size_t n = order.size();
      if (!fits(sizeof(long long) * (2 + n) + sizeof(double) * n * (size_t)nb)) return GAP_EINVAL;
      std::vector<double> ring((size_t)g->wf_cap * g->wf_nbmax);
      HIPCHK(hipMemcpy(ring.data(), g->wf_ring + (size_t)tube * g->wf_cap * g->wf_nbmax, sizeof(double) * ring.size(),
                       hipMemcpyDeviceToHost));
      long long* h = (long long*)host_buf;
      h[0] = (long long)n;
      h[1] = nb;
      double* v = (double*)(h + 2 + n);
      for (size_t j = 0; j < n; ++j) {
        h[2 + j] = st[order[j]];
        std::memcpy(v + j * nb, ring.data() + (size_t)order[j] * g->wf_nbmax, sizeof(double) * nb);
      }
      k_fill_i64<<<1, 256, 0, g->s>>>(g->wf_steps + (size_t)tube * g->wf_cap, g->wf_cap, -1);
      return sync_and_err(g);
    }
    case GAP_DIAG_PHASE: {
      // double[3][nb][180], nb bins of the profile's bin width
      const int B = g->prof_bin;
      const int nb = (N + B - 1) / B;
      const size_t n = (size_t)3 * nb * PHASE_NP;
      if (!fits(sizeof(double) * n)) return refused();
      if (g->phase_cap < n) {
        g->phase_acc = (double*)dalloc(g, sizeof(double) * n);   // kept until the handle ends
        if (!g->phase_acc) return GAP_ENOMEM;
        g->phase_cap = n;
      }
      k_fill_i64<<<std::max(1, (int)std::min<size_t>(1024, (n + 255) / 256)), 256, 0, g->s>>>(
          (long long*)g->phase_acc, (long long)n, 0);
      const int lw = phase_window(B);
      k_phase<<<kDiagGrid, TPB, sizeof(double) * 2 * lw * PHASE_NP, g->s>>>(make_ctx(g), tube, B, nb, g->spec_thr,
                                                                           g->phase_acc, lw);
      if ((e = read_back(g, g->phase_acc, sizeof(double) * n, host_buf))) return e;
      return g->sticky;
    }
    case GAP_DIAG_SPECTRA: {
      if (!fits(sizeof(double) * 3 * SPEC_NB)) return refused();
      k_fill_i64<<<1, 256, 0, g->s>>>((long long*)g->spec_acc, 3 * SPEC_NB, 0);
      k_spectra<<<kDiagGrid, TPB, 0, g->s>>>(make_ctx(g), tube, g->spec_thr, g->spec_acc);
      if ((e = read_back(g, g->spec_acc, sizeof(double) * 3 * SPEC_NB, host_buf))) return e;
      return g->sticky;
    }
    case GAP_DIAG_ESPECTRUM: {
      // double[M/2 + 1], M the next power of two >= N
      int M = 1;
      while (M < N) M *= 2;
      if (!fits(sizeof(double) * (size_t)(M / 2 + 1))) return refused();
      if (!g->fft_buf) {
        int Mmax = 1;
        while (Mmax < g->max_cells) Mmax *= 2;
        g->fft_buf = (double2*)dalloc(g, sizeof(double2) * 2 * (size_t)Mmax);
        g->fft_pow = (double*)dalloc(g, sizeof(double) * ((size_t)Mmax / 2 + 1));
        if (!g->fft_buf || !g->fft_pow) return GAP_ENOMEM;
      }
      const int grid = std::max(1, std::min(1024, (M + 255) / 256));
      const double2* x = fft(g, g->E + Th.cell_off, N, M, g->fft_buf, g->fft_buf + M);
      k_fft_power<<<grid, 256, 0, g->s>>>(x, M, g->fft_pow);
      if ((e = read_back(g, g->fft_pow, sizeof(double) * (size_t)(M / 2 + 1), host_buf))) return e;
      return g->sticky;
    }
    case GAP_DIAG_TIMING: {
      // double[2 * KT_N]: launches and summed milliseconds per kernel group
      if (!fits(sizeof(double) * 2 * KT_N)) return GAP_EINVAL;
      double* o = (double*)host_buf;
      for (int i = 0; i < 2 * KT_N; ++i) o[i] = 0.0;
      for (auto& m : g->ev_marks) {
        float ms = 0.0f;
        HIPCHK(hipEventElapsedTime(&ms, m.second.first, m.second.second));
        o[2 * m.first] += 1.0;
        o[2 * m.first + 1] += ms;
      }
      g->ev_marks.clear();
      g->ev_used = 0;
      return GAP_OK;
    }
    case GAP_DIAG_LAUNCH: {
      if (!fits(sizeof(int32_t) * 4)) return GAP_EINVAL;
      const int32_t v[4] = {lepton_grid(g), g->grid_pho, g->grid_tail, g->R};
      std::memcpy(host_buf, v, sizeof(v));
      return GAP_OK;
    }
    case GAP_DIAG_FORM: {
      if (!fits(sizeof(int32_t))) return GAP_EINVAL;
      const int32_t v = g->form;
      std::memcpy(host_buf, &v, sizeof(v));
      return GAP_OK;
    }
    case GAP_DIAG_DERIVED: {
      if (!fits(sizeof(double) * 8)) return GAP_EINVAL;
      const Derived& d = g->D[tube];
      double v[8] = {d.d_cm, d.lam, d.rc, d.dt, d.H, d.w0, d.s_co, (double)d.N};
      std::memcpy(host_buf, v, sizeof(v));
      return GAP_OK;
    }
    case GAP_DIAG_PROTONS: {
      std::vector<char> recs;
      if (g->any_protons) {
        long long n = 0;
        HIPCHK(hipMemcpy(&n, g->pr_n, sizeof(long long), hipMemcpyDeviceToHost));
        n = std::min<long long>(n, g->pr_cap);
        const ProBuf& R = g->pr[g->pr_cur];
        std::vector<int32_t> cell(n), tb(n);
        std::vector<uint32_t> frac(n);
        std::vector<float> u(n), w(n);
        std::vector<uint64_t> id(n);
        if (n > 0) {
          HIPCHK(hipMemcpy(cell.data(), R.cell, 4 * n, hipMemcpyDeviceToHost));
          HIPCHK(hipMemcpy(frac.data(), R.frac, 4 * n, hipMemcpyDeviceToHost));
          HIPCHK(hipMemcpy(u.data(), R.u, 4 * n, hipMemcpyDeviceToHost));
          HIPCHK(hipMemcpy(w.data(), R.w, 4 * n, hipMemcpyDeviceToHost));
          HIPCHK(hipMemcpy(id.data(), R.id, 8 * n, hipMemcpyDeviceToHost));
          HIPCHK(hipMemcpy(tb.data(), R.tube, 4 * n, hipMemcpyDeviceToHost));
        }
        for (long long i = 0; i < n; ++i) {
          if (w[i] == 0.0f || tb[i] != tube) continue;
          char r[24];
          std::memcpy(r, &cell[i], 4);
          std::memcpy(r + 4, &frac[i], 4);
          std::memcpy(r + 8, &u[i], 4);
          std::memcpy(r + 12, &w[i], 4);
          std::memcpy(r + 16, &id[i], 8);
          recs.insert(recs.end(), r, r + 24);
        }
      }
      if (!fits(recs.size())) return GAP_EINVAL;
      if (!recs.empty()) std::memcpy(host_buf, recs.data(), recs.size());
      return GAP_OK;
    }
    case GAP_DIAG_LEPTONS:
    case GAP_DIAG_PHOTONS: {
      size_t n = 0;
      if ((e = export_store(g, kind == GAP_DIAG_PHOTONS, tube, host_buf, buf_bytes, &n))) return e;
      return fits(n) ? GAP_OK : GAP_EINVAL;
    }
    default:
      (void)need;
      return refused();
  }
} GAP_NO_THROW

int gap_set_state(gap_t* g, int32_t kind, int32_t tube, const void* host_buf, size_t bytes) try {
  if (!g || !host_buf || tube < 0 || tube >= g->n_tubes) return GAP_EINVAL;
  if (kind == GAP_STATE_TIMING) {
    if (bytes < 4) return GAP_EINVAL;
    int32_t on;
    std::memcpy(&on, host_buf, 4);
    g->timing = g->apart = on != 0;
    g->ev_marks.clear();
    g->ev_used = 0;
    return GAP_OK;
  }
  if (kind == GAP_STATE_PROFILE_BIN) {
    if (bytes < 4) return GAP_EINVAL;
    int32_t b;
    std::memcpy(&b, host_buf, 4);
    if (b < 1) return GAP_EINVAL;
    g->prof_bin = b;
    return GAP_OK;
  }
  if (kind == GAP_STATE_WATERFALL) {
    if (bytes < 12) return GAP_EINVAL;
    int32_t v[3];
    std::memcpy(v, host_buf, 12);
    if (v[0] < 0 || (v[0] > 0 && (v[1] < 1 || v[2] < 1 || v[2] > (1 << 16)))) return GAP_EINVAL;
    // a captured graph holds the old record launch (or none): drop it
    drop_graph(g);
    join_photon_side(g);
    HIPCHK(hipStreamSynchronize(g->s));
    wf_release(g);
    if (v[0] == 0) return GAP_OK;
    int max_n = 1;
    for (int t = 0; t < g->n_tubes; ++t) max_n = std::max(max_n, g->P[t].n_cells);
    const int nbmax = (max_n + v[1] - 1) / v[1];
    const size_t nrec = (size_t)g->n_tubes * (size_t)v[2];
    auto get = [&](size_t bytes) -> void* {
      bytes = (bytes + 255) & ~(size_t)255;
      g->wf_mem.push_back(nullptr);
      void* p = nullptr;
      if (g->custom_alloc) p = g->al.alloc(bytes, g->al.ctx);
      else if (hipMalloc(&p, bytes) != hipSuccess) p = nullptr;
      if (p) g->wf_mem.back() = p;
      else g->wf_mem.pop_back();
      return p;
    };
    g->wf_ring = (double*)get(sizeof(double) * nrec * (size_t)nbmax);
    g->wf_steps = (long long*)get(sizeof(long long) * nrec);
    if (!g->wf_ring || !g->wf_steps) {
      wf_release(g);
      return GAP_ENOMEM;
    }
    k_fill_i64<<<std::max(1, (int)std::min<size_t>(1024, (nrec + 255) / 256)), 256, 0, g->s>>>(g->wf_steps,
                                                                                               (long long)nrec, -1);
    g->wf_every = v[0];
    g->wf_B = v[1];
    g->wf_cap = v[2];
    g->wf_nbmax = nbmax;
    return sync_and_err(g);
  }
  if (kind == GAP_STATE_RAISE) {
    // the device error word as a kernel sets it (tests of the error path)
    if (bytes < 4) return GAP_EINVAL;
    int32_t bits;
    std::memcpy(&bits, host_buf, 4);
    if (bits & ~(E_CAP | E_TILE | E_NAN | E_SCAN)) return GAP_EINVAL;
    k_raise<<<1, 1, 0, g->s>>>(g->err, bits);
    return GAP_OK;
  }
  if (kind == GAP_STATE_LAUNCH) {
    if (bytes < 16) return GAP_EINVAL;
    int32_t v[4];
    std::memcpy(v, host_buf, 16);
    auto grid_ok = [](int x, int round) { return x >= 8 && x % 8 == 0 && x <= 4 * round; };
    if (!grid_ok(v[0], g->round_lep) || !grid_ok(v[1], g->round_pho) || !grid_ok(v[2], 16 * g->cus / 4) ||
        v[3] < 1 || v[3] > g->rmax)
      return GAP_EINVAL;
    g->grid_lep = v[0];
    g->grid_lep_set = true;
    g->grid_pho = v[1];
    g->grid_tail = v[2];
    g->R = v[3];
    drop_graph(g);
    return GAP_OK;
  }
  g->win.valid = false;     // any other state change ends a pending window
  // and the photon store's cold guarantee (a tube's step or parameters may
  // change); the next re-sort restores it
  k_cold_off<<<1, 1, 0, g->s>>>(g->pho.ctl);
  if (kind == GAP_STATE_DRIVE) {
    if (bytes < 16) return GAP_EINVAL;
    double v[2];
    std::memcpy(v, host_buf, 16);
    if (!std::isfinite(v[0]) || !(v[1] > 0) || v[1] >= 65536.0) return GAP_EINVAL;
    int e = sync_and_err(g);
    if (e == GAP_EDEVICE) return e;
    if ((e = download_tubes(g))) return e;
    gap_params& q = g->P[tube];
    Tube& T = g->th[tube];
    q.alpha = v[0];
    q.inj_weight = v[1];
    T.drive = q.alpha * g->D[tube].s_co * g->D[tube].dt;
    T.inj_w = (float)q.inj_weight;
    T.inj_T = std::llrint((double)T.inj_w * kTwo24);
    T.inj_per_step = q.inj_rate * q.ppc_ref / ((q.flags & GAP_INJ_FIXED) ? 1.0 : q.inj_weight);
    if ((e = upload_tubes(g))) return e;
    g->win.valid = false;
    return GAP_OK;
  }
  if (g->n_tubes != 1) return GAP_ESTATE;
  int e = sync_and_err(g);
  if (e == GAP_EDEVICE) return e;
  if ((e = download_tubes(g))) return e;
  Tube& T = g->th[0];
  const gap_params& q = g->P[0];
  const int N = q.n_cells;
  const bool frozen = (q.flags & GAP_FIELD_FROZEN) != 0;
  const char* b = (const char*)host_buf;
  switch (kind) {
    case GAP_STATE_PARTICLES: {
      if (bytes < 16) return GAP_EINVAL;
      int64_t nl, np;
      std::memcpy(&nl, b, 8);
      std::memcpy(&np, b + 8, 8);
      if (nl < 0 || np < 0 || bytes < 16 + (size_t)nl * 24 + (size_t)np * 32) return GAP_EINVAL;
      if (nl > g->lep.limit || np > g->pho.limit) return GAP_ECAP;
      // every record is looked at before anything changes
      for (int sp = 0; sp < 2; ++sp) {
        const bool ph = sp == 1;
        const size_t rs = ph ? REC_PHO : REC_LEP;
        const char* r = ph ? b + 16 + nl * REC_LEP : b + 16;
        for (int64_t i = 0; i < (ph ? np : nl); ++i, r += rs) {
          int32_t cell; uint32_t frac; float mark;
          std::memcpy(&cell, r, 4);
          std::memcpy(&frac, r + 4, 4);
          std::memcpy(&mark, r + (ph ? 8 : 12), 4);
          if (cell < 0 || cell >= N || frac >= (1u << FRAC) || mark == 0.0f) return GAP_EINVAL;
        }
      }
      for (int sp = 0; sp < 2; ++sp) {
        const bool ph = sp == 1;
        Store& st = ph ? g->pho : g->lep;
        const int64_t n = ph ? np : nl;
        const char* r = ph ? b + 16 + nl * REC_LEP : b + 16;
        const size_t rs = ph ? REC_PHO : REC_LEP;
        const int64_t piece = (int64_t)(g->lep.capacity * sizeof(uint4) / REC_PHO);
        for (int64_t lo = 0; lo < n; lo += piece) {
          const int64_t m = std::min(n - lo, piece);
          HIPCHK(hipMemcpyAsync(g->bq, r + rs * (size_t)lo, rs * (size_t)m, hipMemcpyHostToDevice, g->s));
          k_rec_unpack<<<(int)std::min<int64_t>(kGrid, (m + TPB - 1) / TPB), TPB, 0, g->s>>>(
              make_ctx(g), ph ? 0 : 1, T.tile_first, (const uint2*)g->bq, lo, m);
        }
        HIPCHK(hipStreamSynchronize(g->s));
        Ctl cc = read_ctl(st);
        cc.n_sorted_chunks = 0;
        cc.tail = n;
        cc.tail_snap = 0;
        HIPCHK(hipMemcpy(st.ctl, &cc, sizeof(Ctl), hipMemcpyHostToDevice));
      }
      T.dq = 0;
      T.dcur = 0;
      atm_reset(T);
      if ((e = upload_tubes(g))) return e;
      rebucket_all(g);
      g->since_rb = 0;
      if (frozen) {
        const int grid = std::max(1, (int)std::min<long long>(1024, (g->total_nodes + 255) / 256));
        k_fill_i64<<<grid, 256, 0, g->s>>>(g->rho, g->total_nodes, 0);
        k_deposit_all<<<kGrid, TPB, 0, g->s>>>(make_ctx(g));
        if (g->any_protons) k_deposit_protons<<<kGrid, TPB, 0, g->s>>>(make_ctx(g));
        // keep E: only record the node charge
        FieldCtx f = make_fctx(g, 1);
        k_field_a<<<g->n_fb, FB_THREADS, 0, g->s>>>(f);
        k_field_b<<<g->n_fb, FB_THREADS, 0, g->s>>>(f);
      } else {
        rebuild_field(g);
      }
      return sync_and_err(g);
    }
    case GAP_STATE_ES_STEP: {
      if (bytes < 16) return GAP_EINVAL;
      std::memcpy(&T.Es, b, 8);
      std::memcpy(&T.step, b + 8, 8);
      g->host_step = T.step;
      atm_reset(T);
      if ((e = upload_tubes(g))) return e;
      if (!frozen) rebuild_field(g);
      return sync_and_err(g);
    }
    case GAP_STATE_FIELD: {
      if (bytes < sizeof(float) * N + 8) return GAP_EINVAL;
      std::vector<float> E(N);
      std::memcpy(E.data(), b, sizeof(float) * N);
      std::memcpy(&T.Es, b + sizeof(float) * N, 8);
      std::vector<float> eb(N + 1);
      if (q.flags & GAP_PERIODIC) {
        for (int i = 0; i < N; ++i) eb[i] = (float)(0.5 * ((double)E[(i + N - 1) % N] + (double)E[i]));
        eb[N] = eb[0];
      } else {
        eb[0] = (float)(0.5 * (T.Es + (double)E[0]));
        for (int i = 1; i < N; ++i) eb[i] = (float)(0.5 * ((double)E[i - 1] + (double)E[i]));
        eb[N] = E[N - 1];
      }
      HIPCHK(hipMemcpy(g->E + T.cell_off, E.data(), sizeof(float) * N, hipMemcpyHostToDevice));
      HIPCHK(hipMemcpy(g->ebar + T.node_off, eb.data(), sizeof(float) * (N + 1), hipMemcpyHostToDevice));
      if (q.flags & GAP_FILTER) {
        // the set field is the filtered update's new reference
        std::vector<double> e0(E.begin(), E.end());
        HIPCHK(hipMemcpy(g->E0 + T.cell_off, e0.data(), sizeof(double) * N, hipMemcpyHostToDevice));
      }
      if ((e = upload_tubes(g))) return e;
      return sync_and_err(g);
    }
    case GAP_STATE_PROTONS: {
      if (!g->any_protons) return GAP_ESTATE;
      if (bytes < 8) return GAP_EINVAL;
      int64_t n;
      std::memcpy(&n, b, 8);
      if (n < 0 || bytes < 8 + (size_t)n * 24) return GAP_EINVAL;
      if (n > g->pr_cap) return GAP_ECAP;
      std::vector<int32_t> cell(n), tb(n, 0);
      std::vector<uint32_t> frac(n);
      std::vector<float> u(n), w(n);
      std::vector<uint64_t> id(n);
      const char* r = b + 8;
      for (int64_t i = 0; i < n; ++i, r += 24) {
        std::memcpy(&cell[i], r, 4);
        std::memcpy(&frac[i], r + 4, 4);
        std::memcpy(&u[i], r + 8, 4);
        std::memcpy(&w[i], r + 12, 4);
        std::memcpy(&id[i], r + 16, 8);
        if (cell[i] < 0 || cell[i] >= N || frac[i] >= (1u << FRAC) || !(w[i] != 0.0f)) return GAP_EINVAL;
      }
      const ProBuf& R = g->pr[g->pr_cur];
      if (n > 0) {
        HIPCHK(hipMemcpy(R.cell, cell.data(), 4 * n, hipMemcpyHostToDevice));
        HIPCHK(hipMemcpy(R.frac, frac.data(), 4 * n, hipMemcpyHostToDevice));
        HIPCHK(hipMemcpy(R.u, u.data(), 4 * n, hipMemcpyHostToDevice));
        HIPCHK(hipMemcpy(R.w, w.data(), 4 * n, hipMemcpyHostToDevice));
        HIPCHK(hipMemcpy(R.id, id.data(), 8 * n, hipMemcpyHostToDevice));
        HIPCHK(hipMemcpy(R.tube, tb.data(), 4 * n, hipMemcpyHostToDevice));
      }
      const long long nn = n;
      HIPCHK(hipMemcpy(g->pr_n, &nn, sizeof(long long), hipMemcpyHostToDevice));
      T.cnt[C_PROTONS] = n;
      T.dq = 0;
      T.dcur = 0;
      atm_reset(T);
      if ((e = upload_tubes(g))) return e;
      if (frozen) {
        const int grid = std::max(1, (int)std::min<long long>(1024, (g->total_nodes + 255) / 256));
        k_fill_i64<<<grid, 256, 0, g->s>>>(g->rho, g->total_nodes, 0);
        k_deposit_all<<<kGrid, TPB, 0, g->s>>>(make_ctx(g));
        k_deposit_protons<<<kGrid, TPB, 0, g->s>>>(make_ctx(g));
        FieldCtx f = make_fctx(g, 1);
        k_field_a<<<g->n_fb, FB_THREADS, 0, g->s>>>(f);
        k_field_b<<<g->n_fb, FB_THREADS, 0, g->s>>>(f);
      } else {
        rebuild_field(g);
      }
      return sync_and_err(g);
    }
    case GAP_STATE_ATMOSPHERE: {
      if (bytes < 16) return GAP_EINVAL;
      int32_t prev[2];
      std::memcpy(prev, b, 8);
      if (prev[0] < 0 || prev[1] < 0) return GAP_EINVAL;
      const int par = (int)((T.step - 1) & 1);
      for (int sp = 0; sp < 2; ++sp) {
        T.atm_cnt[2 * sp + par] = prev[sp];
        T.atm_cnt[2 * sp + (par ^ 1)] = 0;
      }
      std::memcpy(&T.atm_count, b + 8, 8);
      if ((e = upload_tubes(g))) return e;
      return sync_and_err(g);
    }
    case GAP_STATE_INJECTION: {
      if (bytes < 16) return GAP_EINVAL;
      std::memcpy(&T.inj_acc, b, 8);
      std::memcpy(&T.inj_count, b + 8, 8);
      if ((e = upload_tubes(g))) return e;
      return sync_and_err(g);
    }
    default:
      return GAP_EINVAL;
  }
} GAP_NO_THROW

int gap_autotune(gap_t* g, int32_t trial_steps, int32_t* chosen) try {
  if (!g || trial_steps < 1 || !chosen) return GAP_EINVAL;
  int e = sync_and_err(g);
  if (e) return e;
  return autotune(g, trial_steps, chosen);
} GAP_NO_THROW

int gap_window_forward(gap_t* g, int64_t window_steps, int32_t ckpt_every, double* loss) try {
  if (!g || window_steps < 1 || ckpt_every < 1 || !loss) return GAP_EINVAL;
  if (g->any_filter) return GAP_EINVAL;   // the adjoint is of the unfiltered update
  if (g->sticky) return g->sticky;
  return window_forward(g, window_steps, ckpt_every, loss);
} GAP_NO_THROW

int gap_window_backward(gap_t* g, double* dL_dalpha, double* dL_dninj) try {
  if (!g || !dL_dalpha || !dL_dninj) return GAP_EINVAL;
  if (g->sticky) return g->sticky;
  return backward(g, dL_dalpha, dL_dninj);
} GAP_NO_THROW

int gap_backward(gap_t* g, int64_t window_steps, int32_t ckpt_every, double* loss, double* dL_dalpha,
                 double* dL_dninj) {
  if (!g || !loss || !dL_dalpha || !dL_dninj) return GAP_EINVAL;
  int e = gap_window_forward(g, window_steps, ckpt_every, loss);
  if (e) return e;
  return gap_window_backward(g, dL_dalpha, dL_dninj);
}

void gap_free(gap_t* g) {
  if (!g) return;
  release(g);
  delete g;
}

const char* gap_strerror(int code) {
  switch (code) {
    case GAP_OK: return "ok";
    case GAP_EINVAL: return "invalid argument";
    case GAP_ENOMEM: return "out of device memory";
    case GAP_ECAP: return "particle store full: particles were dropped";
    case GAP_ETILE: return "a particle left its tile window";
    case GAP_ENAN: return "non-finite field";
    case GAP_EDEVICE: return "HIP runtime error";
    case GAP_ESTATE: return "call not valid in the current state";
    default: return "unknown error";
  }
}

int gap_e_spectrum_noalloc(gap_t* g, int32_t tube, double* power, int64_t power_len) {
  if (!g || tube < 0 || tube >= g->n_tubes || !power) return GAP_EINVAL;
  const int N = g->P[tube].n_cells;
  int M = 1;
  while (M < N) M *= 2;
  if (M > kScratchMaxM) return GAP_EINVAL;                  // beyond the static workspace
  if (power_len < (int64_t)M / 2 + 1) return GAP_EINVAL;
  // the transform of GAP_DIAG_ESPECTRUM, with its ping-pong buffers in the
  // static workspace (every entry is written before it is read) and the
  // result in the caller's buffer; nothing is allocated, nothing waits
  const int grid = std::max(1, std::min(1024, (M + 255) / 256));
  const double2* x = fft(g, g->E + g->th[tube].cell_off, N, M, g->scratch, g->scratch + M);
  k_fft_power<<<grid, 256, 0, g->s>>>(x, M, power);
  return hipGetLastError() == hipSuccess ? GAP_OK : GAP_EDEVICE;
}

int gap_qed_sample(gap_t* g, int32_t kind, const double* chi, const uint32_t* words, int64_t n, double* out) try {
  if (!g || (kind != 0 && kind != 1) || n < 0 || (n > 0 && (!chi || !words || !out))) return GAP_EINVAL;
  if (n == 0) return GAP_OK;
  if (g->sticky) return g->sticky;
  for (int64_t i = 0; i < n; ++i)
    if (!(chi[i] >= 0.0) || !std::isfinite(chi[i])) return GAP_EINVAL;
  int e;
  if ((e = upload_quantum_tables(g))) return e;
  float* dchi = (float*)dalloc(g, sizeof(float) * n);
  uint32_t* dw = (uint32_t*)dalloc(g, sizeof(uint32_t) * n);
  float* dout = (float*)dalloc(g, sizeof(float) * n);
  std::vector<float> hchi(chi, chi + n), hout(n);
  e = GAP_OK;
  if (!dchi || !dw || !dout) e = GAP_ENOMEM;
  if (!e && hipMemcpyAsync(dchi, hchi.data(), sizeof(float) * n, hipMemcpyHostToDevice, g->s) != hipSuccess) e = GAP_EDEVICE;
  if (!e && hipMemcpyAsync(dw, words, sizeof(uint32_t) * n, hipMemcpyHostToDevice, g->s) != hipSuccess) e = GAP_EDEVICE;
  if (!e) {
    const int grid = (int)std::min<int64_t>(4096, (n + 255) / 256);
    k_qed_sample<<<grid, 256, 0, g->s>>>(kind, dchi, dw, n, g->qs, g->qb, dout);
    if (hipMemcpyAsync(hout.data(), dout, sizeof(float) * n, hipMemcpyDeviceToHost, g->s) != hipSuccess ||
        hipStreamSynchronize(g->s) != hipSuccess)
      e = GAP_EDEVICE;
  }
  (void)hipStreamSynchronize(g->s);
  for (void* p : {(void*)dchi, (void*)dw, (void*)dout}) dfree(g, p);
  if (e) return e;
  for (int64_t i = 0; i < n; ++i) out[i] = hout[i];
  return GAP_OK;
} GAP_NO_THROW

int gap_sync_inverse_host(const float* r, float* xi, int64_t n) try {
  if (n < 0 || (n > 0 && (!r || !xi))) return GAP_EINVAL;
  const std::vector<float>& tab = sync_table();
  for (int64_t i = 0; i < n; ++i) {
    if (!(r[i] > 0.0f && r[i] < 1.0f)) return GAP_EINVAL;
    xi[i] = sync_sample_host(r[i], tab.data());
  }
  return GAP_OK;
} GAP_NO_THROW

}  // extern "C"
