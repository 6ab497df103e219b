// Internal host interface shared by qb_lib.hip and the per-tile
// compilation units: the plan object, launch helpers and the collision
// pipelines (forward and reverse) instantiated for every tile shape.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <string>
#include <vector>

#include "qb.h"
#include "qb_adjoint.hpp"
#include "qb_kernels.hpp"

using qb::DevPlan;

static_assert(qb::groups_of(QB_F64) == qb::grouped<double> && qb::groups_of(QB_F32) == qb::grouped<float>,
              "host and device agree on which precision sums in groups");

// Records the text of a failed HIP call for qb_last_error(); true on success.
bool hip_ok(hipError_t e, const char* what);
// Records a message for qb_last_error().
void set_error(const char* what);

// Workgroups of `threads` threads of kernel `kern` resident on the current
// device at once (occupancy x compute units), rounded down to a multiple of
// 8 (one per XCD, so a grid stride keeps its XCD); at least 8.
int persistent_grid(const void* kern, int threads);

// Bump allocator over caller-owned device memory: the library never
// allocates device memory itself.  In measuring mode it only adds up the
// aligned sizes (the pointers stay null), which is how the workspace size
// of a problem is computed from the same layout code that carves it.
struct Arena {
  char* base = nullptr;
  size_t cap = 0, used = 0;
  bool measure = true;
  void reset(void* b, size_t c, bool m) {
    base = (char*)b;
    cap = c;
    used = 0;
    measure = m;
  }
  bool take(void** p, size_t n) {
    const size_t off = (used + 255) & ~(size_t)255;
    if (!measure && off + n > cap) return false;
    *p = measure ? nullptr : base + off;
    used = off + n;
    return true;
  }
};

inline int blocks(size_t n, int b) { return (int)((n + b - 1) / b); }

struct qb_plan_s {
  qb_problem prob;
  Arena ws;   // the plan's workspace (tables, walls, collision and state buffers)
  Arena adj;  // the reverse-mode workspace (qb_plan_enable_adjoint)
  int P, E, NT, TPR;
  int wcells;  // cells per collision launch (the workspace holds this many)
  int i3cells;  // cells per launch of k_i3 (its buffers hold this many)
  bool one_group = false;  // one summation group each in k_i3 and k_terms: float32, and float64 in
                           // a workspace too small for the groups
  int vjp_cells = 0;       // the same of the reverse-mode pipeline
  bool vjp_one = false;
  bool i3_pair = true;  // I_3 kernel pairs the Gauss-Legendre nodes (tuned; default per tile)
  int vjp_variant = 0;  // I_3 adjoint: 0 row w_bar in memory, 1 in registers (cfg_vjp; tuned)
  int vjp_E = 0;        // tile shape of the reverse-mode pipeline (cfg_vjp; tuned; 0: the forward tile)
  int vjp_tab = 0;      // its table set
  bool vjp_tile_set = false, vjp_variant_set = false;  // chosen by the caller or the tuner, not by cfg_vjp
  int term_sel = 3;     // collision terms assembled: 1 C_c, 2 C_d, 3 both
  int limiter = 0;      // transport slope limiter: 0 minmod, 1 superbee, 2 MC, 3 van Leer
  int field_mode = 0;   // field term: 0 inside the Heun step, 1 exact rotation split around it
  bool persistent = false;  // collision kernels grid-stride over their tasks from a resident-sized grid
  // quadrature tables in the FFT engine's element order, one set per tile
  // shape E (elements per thread) that has been selected on this plan
  struct TabSet {
    int E = 0;
    bool built = false;
    void *tw = nullptr, *phip = nullptr, *Kt = nullptr, *psi = nullptr, *psip = nullptr, *psiw = nullptr,
         *psips = nullptr, *negk = nullptr;
  };
  std::vector<TabSet> tabs;
  int cur_tab = 0;
  void *phx, *phy, *wm;  // natural order, independent of the tile
  void *spec, *wP, *terms, *acc, *i3s = nullptr, *i3o, *i3sum, *i3p, *i3ps;
  void *st0, *st1, *st2, *cbuf, *bcw;
  double* flux;
  // adjoint workspace (qb_plan_enable_adjoint)
  bool adjoint = false;
  void *lamP = nullptr, *acot = nullptr, *gspec = nullptr, *gf0 = nullptr, *i3g = nullptr,
       *i3sb = nullptr, *gsum = nullptr, *i3t = nullptr, *lamh = nullptr;
  void *fwa = nullptr;
  void *wn = nullptr, *wa = nullptr, *w1 = nullptr, *wb = nullptr, *lb = nullptr, *ls = nullptr, *la = nullptr,
       *cg = nullptr, *g0 = nullptr, *ext = nullptr;
  double* lflux = nullptr;
  qb::BcDev bl, br;
  // kernel timing
  bool profiling = false;
  struct Rec {
    int kernel;
    hipEvent_t a, b;
    bool counts;
  };
  std::vector<Rec> recs;
  std::vector<hipEvent_t> pool;

  bool measuring() const { return ws.measure; }
  // carve n bytes of the plan workspace (false once it is exhausted)
  bool alloc(void** p, size_t n) {
    if (ws.take(p, n)) return true;
    set_error("plan workspace exhausted");
    return false;
  }
  bool alloc_adj(void** p, size_t n) {
    if (adj.take(p, n)) return true;
    set_error("adjoint workspace exhausted");
    return false;
  }
  size_t bytes() const { return ws.used + (adjoint ? adj.used : 0); }
  ~qb_plan_s() {
    for (auto& r : recs) {
      (void)hipEventDestroy(r.a);
      (void)hipEventDestroy(r.b);
    }
    for (hipEvent_t e : pool) (void)hipEventDestroy(e);
  }
  hipEvent_t event() {
    if (!pool.empty()) {
      hipEvent_t e = pool.back();
      pool.pop_back();
      return e;
    }
    hipEvent_t e = nullptr;
    (void)hipEventCreate(&e);
    return e;
  }
  // bracket one launch: call begin() before and end() after the launch; not
  // `counts`: more of a launch that has been counted
  int begin(int kernel, hipStream_t s, bool counts = true) {
    if (!profiling) return -1;
    Rec r{kernel, event(), event(), counts};
    (void)hipEventRecord(r.a, s);
    recs.push_back(r);
    return (int)recs.size() - 1;
  }
  void end(int id, hipStream_t s) {
    if (id >= 0) (void)hipEventRecord(recs[id].b, s);
  }
};

// Summation groups of the I_3 nodes (see k_i3): 4 pairs of nodes to a group,
// 2 or 3 where there are too few for 4 groups.  Unpaired, a group holds as
// many nodes (2 gs), so that both kernels run in the same buffers.
inline void node_groups(int M, bool paired, bool one, int& gs, int& ng) {
  const int npair = (M + 1) / 2;
  gs = one ? npair : std::min(4, std::max(2, (npair + 3) / 4));
  ng = (npair + gs - 1) / gs;
  if (!paired) gs *= 2;
}
inline int node_groups(const qb_problem& p, bool one) {
  int gs, ng;
  node_groups(p.M, true, one, gs, ng);
  return ng;
}
// Directions per group of k_terms: 4 pairs, 8 transforms beside the final one.
constexpr int kTermDirs = 8;
inline int term_groups(int J, bool one) { return one ? 1 : (J + kTermDirs - 1) / kTermDirs; }

// Cells per launch of k_i3 in chunks of wcells cells.  At most as many as the
// I_3 buffers of one task per (cell, j) would hold, or 7.5 GB of them: a plan
// of many cells then takes little more than with one group (+15 % at J = 32),
// where all cells in one launch would take ng times as much.  (44 cells at
// N = 32, J = 32, M = 57: 14.0 ms, with 3.8 GB 14.3; 60 cells at N = 64,
// J = 24, M = 45: 90.5 and 91.4; more than 7.5 GB gains nothing on either.)
// Up to that, the number that leaves the fewest rounds of resident workgroups
// partly empty over the launches: 60 cells at N = 32, J = 36, M = 48 take 17.2
// ms in one launch, 18.5 in launches of 18 cells (15.2 rounds each).
inline int i3_launch_cells(const qb_problem& p, int wcells, bool one) {
  const int ng = node_groups(p, one), per_cell = p.J * ng;
  const int tasks = p.N == 16 ? 65536 : p.N == 32 ? 16384 : 4096;
  const int most = std::min(wcells, std::max({1, (wcells + ng - 1) / ng, tasks / per_cell}));
  const int resident = p.N == 16 ? 1024 : p.N == 32 ? 512 : 256;  // workgroups of the starting tile on the card
  auto rounds = [&](int cells) { return ((int64_t)cells * per_cell + resident - 1) / resident; };
  int best = most;
  int64_t least = INT64_MAX;
  for (int n = most; n >= (most + 1) / 2; --n) {
    const int64_t r = wcells / n * rounds(n) + rounds(wcells % n);
    if (r < least) least = r, best = n;
  }
  return best;
}

// Device view of the plan with the table set `tab` (the forward pipeline
// uses cur_tab, the reverse-mode pipeline vjp_tab).
template <typename T>
inline DevPlan<T> devplan(qb_plan_s* pl, int tab) {
  DevPlan<T> d;
  d.Nx = pl->prob.Nx;
  d.N = pl->prob.N;
  d.J = pl->prob.J;
  d.M = pl->prob.M;
  d.P = pl->P;
  d.L = (T)pl->prob.L;
  d.wc = (pl->term_sel & 1) ? (T)1 : (T)0;
  d.wd = (pl->term_sel & 2) ? (T)1 : (T)0;
  const qb_plan_s::TabSet& ts = pl->tabs[tab];
  d.tw = (const T*)ts.tw;
  d.phip = (const T*)ts.phip;
  d.Kt = (const T*)ts.Kt;
  d.psi = (const T*)ts.psi;
  d.psip = (const T*)ts.psip;
  d.psiw = (const T*)ts.psiw;
  d.psips = (const T*)ts.psips;
  d.negk = (const unsigned*)ts.negk;
  d.phx = (const T*)pl->phx;
  d.phy = (const T*)pl->phy;
  d.wm = (const T*)pl->wm;
  d.spec = (T*)pl->spec;
  d.wP = (T*)pl->wP;
  d.terms = (T*)pl->terms;
  d.acc = (T*)pl->acc;
  d.i3s = (T*)pl->i3s;
  d.i3o = (T*)pl->i3o;
  d.i3sum = (T*)pl->i3sum;
  d.i3p = (T*)pl->i3p;
  d.i3ps = (T*)pl->i3ps;
  node_groups(d.M, pl->i3_pair, pl->one_group, d.gs, d.ng);
  d.tg = term_groups(d.J, pl->one_group);
  d.td = pl->one_group ? d.J : kTermDirs;
  d.lamP = (T*)pl->lamP;
  d.acot = (T*)pl->acot;
  d.gspec = (T*)pl->gspec;
  d.gf0 = (T*)pl->gf0;
  d.i3g = (T*)pl->i3g;
  d.i3sb = (T*)pl->i3sb;
  d.gsum = (T*)pl->gsum;
  d.fwa = (T*)pl->fwa;
  d.i3t = (T*)pl->i3t;
  d.lamh = (T*)pl->lamh;
  return d;
}


// C[w] for the cells [cell0, cell0 + ncells) of the Pauli state arrays w, c
// ([4][Nx][N][N]); ncells <= wcells, the workspace holds the chunk's cells
// from index 0.  Defined in qb_pipelines.hpp.
template <typename T, int P, int E>
bool collision_pipeline(qb_plan_s* pl, const T* w, T* c, int ncells, int cell0, hipStream_t s);

// out = C'(w)^T lam for the same cells (Pauli gradients).
template <typename T, int P, int E>
bool collision_vjp_pipeline(qb_plan_s* pl, const T* w, const T* lam, T* out, int ncells, int cell0,
                            hipStream_t s);
