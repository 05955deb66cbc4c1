// Batched ensembles: many independent simulations of uneven cubic sizes
// advanced together.
//
// The paper points at large ensembles of simulations (uncertainty
// quantification) as a use of faster-than-real-time runs (Discussion) and at
// tuning the parallel-loop tiling per architecture (Results, single-node
// performance).  Here every pass of the ImEx-ARK stage cycle is ONE kernel
// launch for the whole ensemble: a work list gives each member a contiguous
// range of work-groups, a work-group finds its member by binary search, and
// the member's grid size selects the inlined kernel body.  Step control
// (embedded error, WRMS, accept / reject, next step size) runs on the device
// per member, so one step of every member is a fixed sequence of launches
// that is captured once in a hipGraph and replayed.  The work-group size of
// each pass kind is chosen by an autotuner (two variants, timed on the
// ensemble itself).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <new>
#include <vector>

#include "../../include/pf.h"
#include "pf_context.hpp"
#include "pf_kernels.hpp"

using namespace pf;

namespace pf {

// grid lengths the batched kernels are compiled for
#define PF_ENS_SIZES(X) X(32) X(48) X(64) X(96) X(128)

static bool ens_size_ok(int n) {
  switch (n) {
#define PF_C(N) case N:
    PF_ENS_SIZES(PF_C)
#undef PF_C
    return true;
    default:
      return false;
  }
}

// per-member device descriptor
template <typename T, typename TE>
struct EMemb {
  Geo g;
  ModelK mk;
  cx<double>* ybuf[2];
  cx<TE>* FE[6];
  cx<T>* T1;
  cx<T>* T3;
  const cx<T>* twN;  // w_N: z, y and the x real length
  const cx<T>* twM;  // w_{N/2}: the packed x transform
};

// per-member integration state (device, mirrored on the host between calls)
// dt is the next attempt (the proposal dt_next capped by dt_max and clipped to
// t_final); dt_next is the controller's proposal itself, kept so that a later
// advance to a larger t_final resumes from it.
struct EState {
  double t, dt, tf, err, dt_last, dt_next;
  double rtol, atol, dt0, dt_min, dt_max;
  long long steps, attempts, rejects, n_rhs;
  int cur, done, rejrow, adaptive, max_rejects;
  int prevrej;  // the last attempt was rejected (caps the next proposal's growth)
};

// A member's coefficients (its own dt), read through the scalar cache: uniform
// operands that no kernel of a pass writes.
typedef const __attribute__((address_space(4))) ArkTab* TabK;
__device__ inline TabK member_tab(const ArkTab* tabs, int m) { return (TabK)(uintptr_t)(tabs + m); }

// kernel kinds with their own work list and work-group size
enum EKind { EK_STAGE = 0, EK_YFFT4, EK_YFFT3, EK_THETA, EK_ELASTIC, EK_DRIVE, EK_FWD_AC, EK_COUNT };
static const char* const ek_names[EK_COUNT] = {"stage_invz", "ypass4", "ypass3", "xpass_theta",
                                               "zpass_elastic", "xpass_drive", "zpass_fwd_ac"};

// Columns per work-group of eb threads for lines of n points: the largest
// power of two that fits, so every row segment starts on a 128-byte boundary
// (a width like 10 or 21 columns for the 48- and 96-point lines would make
// each segment straddle cache lines); the remaining threads idle.
constexpr int ens_tx(int eb, int n, int re) {
  const int tl = line_threads(n, re);
  const int fit = eb / tl < 1 ? 1 : eb / tl;
  int tx = 1;
  while (2 * tx <= fit) tx *= 2;
  return tx;
}
constexpr int ens_rb(int eb, int m) {
  const int tl = line_threads(m);
  return eb / tl < 1 ? 1 : eb / tl;
}
// LDS elements a work-group of eb threads needs for any size in the set
constexpr int ens_lds(int eb) {
  int mx = 0;
  const int ns[5] = {32, 48, 64, 96, 128};
  for (int i = 0; i < 5; ++i) {
    const int n = ns[i];
    const int c8 = n * (ens_tx(eb, n, 8) + 1), c4 = n * (ens_tx(eb, n, 4) + 1);
    const int r = ens_rb(eb, n / 2) * (n / 2 + 2);
    mx = c8 > mx ? c8 : mx;
    mx = c4 > mx ? c4 : mx;
    mx = r > mx ? r : mx;
  }
  return mx;
}

__device__ inline int find_member(const int* start, int M, int b) {
  int lo = 0, hi = M;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (start[mid] <= b)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// ---- batched kernels -------------------------------------------------------
// The member's arrays for one attempted step (its current and spare state).
template <typename T, typename TE>
__device__ inline StepArgs<TE> member_step(const EMemb<T, TE>& e, const EState& x) {
  StepArgs<TE> sa;
  sa.y = e.ybuf[x.cur];
#pragma unroll
  for (int j = 0; j < 6; ++j) sa.FE[j] = e.FE[j];
  sa.FI_out = nullptr;
  sa.FEc_out = nullptr;
  sa.ynew = e.ybuf[1 - x.cur];
  sa.err_out = nullptr;
  sa.rtol = x.rtol;
  sa.atol = x.atol;
  sa.sc = 1.0 / sqrt((double)e.g.nx * e.g.ny * e.g.nz);
  return sa;
}

// FP64 column passes keep the twiddle table in LDS and exchange with LDS-only
// barriers, so that loads and stores stay under way across them: members of
// 48^3 to 128^3 together, y passes 75 -> 69 us (three fields) and 95 -> 86 us
// (four), elastic 127 -> 118 us, the stage passes 3 to 7 %.  (Single grids'
// stage passes gained nothing at 512^3.)  FP32 passes were not measured so and
// keep the table in memory.
template <typename T>
constexpr int ens_lb = sizeof(T) == 8 ? 1 : 0;
template <typename T>
struct ColTable {
  cx<T> w[ens_lb<T> ? 128 : 1];
};
// complete after the pass's first barrier
template <int EB, typename T, typename TE>
__device__ inline const cx<T>* col_table(const EMemb<T, TE>& e, ColTable<T>& t) {
  if constexpr (ens_lb<T> == 0) {
    return e.twN;
  } else {
    for (int j = threadIdx.x; j < e.g.nz; j += EB) t.w[j] = e.twN[j];
    return t.w;
  }
}

template <typename T, typename TE, int EB, int NP>
__global__ void __launch_bounds__(EB) kb_stage(const EMemb<T, TE>* mem, const EState* st, const int* start, int M,
                                               const ArkTab* tabs) {
  __shared__ cx<T> lds[ens_lds(EB)];
  __shared__ ColTable<T> table;
  const int m = find_member(start, M, blockIdx.x);
  if (st[m].done) return;
  const EMemb<T, TE>& e = mem[m];
  const int item = blockIdx.x - start[m];
  StepArgs<TE> sa = member_step(e, st[m]);
  const TabK tb = member_tab(tabs, m);
  if (e.mk.fEa != 0.0) sa.FEc_out = e.FE[NP];
  const cx<T>* twl = col_table<EB>(e, table);
  switch (e.g.nz) {
#define PF_C(N)                                                                                              \
  case N:                                                                                                    \
    body_stage<T, TE, N, ens_tx(EB, N, 8), 8, NP, true, ens_lb<T>>(sa, tb, e.g, e.mk, e.T3, twl, e.T1, item,           \
                                                           threadIdx.x, lds);                               \
    break;
    PF_ENS_SIZES(PF_C)
#undef PF_C
  }
}

template <typename T, typename TE, int EB, int S, int NF>
__global__ void __launch_bounds__(EB) kb_ypass(const EMemb<T, TE>* mem, const EState* st, const int* start, int M) {
  __shared__ cx<T> lds[ens_lds(EB)];
  __shared__ ColTable<T> table;
  const int m = find_member(start, M, blockIdx.x);
  if (st[m].done) return;
  const EMemb<T, TE>& e = mem[m];
  const int tile = blockIdx.x - start[m];
  cx<T>* buf = NF == 4 ? e.T1 : e.T3;
  const cx<T>* twl = col_table<EB>(e, table);
  switch (e.g.nz) {
#define PF_C(N)                                                                                             \
  case N:                                                                                                   \
    body_colfft<T, N, ens_tx(EB, N, 8), 8, S, 1, true, ens_lb<T>>(buf, buf, e.g, NF, twl, (T)1, tile, threadIdx.x, lds); \
    break;
    PF_ENS_SIZES(PF_C)
#undef PF_C
  }
}

// The row passes' twiddle tables in LDS (lines of at most 128 points): read
// from memory between the exchanges, they held up every row behind the loads
// and stores under way (48^3 to 128^3 members together: theta 101 -> 75 us,
// drive 168 -> 135 us).
template <typename T, typename TE>
__device__ inline void row_tables(const EMemb<T, TE>& e, int eb, cx<T>* tN, cx<T>* tM) {
  for (int j = threadIdx.x; j < e.g.nx / 2; j += eb) {
    tN[j] = e.twN[j];
    tM[j] = e.twM[j];
  }
  __syncthreads();
}

template <typename T, typename TE, int EB>
__global__ void __launch_bounds__(EB) kb_theta(const EMemb<T, TE>* mem, const EState* st, const int* start, int M) {
  __shared__ cx<T> lds[ens_lds(EB)];
  __shared__ cx<T> tN[64], tM[64];
  const int m = find_member(start, M, blockIdx.x);
  if (st[m].done) return;
  const EMemb<T, TE>& e = mem[m];
  row_tables(e, EB, tN, tM);
  const int tile = blockIdx.x - start[m];
  switch (e.g.nz) {
#define PF_C(N)                                                                                      \
  case N:                                                                                            \
    body_xpass_theta<T, N / 2, ens_rb(EB, N / 2), true>(e.T1, e.T3, e.g, tN, tM, tile, threadIdx.x,   \
                                                         lds);                                       \
    break;
    PF_ENS_SIZES(PF_C)
#undef PF_C
  }
}

template <typename T, typename TE, int EB>
__global__ void __launch_bounds__(EB) kb_drive(const EMemb<T, TE>* mem, const EState* st, const int* start, int M) {
  __shared__ cx<T> lds[ens_lds(EB)];
  __shared__ cx<T> tN[64], tM[64];
  const int m = find_member(start, M, blockIdx.x);
  if (st[m].done) return;
  const EMemb<T, TE>& e = mem[m];
  row_tables(e, EB, tN, tM);
  const int tile = blockIdx.x - start[m];
  switch (e.g.nz) {
#define PF_C(N)                                                                                        \
  case N:                                                                                              \
    body_xpass_drive<T, N / 2, ens_rb(EB, N / 2), true, RowGeo<N / 2, ens_rb(EB, N / 2)>::SYNC>(       \
        e.T1, e.T3, e.g, e.mk, tN, tM, tile, threadIdx.x, lds);                                        \
    break;
    PF_ENS_SIZES(PF_C)
#undef PF_C
  }
}

template <typename T, typename TE, int EB>
__global__ void __launch_bounds__(EB) kb_elastic(const EMemb<T, TE>* mem, const EState* st, const int* start, int M,
                                                 int stage) {
  __shared__ cx<T> lds[ens_lds(EB)];
  __shared__ ColTable<T> table;
  const int m = find_member(start, M, blockIdx.x);
  if (st[m].done) return;
  const EMemb<T, TE>& e = mem[m];
  const int tile = blockIdx.x - start[m];
  const int acc = e.mk.fEa != 0.0 ? 1 : 0;
  const cx<T>* twl = col_table<EB>(e, table);
  switch (e.g.nz) {
#define PF_C(N)                                                                                           \
  case N:                                                                                                 \
    body_zpass_elastic<T, TE, N, ens_tx(EB, N, 4), 4, true, ens_lb<T>>(e.T3, e.g, e.mk, twl, e.FE[stage], acc, tile, \
                                                               threadIdx.x, lds);                         \
    break;
    PF_ENS_SIZES(PF_C)
#undef PF_C
  }
}

template <typename T, typename TE, int EB>
__global__ void __launch_bounds__(EB) kb_fwd_ac(const EMemb<T, TE>* mem, const EState* st, const int* start, int M,
                                                int stage) {
  __shared__ cx<T> lds[ens_lds(EB)];
  const int m = find_member(start, M, blockIdx.x);
  if (st[m].done) return;
  const EMemb<T, TE>& e = mem[m];
  const int tile = blockIdx.x - start[m];
  switch (e.g.nz) {
#define PF_C(N)                                                                                          \
  case N:                                                                                                \
    body_zpass_fwd_ac<T, TE, N, ens_tx(EB, N, 8), 8, true>(e.T3, e.g, e.mk, e.twN, e.FE[stage], tile,   \
                                                           threadIdx.x, lds);                            \
    break;
    PF_ENS_SIZES(PF_C)
#undef PF_C
  }
}

// Columns per partial pair of the update's sums: the narrower tile's, for both
// work-group sizes (tile_sums), so `pairs` is that tile's work list.
constexpr int ens_pair_cols(int n) { return ens_tx(128, n, 8); }

// Update + embedded error + WRMS partial sums.
template <typename T, typename TE, int EB, int S>
__global__ void __launch_bounds__(EB) kb_final(const EMemb<T, TE>* mem, const EState* st, const int* start, int M,
                                               const ArkTab* tabs, const int* pairs, double* partial) {
  __shared__ cx<T> lds[ens_lds(EB)];
  static_assert(sizeof(lds) >= 16 * EB, "the sums");
  __shared__ ColTable<T> table;
  const int m = find_member(start, M, blockIdx.x);
  if (st[m].done) return;  // uniform per block: the partials of done members are never read
  const EMemb<T, TE>& e = mem[m];
  const int item = blockIdx.x - start[m];
  const StepArgs<TE> sa = member_step(e, st[m]);
  const TabK tb = member_tab(tabs, m);
  const cx<T>* twl = col_table<EB>(e, table);
  double acc, bad;
  switch (e.g.nz) {
#define PF_C(N)                                                                                               \
  case N:                                                                                                     \
    body_final<T, TE, N, ens_tx(EB, N, 8), 8, S, true, ens_lb<T>>(sa, tb, e.g, e.mk, e.T3, twl, item,         \
                                                                  threadIdx.x, lds, acc, bad);               \
    tile_sums<N, ens_tx(EB, N, 8), 8, ens_pair_cols(N), EB>(acc, bad, e.g, item, threadIdx.x,                 \
                                                            reinterpret_cast<double*>(lds),                  \
                                                            partial + 2 * pairs[m]);                         \
    break;
    PF_ENS_SIZES(PF_C)
#undef PF_C
  }
}

__device__ inline double ctrl_factor(double dt, double err, int q, bool after_reject) {
  if (!isfinite(err)) return 0.25 * dt;
  double fac = err == 0.0 ? 5.0 : fmin(5.0, fmax(0.2, 0.9 * pow(err, -1.0 / (q + 1))));
  if (after_reject) fac = fmin(1.0, fac);
  return dt * fac;
}

// Accept / reject decision and next step size of a member from its summed
// error terms a and non-finite count b; returns the next attempt's dt.
__device__ inline double control_member(const Geo& g, EState& st, double a, double b, int q, int has_emb, int nrhs) {
  EState s = st;
  const double n3 = (double)g.nx * g.ny * g.nz;
  double err = has_emb ? sqrt(a / (4.0 * n3)) : 0.0;
  const bool finite = b == 0.0 && isfinite(err);
  if (!finite) err = INFINITY;
  bool ok;
  double nxt;
  if (s.adaptive) {
    ok = finite && err <= 1.0;
    nxt = fmax(ctrl_factor(s.dt, err, q, ok && s.prevrej != 0), s.dt_min);
    s.prevrej = ok ? 0 : 1;
  } else {
    ok = finite;
    nxt = s.dt0;
  }
  s.attempts += 1;
  s.n_rhs += nrhs;
  s.err = err;
  if (ok) {
    s.cur = 1 - s.cur;
    s.t += s.dt;
    s.steps += 1;
    s.dt_last = s.dt;
    s.rejrow = 0;
  } else {
    s.rejects += 1;
    s.rejrow += 1;
  }
  if (!finite && !s.adaptive) {
    s.done = 3;  // non-finite fixed-step run
  } else if (s.rejrow >= s.max_rejects) {
    s.done = 2;  // failed
  } else if (s.t >= s.tf * (1.0 - 1e-15)) {
    s.done = 1;
  }
  // next attempt: the controller's proposal (or dt0), capped and clipped to
  // t_final; the proposal itself is kept for a later advance
  s.dt_next = nxt;
  s.dt = fmin(fmin(nxt, s.dt_max), s.tf - s.t);
  st = s;
  return s.dt;
}

// One work-group per member: sum its partials in a fixed order, then the
// accept / reject decision and the next step size (thread 0).
template <typename T, typename TE>
__global__ void __launch_bounds__(256) kb_control(const EMemb<T, TE>* mem, EState* st, const int* pairs,
                                                  const double* partial, int q, int has_emb, int nrhs,
                                                  ArkTab unit, ArkTab* tabs) {
  __shared__ double sh[16];
  __shared__ double next_dt;
  const int m = blockIdx.x;
  if (st[m].done) return;
  double a = 0.0, b = 0.0;
  for (int i = pairs[m] + threadIdx.x; i < pairs[m + 1]; i += blockDim.x) {
    a += partial[2 * i];
    b += partial[2 * i + 1];
  }
  a = block_sum(a, sh);
  b = block_sum(b, sh);
  if (threadIdx.x == 0) next_dt = control_member(mem[m].g, st[m], a, b, q, has_emb, nrhs);
  __syncthreads();
  // the member's coefficients for its next attempt
  const double dt = next_dt;
  ArkTab& tb = tabs[m];
  if (threadIdx.x < 36) {
    const int k = threadIdx.x / 6, j = threadIdx.x % 6;
    tb.cE[k][j] = dt * unit.cE[k][j];
    tb.cI[k][j] = dt * unit.cI[k][j];
  } else if (threadIdx.x == 36) {
    tb.gdt = dt * unit.gdt;
    tb.dt = dt;
    tb.bl = dt * unit.bl;
    tb.dl = dt * unit.dl;
  }
}

}  // namespace pf

// ---- host side -------------------------------------------------------------------
struct pf_ens {
  int M = 0;
  int mixed = 0;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  std::vector<pf_params> prm;
  std::vector<pf_ctx*> views;
  std::vector<cx<double>*> yb0, yb1;  // state buffers 0 / 1 of each member
  std::vector<void*> allocs;
  void* mem_dev = nullptr;
  EState* st_dev = nullptr;
  EState* st_host = nullptr;  // pinned
  int* start[EK_COUNT][2] = {{nullptr}};
  int ntiles[EK_COUNT][2] = {{0}};
  double* partial = nullptr;  // the update's sums, by `pairs`
  const int* pairs() const { return start[EK_STAGE][0]; }
  int var[EK_COUNT] = {1, 1, 1, 1, 1, 1, 1};
  double tune_ms[EK_COUNT][2] = {{0}};
  ArkTable tab;
  ArkTab unit;                 // coefficients for dt = 1
  ArkTab* tab_dev = nullptr;   // each member's, for its next attempt
  ArkTab* tab_host = nullptr;  // pinned
  hipGraphExec_t exec = nullptr;
  hipGraph_t graph = nullptr;
  std::map<int, std::pair<cx<double>*, cx<double>*>> tw64;  // N -> (w_N, w_{N/2})
  std::map<int, std::pair<cx<float>*, cx<float>*>> tw32;
  int64_t ws_bytes = 0;
  double elapsed_ms = 0.0;
};

#define PF_HIP(call)                                   \
  do {                                                 \
    hipError_t e_ = (call);                            \
    if (e_ != hipSuccess) return PF_ERR_HIP;           \
  } while (0)

static pf_status ens_alloc(pf_ens* E, void** p, size_t bytes) {
  if (hipMalloc(p, bytes) != hipSuccess) {
    *p = nullptr;
    return PF_ERR_OOM;
  }
  E->allocs.push_back(*p);
  E->ws_bytes += (int64_t)bytes;
  return PF_OK;
}

template <int EB>
static int col_tiles(int n, int re) {
  const int tx = ens_tx(EB, n, re);
  return ((n / 2 + 1 + tx - 1) / tx) * n;
}
template <int EB>
static int row_tiles(int n) {
  const int rb = ens_rb(EB, n / 2);
  return (n * n + rb - 1) / rb;
}

template <int EB>
static int kind_tiles(int kind, int n) {
  switch (kind) {
    case EK_STAGE: return 4 * col_tiles<EB>(n, 8);  // one field per work-group (also the update's)
    case EK_ELASTIC: return col_tiles<EB>(n, 4);
    case EK_THETA:
    case EK_DRIVE: return row_tiles<EB>(n);
    default: return col_tiles<EB>(n, 8);
  }
}

static pf_status build_lists(pf_ens* E) {
  for (int k = 0; k < EK_COUNT; ++k)
    for (int v = 0; v < 2; ++v) {
      std::vector<int> st(E->M + 1, 0);
      for (int m = 0; m < E->M; ++m)
        st[m + 1] = st[m] + (v ? kind_tiles<256>(k, E->prm[m].nz) : kind_tiles<128>(k, E->prm[m].nz));
      pf_status s = ens_alloc(E, (void**)&E->start[k][v], sizeof(int) * (E->M + 1));
      if (s != PF_OK) return s;
      PF_HIP(hipMemcpy(E->start[k][v], st.data(), sizeof(int) * (E->M + 1), hipMemcpyHostToDevice));
      E->ntiles[k][v] = st[E->M];
    }
  return ens_alloc(E, (void**)&E->partial, sizeof(double) * 2 * E->ntiles[EK_STAGE][0]);
}

template <typename T, typename TE>
static void launch_kind(pf_ens* E, int kind, int stage) {
  const EMemb<T, TE>* mem = (const EMemb<T, TE>*)E->mem_dev;
  const int v = E->var[kind];
  const int nb = E->ntiles[kind][v];
  const int* st = E->start[kind][v];
  hipStream_t s = E->stream;
  auto go = [&](auto EBC) {
    constexpr int EB = decltype(EBC)::value;
    switch (kind) {
      case EK_STAGE:
        if (stage == E->tab.s) {  // the step's update; embedded pairs only
          switch (E->tab.s) {
            case 3: kb_final<T, TE, EB, 3><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M, E->tab_dev, E->pairs(), E->partial); break;
            case 4: kb_final<T, TE, EB, 4><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M, E->tab_dev, E->pairs(), E->partial); break;
            default: kb_final<T, TE, EB, 6><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M, E->tab_dev, E->pairs(), E->partial); break;
          }
          break;
        }
        switch (stage) {
          case 0: kb_stage<T, TE, EB, 0><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M, E->tab_dev); break;
          case 1: kb_stage<T, TE, EB, 1><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M, E->tab_dev); break;
          case 2: kb_stage<T, TE, EB, 2><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M, E->tab_dev); break;
          case 3: kb_stage<T, TE, EB, 3><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M, E->tab_dev); break;
          case 4: kb_stage<T, TE, EB, 4><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M, E->tab_dev); break;
          default: kb_stage<T, TE, EB, 5><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M, E->tab_dev); break;
        }
        break;
      case EK_YFFT4:
        if (stage < 0)
          kb_ypass<T, TE, EB, -1, 4><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M);
        else
          kb_ypass<T, TE, EB, +1, 4><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M);
        break;
      case EK_YFFT3:
        if (stage < 0)
          kb_ypass<T, TE, EB, -1, 3><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M);
        else
          kb_ypass<T, TE, EB, +1, 3><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M);
        break;
      case EK_THETA: kb_theta<T, TE, EB><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M); break;
      case EK_ELASTIC: kb_elastic<T, TE, EB><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M, stage); break;
      case EK_DRIVE: kb_drive<T, TE, EB><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M); break;
      default: kb_fwd_ac<T, TE, EB><<<nb, EB, 0, s>>>(mem, E->st_dev, st, E->M, stage); break;
    }
  };
  if (v)
    go(std::integral_constant<int, 256>{});
  else
    go(std::integral_constant<int, 128>{});
}

// One attempted step of every active member: 6 x 8 pass launches (mixed: 9), update, control.
template <typename T, typename TE>
static void enqueue_step(pf_ens* E) {
  const ArkTable& tb = E->tab;
  for (int i = 0; i < tb.s; ++i) {
    launch_kind<T, TE>(E, EK_STAGE, i);
    launch_kind<T, TE>(E, EK_YFFT4, +1);  // inverse y of the state
    launch_kind<T, TE>(E, EK_THETA, i);
    launch_kind<T, TE>(E, EK_YFFT3, -1);  // forward y of theta
    launch_kind<T, TE>(E, EK_ELASTIC, i);
    launch_kind<T, TE>(E, EK_YFFT3, +1);  // inverse y of the elastic potentials
    launch_kind<T, TE>(E, EK_DRIVE, i);
    launch_kind<T, TE>(E, EK_YFFT3, -1);  // forward y of the driving force
    if (!fresh_fe<T>) launch_kind<T, TE>(E, EK_FWD_AC, i);
  }
  launch_kind<T, TE>(E, EK_STAGE, tb.s);
  const EMemb<T, TE>* mem = (const EMemb<T, TE>*)E->mem_dev;
  kb_control<T, TE><<<E->M, 256, 0, E->stream>>>(mem, E->st_dev, E->pairs(), E->partial, tb.emb_order, tb.has_emb,
                                                  tb.s, E->unit, E->tab_dev);
}

// Members' states and coefficients (for the dt of their next attempt) to the device.
static pf_status upload_states(pf_ens* E) {
  for (int m = 0; m < E->M; ++m) fill_tab(E->tab, E->st_host[m].dt, E->tab_host[m]);
  PF_HIP(hipMemcpyAsync(E->st_dev, E->st_host, sizeof(EState) * E->M, hipMemcpyHostToDevice, E->stream));
  PF_HIP(hipMemcpyAsync(E->tab_dev, E->tab_host, sizeof(ArkTab) * E->M, hipMemcpyHostToDevice, E->stream));
  return PF_OK;
}

static void drop_graph(pf_ens* E) {
  if (E->exec) hipGraphExecDestroy(E->exec);
  if (E->graph) hipGraphDestroy(E->graph);
  E->exec = nullptr;
  E->graph = nullptr;
}

static pf_status capture_step(pf_ens* E) {
  drop_graph(E);
  PF_HIP(hipStreamBeginCapture(E->stream, hipStreamCaptureModeThreadLocal));
  if (E->mixed)
    enqueue_step<float, float>(E);
  else
    enqueue_step<double, double>(E);
  hipError_t e = hipStreamEndCapture(E->stream, &E->graph);
  if (e != hipSuccess) return PF_ERR_HIP;
  PF_HIP(hipGraphInstantiate(&E->exec, E->graph, nullptr, nullptr, 0));
  return PF_OK;
}

template <typename T, typename TE>
static pf_status build_members(pf_ens* E) {
  std::vector<EMemb<T, TE>> host(E->M);
  for (int m = 0; m < E->M; ++m) {
    pf_ctx* v = E->views[m];
    EMemb<T, TE>& e = host[m];
    std::memset(&e, 0, sizeof(e));
    e.g = v->g;
    e.mk = v->mk;
    e.ybuf[0] = v->y;
    e.ybuf[1] = v->ynew;
    for (int j = 0; j < 6; ++j) e.FE[j] = (cx<TE>*)v->FE[j];
    e.T1 = (cx<T>*)v->scratch;
    e.T3 = e.T1 + 4 * v->g.fs;
    if constexpr (sizeof(T) == 8) {
      e.twN = v->tw64[0];
      e.twM = v->tw64[2];
    } else {
      e.twN = v->tw32[0];
      e.twM = v->tw32[2];
    }
  }
  pf_status s = ens_alloc(E, &E->mem_dev, sizeof(EMemb<T, TE>) * E->M);
  if (s != PF_OK) return s;
  PF_HIP(hipMemcpy(E->mem_dev, host.data(), sizeof(EMemb<T, TE>) * E->M, hipMemcpyHostToDevice));
  return PF_OK;
}

extern "C" {

pf_status pf_ensemble_init(int32_t n, const pf_params* per_member, void* stream, pf_ens** out) {
  if (!out || !per_member || n < 1 || n > 4096) return PF_ERR_ARG;
  *out = nullptr;
  const pf_params& p0 = per_member[0];
  for (int m = 0; m < n; ++m) {
    const pf_params& p = per_member[m];
    if (p.nx != p.ny || p.ny != p.nz || !ens_size_ok(p.nx)) return PF_ERR_UNSUPPORTED_SIZE;
    if (!method_embedded(p.method) || p.method != p0.method || p.precision != p0.precision ||
        p.adaptive != p0.adaptive)
      return PF_ERR_ARG;
    if (p.precision != PF_FP64 && p.precision != PF_MIXED) return PF_ERR_ARG;
    if (p.dx <= 0.0 || (p.adaptive && (p.rtol < 0.0 || p.atol <= 0.0))) return PF_ERR_ARG;
    if (p.norm_space != 0) return PF_ERR_ARG;  // ensembles take the k-space norm only
    if (p.elastic_inhom != 0) return PF_ERR_ARG;  // and the homogeneous elasticity
  }
  int ndev = 0;  // no usable device: a HIP error, before any allocation
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) return PF_ERR_HIP;
  pf_ens* E = new (std::nothrow) pf_ens();
  if (!E) return PF_ERR_OOM;
  E->M = n;
  E->mixed = p0.precision == PF_MIXED;
  E->prm.assign(per_member, per_member + n);
  if (stream) {
    E->stream = (hipStream_t)stream;
  } else {
    if (hipStreamCreateWithFlags(&E->stream, hipStreamNonBlocking) != hipSuccess) {
      delete E;
      return PF_ERR_HIP;
    }
    E->own_stream = true;
  }
  E->tab = table_for(p0.method);
  fill_tab(E->tab, 1.0, E->unit);
  pf_status s = PF_OK;
  // per-size twiddle tables
  for (int m = 0; m < n && s == PF_OK; ++m) {
    const int N = per_member[m].nz;
    if (E->tw64.count(N)) continue;
    std::vector<cx<double>> a(N), b(N / 2);
    std::vector<cx<float>> af(N), bf(N / 2);
    make_twiddles64(N, a.data());
    make_twiddles64(N / 2, b.data());
    make_twiddles32(N, af.data());
    make_twiddles32(N / 2, bf.data());
    cx<double>*d0, *d1;
    cx<float>*f0, *f1;
    s = ens_alloc(E, (void**)&d0, sizeof(cx<double>) * N);
    if (s == PF_OK) s = ens_alloc(E, (void**)&d1, sizeof(cx<double>) * (N / 2));
    if (s == PF_OK) s = ens_alloc(E, (void**)&f0, sizeof(cx<float>) * N);
    if (s == PF_OK) s = ens_alloc(E, (void**)&f1, sizeof(cx<float>) * (N / 2));
    if (s != PF_OK) break;
    hipMemcpy(d0, a.data(), sizeof(cx<double>) * N, hipMemcpyHostToDevice);
    hipMemcpy(d1, b.data(), sizeof(cx<double>) * (N / 2), hipMemcpyHostToDevice);
    hipMemcpy(f0, af.data(), sizeof(cx<float>) * N, hipMemcpyHostToDevice);
    hipMemcpy(f1, bf.data(), sizeof(cx<float>) * (N / 2), hipMemcpyHostToDevice);
    E->tw64[N] = std::make_pair(d0, d1);
    E->tw32[N] = std::make_pair(f0, f1);
  }
  // per-member buffers and view contexts
  for (int m = 0; m < n && s == PF_OK; ++m) {
    pf_ctx* v = new (std::nothrow) pf_ctx();
    if (!v) {
      s = PF_ERR_OOM;
      break;
    }
    ctx_setup(v, &per_member[m], E->stream);
    v->owns = false;
    E->views.push_back(v);
    const Geo& g = v->g;
    const size_t k64 = sizeof(cx<double>) * 4 * (size_t)g.fs;
    const size_t fe = (E->mixed ? sizeof(cx<float>) : sizeof(cx<double>)) * 4 * (size_t)g.fs;
    const size_t tb = (E->mixed ? sizeof(cx<float>) : sizeof(cx<double>)) * 7 * (size_t)g.fs;
    const size_t rb = sizeof(double) * 4 * (size_t)g.nx * g.ny * g.nz;
    v->scratch_bytes = std::max(tb, rb);
    s = ens_alloc(E, (void**)&v->y, k64);
    if (s == PF_OK) s = ens_alloc(E, (void**)&v->ynew, k64);
    E->yb0.push_back(v->y);
    E->yb1.push_back(v->ynew);
    for (int i = 0; i < E->tab.s && s == PF_OK; ++i) s = ens_alloc(E, &v->FE[i], fe);
    if (s == PF_OK) s = ens_alloc(E, &v->scratch, v->scratch_bytes);
    if (s == PF_OK) s = ens_alloc(E, (void**)&v->partial, sizeof(double) * 4 * v->nblk_red);
    if (s == PF_OK) s = ens_alloc(E, (void**)&v->red, sizeof(double) * 8);
    if (s == PF_OK && hipHostMalloc((void**)&v->host_red, sizeof(double) * 8, 0) != hipSuccess) s = PF_ERR_OOM;
    if (s != PF_OK) break;
    const int N = g.nz;
    v->tw64[0] = v->tw64[1] = v->tw64[3] = E->tw64[N].first;
    v->tw64[2] = E->tw64[N].second;
    v->tw32[0] = v->tw32[1] = v->tw32[3] = E->tw32[N].first;
    v->tw32[2] = E->tw32[N].second;
    if (hipMemsetAsync(v->y, 0, k64, E->stream) != hipSuccess) s = PF_ERR_HIP;
  }
  if (s == PF_OK) s = E->mixed ? build_members<float, float>(E) : build_members<double, double>(E);
  if (s == PF_OK) s = build_lists(E);
  if (s == PF_OK) s = ens_alloc(E, (void**)&E->st_dev, sizeof(EState) * n);
  if (s == PF_OK && hipHostMalloc((void**)&E->st_host, sizeof(EState) * n, 0) != hipSuccess) s = PF_ERR_OOM;
  if (s == PF_OK) s = ens_alloc(E, (void**)&E->tab_dev, sizeof(ArkTab) * n);
  if (s == PF_OK && hipHostMalloc((void**)&E->tab_host, sizeof(ArkTab) * n, 0) != hipSuccess) s = PF_ERR_OOM;
  if (s == PF_OK) {
    for (int m = 0; m < n; ++m) {
      EState& x = E->st_host[m];
      std::memset(&x, 0, sizeof(x));
      const pf_params& p = per_member[m];
      x.dt = p.dt0;
      x.dt_next = p.dt0;
      x.rtol = p.rtol;
      x.atol = p.atol;
      x.dt0 = p.dt0;
      x.dt_min = p.dt_min;
      x.dt_max = p.dt_max;
      x.adaptive = p.adaptive;
      x.max_rejects = p.max_rejects > 0 ? p.max_rejects : 10;
      x.done = 1;
    }
    if (hipStreamSynchronize(E->stream) != hipSuccess) s = PF_ERR_HIP;
  }
  if (s != PF_OK) {
    pf_ensemble_finalize(E);
    return s;
  }
  *out = E;
  return PF_OK;
}

void pf_ensemble_finalize(pf_ens* E) {
  if (!E) return;
  if (E->stream) hipStreamSynchronize(E->stream);
  drop_graph(E);
  for (pf_ctx* v : E->views) {
    if (v && v->host_red) hipHostFree(v->host_red);
    pf_finalize(v);
  }
  for (void* p : E->allocs) hipFree(p);
  if (E->st_host) hipHostFree(E->st_host);
  if (E->tab_host) hipHostFree(E->tab_host);
  if (E->own_stream && E->stream) hipStreamDestroy(E->stream);
  delete E;
}

int32_t pf_ensemble_size_supported(int32_t n) { return ens_size_ok(n) ? 1 : 0; }

int64_t pf_ensemble_workspace_bytes(const pf_ens* E) { return E ? E->ws_bytes : 0; }

// The member's view context with y / ynew pointing at its current / spare
// state buffer.
static pf_status view_for(pf_ens* E, int32_t m, pf_ctx** v) {
  if (!E || m < 0 || m >= E->M) return PF_ERR_ARG;
  pf_ctx* c = E->views[m];
  const int cur = E->st_host[m].cur;
  c->y = cur ? E->yb1[m] : E->yb0[m];
  c->ynew = cur ? E->yb0[m] : E->yb1[m];
  *v = c;
  return PF_OK;
}

pf_status pf_ensemble_set_state(pf_ens* E, int32_t m, const double* c, const double* eta, int32_t on_device,
                                double t0) {
  if (!E || m < 0 || m >= E->M) return PF_ERR_ARG;
  E->st_host[m].cur = 0;  // state buffer 0 becomes current
  pf_ctx* v;
  pf_status s = view_for(E, m, &v);
  if (s != PF_OK) return s;
  s = pf_set_state(v, c, eta, on_device, t0);
  if (s != PF_OK) return s;
  EState& x = E->st_host[m];
  x.t = t0;
  x.dt = E->prm[m].dt0;
  x.dt_next = E->prm[m].dt0;
  x.steps = x.attempts = x.rejects = x.n_rhs = 0;
  x.rejrow = 0;
  x.prevrej = 0;
  x.done = 1;
  return PF_OK;
}

pf_status pf_ensemble_get_state(pf_ens* E, int32_t m, double* c, double* eta, int32_t on_device) {
  pf_ctx* v;
  pf_status s = view_for(E, m, &v);
  if (s != PF_OK) return s;
  return pf_get_state(v, c, eta, on_device);
}

pf_status pf_ensemble_get_state_hat(pf_ens* E, int32_t m, void* y_hat) {
  pf_ctx* v;
  pf_status s = view_for(E, m, &v);
  if (s != PF_OK) return s;
  return pf_get_state_hat(v, y_hat);
}

pf_status pf_ensemble_diagnostics(pf_ens* E, int32_t m, double* mass, double* vf, double* vf_thr) {
  pf_ctx* v;
  pf_status s = view_for(E, m, &v);
  if (s != PF_OK) return s;
  return pf_diagnostics(v, mass, vf, vf_thr);
}

pf_status pf_ensemble_free_energy(pf_ens* E, int32_t m, double* F) {
  pf_ctx* v;
  pf_status s = view_for(E, m, &v);
  if (s != PF_OK) return s;
  return pf_free_energy(v, F);
}

}  // extern "C"

namespace pf {
// Member access for the surrogate's ensemble advance (same library).
int ens_members(const pf_ens* E) { return E ? E->M : 0; }
int ens_member_n(const pf_ens* E, int m) { return (E && m >= 0 && m < E->M) ? E->prm[m].nz : 0; }
double ens_member_time(const pf_ens* E, int m) { return (E && m >= 0 && m < E->M) ? E->st_host[m].t : 0.0; }
hipStream_t ens_stream(const pf_ens* E) { return E ? E->stream : nullptr; }
// Sets member m's real-space state (device [4][n^3]) and time t, keeping its
// proposed step size and its step counters.
pf_status ens_member_set(pf_ens* E, int m, const double* u, double t) {
  if (!E || m < 0 || m >= E->M || !u) return PF_ERR_ARG;
  EState& x = E->st_host[m];
  x.cur = 0;
  pf_ctx* v;
  pf_status s = view_for(E, m, &v);
  if (s != PF_OK) return s;
  const long long P = (long long)v->g.nx * v->g.ny * v->g.nz;
  s = pf_set_state(v, u, u + P, 1, t);
  if (s != PF_OK) return s;
  x.t = t;
  x.rejrow = 0;
  x.done = 1;
  return PF_OK;
}
}  // namespace pf

extern "C" {

int64_t pf_ensemble_kspace_pitch(const pf_ens* E, int32_t m) {
  if (!E || m < 0 || m >= E->M) return 0;
  return E->views[m]->g.P;
}

pf_status pf_ensemble_advance(pf_ens* E, const double* t_final, int32_t max_steps, pf_stats* per_member) {
  if (!E || !t_final || max_steps < 1) return PF_ERR_ARG;
  for (int m = 0; m < E->M; ++m) {
    EState& x = E->st_host[m];
    x.tf = t_final[m];
    x.rejrow = 0;
    x.done = (x.t >= x.tf * (1.0 - 1e-15)) ? 1 : 0;
    if (!x.done) x.dt = std::min(std::min(x.dt_next, x.dt_max), x.tf - x.t);
  }
  pf_status up = upload_states(E);
  if (up != PF_OK) return up;
  if (!E->exec) {
    pf_status s = capture_step(E);
    if (s != PF_OK) return s;
  }
  hipEvent_t e0, e1;
  PF_HIP(hipEventCreate(&e0));
  PF_HIP(hipEventCreate(&e1));
  PF_HIP(hipEventRecord(e0, E->stream));
  int steps = 0;
  pf_status status = PF_OK;
  const int chunk = 4;
  while (steps < max_steps) {
    for (int k = 0; k < chunk && steps < max_steps; ++k, ++steps) PF_HIP(hipGraphLaunch(E->exec, E->stream));
    PF_HIP(hipMemcpyAsync(E->st_host, E->st_dev, sizeof(EState) * E->M, hipMemcpyDeviceToHost, E->stream));
    PF_HIP(hipStreamSynchronize(E->stream));
    bool all = true;
    for (int m = 0; m < E->M; ++m) all = all && E->st_host[m].done != 0;
    if (all) break;
  }
  PF_HIP(hipEventRecord(e1, E->stream));
  PF_HIP(hipEventSynchronize(e1));
  float ms = 0.f;
  hipEventElapsedTime(&ms, e0, e1);
  hipEventDestroy(e0);
  hipEventDestroy(e1);
  E->elapsed_ms += ms;
  for (int m = 0; m < E->M; ++m) {
    const EState& x = E->st_host[m];
    if (x.done == 2) status = PF_ERR_STEP_FAIL;
    if (x.done == 3 && status == PF_OK) status = PF_ERR_NONFINITE;
    if (x.done == 0 && status == PF_OK) status = PF_ERR_STATE;  // max_steps reached first
    if (per_member) {
      pf_stats& o = per_member[m];
      std::memset(&o, 0, sizeof(o));
      o.steps = x.steps;
      o.attempts = x.attempts;
      o.rejects = x.rejects;
      o.n_rhs = x.n_rhs;
      o.t = x.t;
      o.dt_last = x.dt_last;
      o.dt_next = x.dt_next;
      o.err_last = x.err;
      o.elapsed_ms = ms;
      o.mass = o.F = o.vf = o.vf_threshold = NAN;
      pf_ctx* v = nullptr;
      double d[4];
      if (view_for(E, m, &v) == PF_OK && v->have_state && ctx_diagnostics(v, true, d) == PF_OK) {
        o.mass = d[0];
        o.vf = d[1];
        o.vf_threshold = d[2];
        o.F = d[3];
      }
    }
  }
  return status;
}

pf_status pf_ensemble_autotune(pf_ens* E, int32_t reps) {
  if (!E || reps < 1) return PF_ERR_ARG;
  // time each kind on all members (the states are only read; the stage arrays,
  // the temporaries and, by the timed update, each member's spare state buffer
  // are overwritten)
  for (int m = 0; m < E->M; ++m) E->st_host[m].done = 0;
  pf_status up = upload_states(E);
  if (up != PF_OK) return up;
  hipEvent_t e0, e1;
  PF_HIP(hipEventCreate(&e0));
  PF_HIP(hipEventCreate(&e1));
  for (int k = 0; k < EK_COUNT; ++k) {
    double best = 1e300;
    int bv = 1;
    for (int v = 0; v < 2; ++v) {
      E->var[k] = v;
      const int stage = (k == EK_YFFT4 || k == EK_YFFT3) ? 1 : 0;
      // the stage kernel differs per stage (number of previous stages): time
      // the whole sequence of a step, its update included
      const int s0 = (k == EK_STAGE) ? 0 : stage;
      const int s1 = (k == EK_STAGE) ? E->tab.s + 1 : stage + 1;
      auto run = [&]() {
        for (int st = s0; st < s1; ++st) {
          if (E->mixed)
            launch_kind<float, float>(E, k, st);
          else
            launch_kind<double, double>(E, k, st);
        }
      };
      run();
      PF_HIP(hipEventRecord(e0, E->stream));
      for (int r = 0; r < reps; ++r) run();
      PF_HIP(hipEventRecord(e1, E->stream));
      PF_HIP(hipEventSynchronize(e1));
      PF_HIP(hipGetLastError());
      float ms = 0.f;
      hipEventElapsedTime(&ms, e0, e1);
      E->tune_ms[k][v] = ms / reps;
      if (ms < best) {
        best = ms;
        bv = v;
      }
    }
    E->var[k] = bv;
  }
  hipEventDestroy(e0);
  hipEventDestroy(e1);
  for (int m = 0; m < E->M; ++m) E->st_host[m].done = 1;
  drop_graph(E);  // re-captured with the chosen plans
  return PF_OK;
}

int32_t pf_ensemble_tuning_kinds(void) { return EK_COUNT; }

const char* pf_ensemble_tuning_name(int32_t k) { return (k >= 0 && k < EK_COUNT) ? ek_names[k] : ""; }

pf_status pf_ensemble_tuning_get(pf_ens* E, int32_t k, int32_t* block_threads, double* ms128, double* ms256) {
  if (!E || k < 0 || k >= EK_COUNT) return PF_ERR_ARG;
  if (block_threads) *block_threads = E->var[k] ? 256 : 128;
  if (ms128) *ms128 = E->tune_ms[k][0];
  if (ms256) *ms256 = E->tune_ms[k][1];
  return PF_OK;
}

pf_status pf_ensemble_tuning_set(pf_ens* E, int32_t k, int32_t block_threads) {
  if (!E || k < 0 || k >= EK_COUNT || (block_threads != 128 && block_threads != 256)) return PF_ERR_ARG;
  E->var[k] = block_threads == 256 ? 1 : 0;
  drop_graph(E);
  return PF_OK;
}

}  // extern "C"
