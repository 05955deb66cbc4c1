// Launchers of the stage and update passes over z columns.  The definitions are
// instantiated once per precision (pf_stage_fp64.hip, pf_stage_mixed.hip), apart
// from the rest of the runtime: six stage forms for every line length are most
// of the library's code.
#pragma once

#include "pf_plans.hpp"

namespace pf {

// Stage np + 1 (np previous stages) of the step described by sa: gk holds the
// previous stage's driving force (after its y transform), `out` receives the
// stage's state after the inverse z transform.  False for an unsupported size.
template <typename T, typename TE>
bool launch_stage(pf_ctx* c, const StepArgs<TE>& sa, int np, const cx<T>* gk, cx<T>* out);

// Update, error estimate and WRMS partial sums (c->partial) of the step, whose
// newest driving force is in gk.  Returns the number of partial pairs (the same
// for every tile variant), 0 for an unsupported size.
template <typename T, typename TE>
int launch_final(pf_ctx* c, const StepArgs<TE>& sa, const cx<T>* gk);

// Number of partial pairs launch_final writes on this grid, in the precision
// that has more.
int final_pairs_max(const Geo& g);

#ifdef PF_STAGE_DEFINITIONS
template <typename T, typename TE, int NP>
static void launch_stage_np(pf_ctx* c, const StepArgs<TE>& sa, const cx<T>* gk, cx<T>* out) {
  const Geo& g = c->g;
  col_dispatch(g.nz, [&](auto NC) {
    constexpr int N = decltype(NC)::value;
    with_variant(c->var[CK_STAGE], [&](auto VC) {
      constexpr int RE = col_re(CK_STAGE);
      constexpr int TX = col_tx(N, CK_STAGE, sizeof(cx<T>), decltype(VC)::value);
      const int nbx = (g.nxh + TX - 1) / TX;
      k_stage_invz<T, TE, N, TX, RE, NP><<<dim3(4 * nbx * g.ny), dim3(ColGeo<N, TX, RE>::THREADS), 0, c->stream>>>(
          sa, c->at, g, c->mk, gk, tw<T>(c, 0), out);
    });
  });
}

template <typename T, typename TE>
bool launch_stage(pf_ctx* c, const StepArgs<TE>& sa, int np, const cx<T>* gk, cx<T>* out) {
  if (!col_supported(c->g.nz)) return false;
  switch (np) {
    case 0: launch_stage_np<T, TE, 0>(c, sa, gk, out); break;
    case 1: launch_stage_np<T, TE, 1>(c, sa, gk, out); break;
    case 2: launch_stage_np<T, TE, 2>(c, sa, gk, out); break;
    case 3: launch_stage_np<T, TE, 3>(c, sa, gk, out); break;
    case 4: launch_stage_np<T, TE, 4>(c, sa, gk, out); break;
    case 5: launch_stage_np<T, TE, 5>(c, sa, gk, out); break;
    default: return false;
  }
  return true;
}

template <typename T, typename TE, int S>
static int launch_final_s(pf_ctx* c, const StepArgs<TE>& sa, const cx<T>* gk) {
  const Geo& g = c->g;
  int pairs = 0;
  col_dispatch(g.nz, [&](auto NC) {
    constexpr int N = decltype(NC)::value;
    with_variant(c->var[CK_STAGE], [&](auto VC) {
      constexpr int RE = col_re(CK_STAGE);
      constexpr int TX = col_tx(N, CK_STAGE, sizeof(cx<T>), decltype(VC)::value);
      constexpr int G = col_tx(N, CK_STAGE, sizeof(cx<T>), 0);
      const int nbx = (g.nxh + TX - 1) / TX;
      pairs = 4 * ((g.nxh + G - 1) / G) * g.ny;
      k_finalize<T, TE, N, TX, RE, S, G><<<dim3(4 * nbx * g.ny), dim3(ColGeo<N, TX, RE>::THREADS), 0, c->stream>>>(
          sa, c->at, g, c->mk, gk, tw<T>(c, 0), c->partial);
    });
  });
  return pairs;
}

template <typename T, typename TE>
int launch_final(pf_ctx* c, const StepArgs<TE>& sa, const cx<T>* gk) {
  switch (c->tab.s) {
    case 2: return launch_final_s<T, TE, 2>(c, sa, gk);
    case 3: return launch_final_s<T, TE, 3>(c, sa, gk);
    case 4: return launch_final_s<T, TE, 4>(c, sa, gk);
    case 6: return launch_final_s<T, TE, 6>(c, sa, gk);
    default: return 0;
  }
}
#endif

}  // namespace pf
