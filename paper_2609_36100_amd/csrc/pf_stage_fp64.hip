// Stage and update passes, FP64.
#define PF_STAGE_DEFINITIONS
#include "pf_stage.hpp"

#include <algorithm>

namespace pf {
template bool launch_stage<double, double>(pf_ctx*, const StepArgs<double>&, int, const cx<double>*, cx<double>*);
template int launch_final<double, double>(pf_ctx*, const StepArgs<double>&, const cx<double>*);

int final_pairs_max(const Geo& g) {
  int tx = 1;
  col_dispatch(g.nz, [&](auto NC) {
    constexpr int N = decltype(NC)::value;
    tx = std::min(col_tx(N, CK_STAGE, 16, 0), col_tx(N, CK_STAGE, 8, 0));
  });
  return 4 * ((g.nxh + tx - 1) / tx) * g.ny;
}
}  // namespace pf
