// Stage and update passes, FP64.
#define PF_STAGE_DEFINITIONS
#include "pf_stage.hpp"

namespace pf {
template bool launch_stage<double, double>(pf_ctx*, const StepArgs<double>&, int, const cx<double>*, cx<double>*);
template int launch_final<double, double>(pf_ctx*, const StepArgs<double>&, const cx<double>*);

int final_blocks_max(const Geo& g) {
  int tx = 1 << 20;
  col_dispatch(g.nz, [&](auto NC) {
    constexpr int N = decltype(NC)::value;
    for (int v : {col_tx(N, CK_STAGE, 16, 0), col_tx(N, CK_STAGE, 16, 1), col_tx(N, CK_STAGE, 8, 0),
                  col_tx(N, CK_STAGE, 8, 1)})
      tx = v < tx ? v : tx;
  });
  return 4 * ((g.nxh + tx - 1) / tx) * g.ny;
}
}  // namespace pf
