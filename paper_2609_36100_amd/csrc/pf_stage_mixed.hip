// Stage and update passes, mixed form.
#define PF_STAGE_DEFINITIONS
#include "pf_stage.hpp"

namespace pf {
template bool launch_stage<float, float>(pf_ctx*, const StepArgs<float>&, int, const cx<float>*, cx<float>*);
template int launch_final<float, float>(pf_ctx*, const StepArgs<float>&, const cx<float>*);
}  // namespace pf
