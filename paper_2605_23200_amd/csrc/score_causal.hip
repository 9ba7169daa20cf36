// The sweeps under the causal window (App. A "Mass construction"): the kernels of score_sweep.h whose launches hold a workgroup
// more per unit, for the newest keys, which not every query of the window sees.
#include "score_sweep.h"

namespace ams {

hipError_t launch_causal_sweeps(const ScoreArgs& a, int nb, int head_dim, int mode, bool bf16, hipStream_t s) {
  if (!a.causal) return hipErrorInvalidValue;
  return launch_sweeps<true, SCORERS_MEAN>(a, nb, head_dim, mode, bf16, s);
}

}  // namespace ams
