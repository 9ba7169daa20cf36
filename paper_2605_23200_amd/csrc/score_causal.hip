// The sweeps under the causal window (App. A "Mass construction"): the kernels of score_sweep.h whose launches hold a workgroup
// more per unit, for the newest keys, which not every query of the window sees.
#include "score_sweep.h"

namespace ams {

hipError_t launch_causal_first_sweep(const ScoreArgs& a, int nb, int head_dim, bool moments, bool bf16, hipStream_t s) {
  if (!a.causal) return hipErrorInvalidValue;
  return first_sweep<true>(a, nb, head_dim, moments, bf16, s);
}

hipError_t launch_causal_usage(const ScoreArgs& a, int nb, int head_dim, bool bf16, hipStream_t s) {
  if (!a.causal) return hipErrorInvalidValue;
  return second_sweep<MODE_MEAN, true>(a, nb, head_dim, bf16, s);
}

}  // namespace ams
