// The last-query score under the causal window: see score_last.hip and score_causal.hip.
#include "score_sweep.h"

namespace ams {

hipError_t launch_causal_last_sweeps(const ScoreArgs& a, int nb, int head_dim, int mode, bool bf16, hipStream_t s) {
  if (!a.causal) return hipErrorInvalidValue;
  return launch_sweeps<true, SCORERS_LAST>(a, nb, head_dim, mode, bf16, s);
}

}  // namespace ams
