// The last-query score under the causal window: see score_last.hip and score_causal.hip.
#include "score_sweep.h"

namespace ams {

hipError_t launch_causal_last_usage(const ScoreArgs& a, int nb, int head_dim, int mode, bool bf16, hipStream_t s) {
  if (!a.causal) return hipErrorInvalidValue;
  if (mode == MODE_LAST_LANES) return second_sweep<MODE_LAST_LANES, true>(a, nb, head_dim, bf16, s);
  return mode == MODE_LAST ? second_sweep<MODE_LAST, true>(a, nb, head_dim, bf16, s) : hipErrorInvalidValue;
}

}  // namespace ams
