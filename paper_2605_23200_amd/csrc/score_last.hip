// The second sweep with the last-query score (Sec. 3.3 plug-in scorer): the kernels of score_sweep.h with a second sum over the
// newest queries, or with their lanes' part of the one sum.
#include "score_sweep.h"

namespace ams {

hipError_t launch_last_usage(const ScoreArgs& a, int nb, int head_dim, int mode, bool bf16, hipStream_t s) {
  if (mode == MODE_LAST_LANES) return second_sweep<MODE_LAST_LANES, false>(a, nb, head_dim, bf16, s);
  return mode == MODE_LAST ? second_sweep<MODE_LAST, false>(a, nb, head_dim, bf16, s) : hipErrorInvalidValue;
}

}  // namespace ams
