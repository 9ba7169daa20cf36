// The sweeps of the last-query score (Sec. 3.3 plug-in scorer): the kernels of score_sweep.h with a second sum over the newest
// queries.
#include "score_sweep.h"

namespace ams {

hipError_t launch_last_sweeps(const ScoreArgs& a, int nb, int head_dim, int mode, bool bf16, hipStream_t s) {
  return launch_sweeps<false, SCORERS_LAST>(a, nb, head_dim, mode, bf16, s);
}

}  // namespace ams
