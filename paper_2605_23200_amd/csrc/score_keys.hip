// The key-diversity score (minus the cosine of a key to the unit's mean key) and the similarity of the redundancy-aware
// score (mean cosine to the other keys) for bf16 caches, formed while the two softmax sweeps have the keys in registers.
//
// On their own the two scores stream K twice more (score.hip: keysum_kernel, keydiff_kernel; 0.37 + 0.40 ms next to 0.42 +
// 0.41 ms of sweeps for 256 units of 32768 keys), while the sweeps leave the matrix cores idle for two thirds of the time.
// Here a tile times the identity turns it into one channel per lane for the sums (8 more matrix instructions per block of
// 32 keys, next to 32 for 128 queries), the diagonal of the tile times itself gives the squared lengths (8), and the mean
// key joins the query columns as three bf16 terms (8).  The precision is that of the streaming kernels: the sums of the keys,
// and of the unit vectors with their lengths' reciprocals, in double; the squared lengths and the products with the mean key
// in fp32; the ratio in double.  (Sums of 16 keys in fp32 first took 2 % less, 1166 against 1193 us per step and 1299 against
// 1326, but lose a mean key far below the size of its keys.)  256 units of 32768 keys: 1734 -> 1193 us per step for the key
// diversity, 1927 -> 1326 for the mean cosines with the softmax partials of the cosines taken where they are formed.  fp32
// caches, the causal window (whose sweeps give the newest keys to workgroups of their own) and a pinned one-launch path keep the
// streaming kernels.
#include "score_sweep.h"

namespace ams {
namespace {

template <int NB, int HD, int KEYS>
hipError_t by_fold(const ScoreArgs& a, hipStream_t s) {
  return a.fold ? run_key_sweeps<NB, HD, KEYS, true>(a, s) : run_key_sweeps<NB, HD, KEYS, false>(a, s);
}

template <int HD, int KEYS>
hipError_t by_nb(const ScoreArgs& a, int nb, hipStream_t s) {
  if (nb <= 1) return by_fold<1, HD, KEYS>(a, s);
  if (nb <= 2) return by_fold<2, HD, KEYS>(a, s);
  if (nb <= 4) return by_fold<4, HD, KEYS>(a, s);
  if (nb <= 7) return by_fold<7, HD, KEYS>(a, s);
  if (nb <= 8) return by_fold<8, HD, KEYS>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_key_sweeps(const ScoreArgs& a, int nb, int head_dim, bool cosines, hipStream_t s) {
  if (a.causal || a.chunk > kKeysChunk || !a.g || !a.ksum) return hipErrorInvalidValue;
  if (head_dim == 64) return cosines ? by_nb<64, KEYS_COS>(a, nb, s) : by_nb<64, KEYS_MEAN>(a, nb, s);
  return cosines ? by_nb<128, KEYS_COS>(a, nb, s) : by_nb<128, KEYS_MEAN>(a, nb, s);
}

}  // namespace ams
