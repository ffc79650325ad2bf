// Instantiation unit: compiled once per (family shape, dtype) with
//   -DHJPD_FAM=<family type> -DHJPD_REAL=<float|double> -DHJPD_NAME=<lookup suffix>
// Where the four-node tiles are a unit of their own: -DHJPD_K_HI=3 -DHJPD_K4=<that unit's
// suffix> in the first, -DHJPD_K_LO=4 in the second.
#include "hjpd_launch.hpp"

#define HJPD_CAT2(a, b) a##b
#define HJPD_CAT(a, b) HJPD_CAT2(a, b)

#ifdef HJPD_K4
const void* HJPD_CAT(hjpd_lookup_, HJPD_K4)(int plain, int L, int K, int variant);
#endif

const void* HJPD_CAT(hjpd_lookup_, HJPD_NAME)(int plain, int L, int K, int variant) {
#ifdef HJPD_K4
  if (!plain && K == 4) return HJPD_CAT(hjpd_lookup_, HJPD_K4)(plain, L, K, variant);
#endif
  return hjpd::pick_kernel<HJPD_REAL, hjpd::HJPD_FAM>(plain, L, K, variant);
}
