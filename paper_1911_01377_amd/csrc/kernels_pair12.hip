// The near part's one-box kernels for 1/r^12 (pair_kernel.h).
#include "pair_kernel.h"

namespace useries {

template hipError_t launch_pair_alpha<12>(const PairArgs&, int, const uint4*, const int2*,
                                         const int*, const uint2*, const int*, float4*, double*,
                                         hipStream_t);

}  // namespace useries
