// The near part of one box (pair_kernel.h): the 1/r kernels and the launch by
// power.  The other powers and the batched kernels have files of their own, so
// that they compile side by side.
#include "pair_kernel.h"

namespace useries {

// kernels_pair6.hip, kernels_pair12.hip
extern template hipError_t launch_pair_alpha<6>(const PairArgs&, int, const uint4*, const int2*,
                                                const int*, const uint2*, const int*, float4*,
                                                double*, hipStream_t);
extern template hipError_t launch_pair_alpha<12>(const PairArgs&, int, const uint4*, const int2*,
                                                 const int*, const uint2*, const int*, float4*,
                                                 double*, hipStream_t);

hipError_t launch_pair(const PairArgs& a, int nblocks, const uint4* sorted,
                       const int2* cl_info, const int* cl_col, const uint2* cl_z, const int* zbin,
                       float4* fnear, double* epart, hipStream_t st) {
    if (nblocks <= 0) return hipSuccess;
    switch (a.alpha) {
    case 1:
        return launch_pair_alpha<1>(a, nblocks, sorted, cl_info, cl_col, cl_z, zbin, fnear, epart,
                                    st);
    case 6:
        return launch_pair_alpha<6>(a, nblocks, sorted, cl_info, cl_col, cl_z, zbin, fnear, epart,
                                    st);
    case 12:
        return launch_pair_alpha<12>(a, nblocks, sorted, cl_info, cl_col, cl_z, zbin, fnear, epart,
                                     st);
    default:
        return hipErrorInvalidValue;
    }
}

}  // namespace useries
