// The near part of several boxes by one launch (pair_kernel.h).
#include "pair_kernel.h"

namespace useries {

// Held to 80 registers (6 wavefronts per SIMD instead of 5), without the step
// pipelining and its four registers.  The default kernels (degree 5 and 7 without
// exact Gaussians) fit; 50 of the 66 spill 8 or 12 bytes per lane.
template <int DEG, int NE>
__global__ void __launch_bounds__(64 * kPairWaves) __attribute__((amdgpu_waves_per_eu(6)))
k_pair_batch(const BatchTable* __restrict__ tab,
                                                   const BoxDesc* __restrict__ desc) {
    batch_for(tab, BK_PAIR, [&](int i, int item) {
        const BoxDesc& d = desc[tab->slot[i]];
        pair_body<DEG, NE, 1, false, 0>(d.pair, item, d.sorted, d.cl_info, d.cl_col, d.cl_z, d.zbin,
                                 d.fnear, d.pair_parts);
    });
}

// ne: the largest count of exact Gaussians of the batch's boxes
hipError_t launch_pair_batch(const BatchTable* tab, const BoxDesc* desc, int deg, int ne,
                             int grid, hipStream_t st) {
#define USERIES_PAIR_NE(D, E)                                                                 \
    case E:                                                                                   \
        hipLaunchKernelGGL((k_pair_batch<D, E>), dim3(grid), dim3(64 * kPairWaves), 0, st,    \
                           tab, desc);                                                        \
        break;
#define USERIES_PAIR_DEG(D)                                                                   \
    case D:                                                                                   \
        switch (exact_bucket(ne)) {                                                           \
            USERIES_PAIR_NE(D, 0) USERIES_PAIR_NE(D, 1) USERIES_PAIR_NE(D, 2)                 \
            USERIES_PAIR_NE(D, 3) USERIES_PAIR_NE(D, 5) USERIES_PAIR_NE(D, 8)                 \
        }                                                                                     \
        break;
    switch (deg) {
        USERIES_PAIR_DEG(4) USERIES_PAIR_DEG(5) USERIES_PAIR_DEG(6) USERIES_PAIR_DEG(7)
        USERIES_PAIR_DEG(8) USERIES_PAIR_DEG(9) USERIES_PAIR_DEG(10) USERIES_PAIR_DEG(11)
        USERIES_PAIR_DEG(12) USERIES_PAIR_DEG(13) USERIES_PAIR_DEG(14)
    default:
        return hipErrorInvalidValue;
    }
#undef USERIES_PAIR_DEG
#undef USERIES_PAIR_NE
    return hipGetLastError();
}

}  // namespace useries
