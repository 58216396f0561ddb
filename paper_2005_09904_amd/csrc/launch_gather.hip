// mu = 8, tables in device memory, several input vectors, few lookups.
#include "biq_launch.h"

#include "biq_gather.h"

namespace biq {
namespace {

template <bool HALF>
hipError_t launch_gather_q(int q, const QueryParams& p, hipStream_t s) {
    const int rows = HALF ? 8 : 16;
    const dim3 grid((unsigned)((p.m + rows - 1) / rows), (unsigned)p.splits,
                    (unsigned)((p.batch + kGatherVec - 1) / kGatherVec));
    switch (q) {
        case 1: hipLaunchKernelGGL((gather8_kernel<1, HALF>), grid, dim3(64), 0, s, p); break;
        case 2: hipLaunchKernelGGL((gather8_kernel<2, HALF>), grid, dim3(64), 0, s, p); break;
        case 3: hipLaunchKernelGGL((gather8_kernel<3, HALF>), grid, dim3(64), 0, s, p); break;
        case 4: hipLaunchKernelGGL((gather8_kernel<4, HALF>), grid, dim3(64), 0, s, p); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gather(bool half, int q, const QueryParams& p, hipStream_t s) {
    return half ? launch_gather_q<true>(q, p, s) : launch_gather_q<false>(q, p, s);
}

}  // namespace biq
