// Tables in device memory, few lookups.
#include "biq_launch.h"

#include "biq_gather.h"

namespace biq {
namespace {

template <bool HALF, int LOG_SLICES, bool MULTI>
hipError_t launch_gather_q(int q, const QueryParams& p, hipStream_t s) {
    const int rows = 64 / ((HALF ? 8 : 4) << LOG_SLICES), slices = (p.batch + kGatherVec - 1) / kGatherVec;
    const dim3 grid((unsigned)((p.m + rows - 1) / rows), (unsigned)((slices + (1 << LOG_SLICES) - 1) >> LOG_SLICES),
                    MULTI ? 1u : (unsigned)p.splits);
    const dim3 threads(MULTI ? 64 * (p.splits < kGatherWaves ? p.splits : kGatherWaves) : 64);
    const int lds = MULTI ? p.splits * (HALF ? 8 : 16) * kGatherVec * 4 : 0;
    switch (q) {
        case 1: hipLaunchKernelGGL((gather8_kernel<1, HALF, LOG_SLICES, MULTI>), grid, threads, lds, s, p); break;
        case 2: hipLaunchKernelGGL((gather8_kernel<2, HALF, LOG_SLICES, MULTI>), grid, threads, lds, s, p); break;
        case 3: hipLaunchKernelGGL((gather8_kernel<3, HALF, LOG_SLICES, MULTI>), grid, threads, lds, s, p); break;
        case 4: hipLaunchKernelGGL((gather8_kernel<4, HALF, LOG_SLICES, MULTI>), grid, threads, lds, s, p); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <bool HALF>
hipError_t launch_gather_half(int q, const QueryParams& p, bool multi, hipStream_t s) {
    switch (gather_log_slices(p.batch)) {
        case 0: return multi ? launch_gather_q<HALF, 0, true>(q, p, s) : launch_gather_q<HALF, 0, false>(q, p, s);
        case 1: return multi ? launch_gather_q<HALF, 1, true>(q, p, s) : launch_gather_q<HALF, 1, false>(q, p, s);
        default: return multi ? launch_gather_q<HALF, 2, true>(q, p, s) : launch_gather_q<HALF, 2, false>(q, p, s);
    }
}

template <int MU>
hipError_t launch_gather_mu(const QueryParams& p, bool ascending, hipStream_t s) {
    const GatherUnits g = gather_units_shape(p.log2G, p.m, p.batch, p.splits);
    const dim3 grid((unsigned)g.blocks, (unsigned)g.slice_blocks);
    const int waves = (p.splits + (1 << g.log_splits) - 1) >> g.log_splits;
    const dim3 threads(64 * (waves < kGatherWaves ? waves : kGatherWaves));
    const int lds = p.splits > 1 ? p.splits * (64 >> (p.log2G + g.log_splits)) * (p.batch == 1 ? 1 : kGatherVec) * 4 : 0;
    if (p.batch == 1)
        hipLaunchKernelGGL((gather_units_kernel<MU, 1>), grid, threads, lds, s, p, 0, g.log_splits, (int)ascending);
    else
        hipLaunchKernelGGL((gather_units_kernel<MU, kGatherVec>), grid, threads, lds, s, p, g.log_slices, g.log_splits,
                           (int)ascending);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gather(bool half, int q, const QueryParams& p, bool waves, hipStream_t s) {
    return half ? launch_gather_half<true>(q, p, waves, s) : launch_gather_half<false>(q, p, waves, s);
}

hipError_t launch_gather_units(int mu, const QueryParams& p, bool ascending, hipStream_t s) {
    switch (mu) {
        case 1: return launch_gather_mu<1>(p, ascending, s);
        case 2: return launch_gather_mu<2>(p, ascending, s);
        case 3: return launch_gather_mu<3>(p, ascending, s);
        case 4: return launch_gather_mu<4>(p, ascending, s);
        case 5: return launch_gather_mu<5>(p, ascending, s);
        case 6: return launch_gather_mu<6>(p, ascending, s);
        case 7: return launch_gather_mu<7>(p, ascending, s);
        case 8: return launch_gather_mu<8>(p, ascending, s);
        case 9: return launch_gather_mu<9>(p, ascending, s);
        case 10: return launch_gather_mu<10>(p, ascending, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace biq
