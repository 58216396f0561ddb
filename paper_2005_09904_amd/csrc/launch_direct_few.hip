// Direct kernel: few rows.
#include "biq_launch_direct.inc"

namespace biq {

hipError_t launch_direct_few(int q, int nt, const DirectParams& p, dim3 grid, int lds, hipStream_t s) {
    return launch_direct_q<DIRECT_FEW>(q, nt, p, grid, lds, s);
}

}  // namespace biq
