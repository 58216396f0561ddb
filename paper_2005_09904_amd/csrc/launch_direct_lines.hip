// Direct kernel: few rows, whole lines of them at a time.
#include "biq_launch_direct.inc"

namespace biq {

hipError_t launch_direct_lines(int q, int nt, const DirectParams& p, dim3 grid, int lds, hipStream_t s) {
    return launch_direct_q<DIRECT_LINES>(q, nt, p, grid, lds, s);
}

}  // namespace biq
