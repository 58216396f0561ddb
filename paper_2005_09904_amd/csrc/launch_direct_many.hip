// Direct kernel: many rows.
#include "biq_launch_direct.inc"

namespace biq {

hipError_t launch_direct_many(int q, int nt, const DirectParams& p, dim3 grid, int lds, hipStream_t s) {
    return launch_direct_q<DIRECT_MANY>(q, nt, p, grid, lds, s);
}

}  // namespace biq
