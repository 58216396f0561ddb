// Block-scaled matrix-core kernel, 4 wave group(s) along the contraction.
#include "biq_launch_digits.inc"

namespace biq {

hipError_t launch_digits_ws4(int q, int rpw, int ct, const DigitParams& p, int grid, int lds, hipStream_t s) {
    return launch_digits_ws<4>(q, rpw, ct, p, grid, lds, s);
}

}  // namespace biq
