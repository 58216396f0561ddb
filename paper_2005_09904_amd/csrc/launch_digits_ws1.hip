// Block-scaled matrix-core kernel, 1 wave group(s) along the contraction.
#include "biq_launch_digits.inc"

namespace biq {

hipError_t launch_digits_ws1(int q, int rpw, int ct, const DigitParams& p, int grid, int lds, hipStream_t s) {
    return launch_digits_ws<1>(q, rpw, ct, p, grid, lds, s);
}

hipError_t launch_xdigits(int ct, const float* X, uint8_t* Xd, int* form, int n, int batch, int groups, int col_groups,
                          hipStream_t s) {
    const dim3 grid(groups * col_groups * ct);
    if (ct == 2) hipLaunchKernelGGL(xdigits_kernel<2>, grid, dim3(256), 0, s, X, Xd, form, n, batch, groups);
    else hipLaunchKernelGGL(xdigits_kernel<1>, grid, dim3(256), 0, s, X, Xd, form, n, batch, groups);
    return hipGetLastError();
}

}  // namespace biq
