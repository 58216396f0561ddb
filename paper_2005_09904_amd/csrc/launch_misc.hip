// The small kernels: key packing, index extraction, tables to device memory, sum of partial
// results, quantiser.
#include "biq_launch.h"

#include "biq_quantize.h"

namespace biq {

hipError_t launch_reduce_splits(const float* partial, float* Y, long long count, int splits, hipStream_t s) {
    const bool vec4 = (count % 4 == 0) && ((reinterpret_cast<uintptr_t>(partial) & 15) == 0) &&
                      ((reinterpret_cast<uintptr_t>(Y) & 15) == 0);
    if (vec4)
        hipLaunchKernelGGL(reduce_splits_kernel<4>, dim3((unsigned)((count / 4 + 255) / 256)), dim3(256), 0, s,
                           partial, Y, count, splits);
    else
        hipLaunchKernelGGL(reduce_splits_kernel<1>, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s,
                           partial, Y, count, splits);
    return hipGetLastError();
}

hipError_t launch_pack(const int8_t* B, uint32_t* K, long long key_rows, int n, int stride_dw, hipStream_t s) {
    const long long total = key_rows * stride_dw;
    const unsigned grid = (unsigned)((total + 255) / 256);
    if (total < (1ll << 31) && key_rows * n < (1ll << 32))
        hipLaunchKernelGGL(pack_kernel<uint32_t>, dim3(grid), dim3(256), 0, s, B, K, (uint32_t)key_rows, n, stride_dw);
    else
        hipLaunchKernelGGL(pack_kernel<unsigned long long>, dim3(grid), dim3(256), 0, s, B, K, (unsigned long long)key_rows, n,
                           stride_dw);
    return hipGetLastError();
}

namespace {

template <typename KEY>
hipError_t launch_unpack_keys_t(int mu, const uint32_t* K, KEY* keys, long long key_rows, int C, int stride_dw,
                                hipStream_t s) {
#define BIQ_UNPACK_CASE(MU)                                                                          \
    case MU: {                                                                                       \
        const long long total = key_rows * ((C + KeyUnit<MU>::UK - 1) / KeyUnit<MU>::UK);            \
        hipLaunchKernelGGL((unpack_keys_kernel<MU, KEY>), dim3((unsigned)((total + 255) / 256)),     \
                           dim3(256), 0, s, K, keys, key_rows, C, stride_dw);                        \
        break;                                                                                       \
    }
    switch (mu) {
        BIQ_UNPACK_CASE(1) BIQ_UNPACK_CASE(2) BIQ_UNPACK_CASE(3) BIQ_UNPACK_CASE(4) BIQ_UNPACK_CASE(5)
        BIQ_UNPACK_CASE(6) BIQ_UNPACK_CASE(7) BIQ_UNPACK_CASE(8) BIQ_UNPACK_CASE(9) BIQ_UNPACK_CASE(10)
        default: return hipErrorInvalidValue;
    }
#undef BIQ_UNPACK_CASE
    return hipGetLastError();
}

}  // namespace

hipError_t launch_unpack_keys(int mu, bool wide_keys, const uint32_t* K, void* keys, long long key_rows, int C,
                              int stride_dw, hipStream_t s) {
    return wide_keys ? launch_unpack_keys_t<uint16_t>(mu, K, static_cast<uint16_t*>(keys), key_rows, C, stride_dw, s)
                     : launch_unpack_keys_t<uint8_t>(mu, K, static_cast<uint8_t*>(keys), key_rows, C, stride_dw, s);
}

hipError_t launch_build_lut(int mu, const float* X, float* LUT, int n, int batch, int C, hipStream_t s) {
    const int HG = mu > 4 ? (1 << (mu - 4)) : 1;
    const bool vec4 = (batch % 4 == 0) && ((reinterpret_cast<uintptr_t>(LUT) & 15) == 0);
    const int bv = vec4 ? batch / 4 : batch;
    // box of a workgroup: up to 64 vector groups, then key groups, then chunks, 256 threads in all
    int lta = 0, lth = 0;
    while (lta < 6 && (1 << lta) < bv) ++lta;
    while (lta + lth < 8 && (1 << lth) < HG) ++lth;
    const int ltc = 8 - lta - lth;
    const long long a_tiles = ((long long)bv + (1 << lta) - 1) >> lta;
    const long long h_tiles = ((long long)HG + (1 << lth) - 1) >> lth;
    const long long c_tiles = ((long long)C + (1 << ltc) - 1) >> ltc;
    const long long boxes = a_tiles * h_tiles * c_tiles;
    if (boxes > 0x7fffffffll) return hipErrorInvalidValue;
    const unsigned grid = (unsigned)boxes;
#define BIQ_LUT_CASE(MU)                                                                           \
    case MU:                                                                                       \
        if (vec4)                                                                                  \
            hipLaunchKernelGGL((build_lut_kernel<MU, 4>), dim3(grid), dim3(256), 0, s, X, LUT, n,  \
                               batch, C, lta, lth, ltc, (int)a_tiles, (int)h_tiles);               \
        else                                                                                       \
            hipLaunchKernelGGL((build_lut_kernel<MU, 1>), dim3(grid), dim3(256), 0, s, X, LUT, n,  \
                               batch, C, lta, lth, ltc, (int)a_tiles, (int)h_tiles);               \
        break;
    switch (mu) {
        BIQ_LUT_CASE(1) BIQ_LUT_CASE(2) BIQ_LUT_CASE(3) BIQ_LUT_CASE(4) BIQ_LUT_CASE(5)
        BIQ_LUT_CASE(6) BIQ_LUT_CASE(7) BIQ_LUT_CASE(8) BIQ_LUT_CASE(9) BIQ_LUT_CASE(10)
        default: return hipErrorInvalidValue;
    }
#undef BIQ_LUT_CASE
    return hipGetLastError();
}

hipError_t launch_quantize(const float* W, uint32_t* K, float* alpha, int m, int n, int q, int stride_dw,
                           hipStream_t s) {
    if (n > kQuantMaxN) return hipErrorInvalidValue;
    // 256-element pieces per wave: every count up to 16, even ones beyond (quant_shape)
    const QuantShape g = quant_shape(n);
    const dim3 grid((m + (4 / g.waves) - 1) / (4 / g.waves));
#define BIQ_QUANT_INST(NT, WPR, TAIL) \
    hipLaunchKernelGGL((quantize_wave_kernel<NT, WPR, TAIL>), grid, dim3(kQuantThreads), 0, s, W, K, alpha, m, n, q, stride_dw)
#define BIQ_QUANT_CASE(NT)                                                        \
    case NT:                                                                      \
        if (g.waves == 1 && g.tail == 0) BIQ_QUANT_INST(NT, 1, 0);                \
        else if (g.waves == 1) BIQ_QUANT_INST(NT, 1, quant_tail(NT));             \
        else if constexpr (NT > 8) {                                              \
            if (g.tail == 0) BIQ_QUANT_INST(NT, 4, 0);                            \
            else BIQ_QUANT_INST(NT, 4, quant_tail(NT));                           \
        }                                                                         \
        break;
    switch (g.pieces) {
        BIQ_QUANT_CASE(1) BIQ_QUANT_CASE(2) BIQ_QUANT_CASE(3) BIQ_QUANT_CASE(4) BIQ_QUANT_CASE(5) BIQ_QUANT_CASE(6)
        BIQ_QUANT_CASE(7) BIQ_QUANT_CASE(8) BIQ_QUANT_CASE(9) BIQ_QUANT_CASE(10) BIQ_QUANT_CASE(11) BIQ_QUANT_CASE(12)
        BIQ_QUANT_CASE(13) BIQ_QUANT_CASE(14) BIQ_QUANT_CASE(15) BIQ_QUANT_CASE(16) BIQ_QUANT_CASE(18) BIQ_QUANT_CASE(20)
        BIQ_QUANT_CASE(22) BIQ_QUANT_CASE(24) BIQ_QUANT_CASE(26) BIQ_QUANT_CASE(28) BIQ_QUANT_CASE(30) BIQ_QUANT_CASE(32)
        default: return hipErrorInvalidValue;
    }
#undef BIQ_QUANT_INST
#undef BIQ_QUANT_CASE
    return hipGetLastError();
}

}  // namespace biq
