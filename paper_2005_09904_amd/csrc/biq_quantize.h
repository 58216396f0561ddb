// Binary-coding quantisation of a weight matrix, row by row (Sec. II-B, Eq. 1):
// w ~ sum_i alpha_i b_i, b_i in {-1,+1}^n.  The paper only names the heuristic ("greedy
// approximation"); this is the greedy procedure Eq. 1 suggests, one plane at a time on the
// residual r (r = w at the start):
//     b_i = sign(r) (sign(0) = +1),  alpha_i = mean |r|,  r <- r - alpha_i b_i
// Each step is the exact minimiser of Eq. 1 for q = 1 applied to the residual.  The signs are
// written straight in the packed key format (bit j of the row <-> element j, +1 <-> 1), the
// scales as alpha[q][m]: the outputs feed biq_gemm without a pass over int8 signs.
//
// The residual lives in registers.  Rows up to 8192 elements: one wave per row, no barriers.  Longer
// rows (up to 32768): the four waves of a workgroup share a row, one barrier per plane for the sum.  Sums
// are taken in a fixed order (four chains per lane over its elements, then a butterfly inside the
// wave, then over the waves), so the result does not depend on timing.
//
// Bound by memory (4 bytes in, q / 8 out per element) once the arithmetic is short enough: per element
// and plane one add of |r|, one v_alignbit that shifts the sign into the lane's key bits, one
// v_bfi and one subtraction.  A lane reads 16 bytes at a time (a wave a whole KiB), so it holds 4
// neighbours of every 256; eight such nibbles fill a register, and an 8 x 8 transpose of nibbles over 8
// lanes (three exchanges, 8 instructions per 32 elements) makes them key dwords.  Before, a ballot per
// 64 elements went through LDS, written by one lane at a time.  Before -> now: 4096^2, 3 planes 31.1 ->
// 14.6 us (5.0 TB/s), 16384 x 4096, 2 planes 69 -> 42.7 (6.7 TB/s), 4096 x 6000, 4 planes 126 -> 32.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "biq_quantize_shape.h"

namespace biq {

constexpr int kQuantThreads = 256;

// Lane i gets lane i ^ 1's / i ^ 2's / i ^ 4's value.
__device__ __forceinline__ uint32_t quant_xor1(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true); }
__device__ __forceinline__ uint32_t quant_xor2(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true); }
__device__ __forceinline__ uint32_t quant_xor4(uint32_t v) {
    const int m = __builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true);              // row_half_mirror: i ^ 7
    return (uint32_t)__builtin_amdgcn_update_dpp(0, m, 0x1B, 0xf, 0xf, true);                 // quad_perm [3,2,1,0]: i ^ 3
}

// WPR waves per row (1: four rows per workgroup; 4: one row per workgroup), NT pieces of 256 elements per wave:
// n <= 256 * NT * WPR.  Lane l of wave w (of the row's WPR waves) holds elements
// (t * WPR + w) * 256 + 4 l + c, t = 0 .. NT - 1, c = 0 .. 3.  TAIL: the pieces of a wave, the last ones, that may hold
// fewer than 256 or lie past the row (0: n = 256 * NT * WPR); only their residuals are masked, two of six instructions per element and plane.
// An instance for nearly every NT: a row of few pieces more than a power of two does not pay for twice as many (777 x 4560, 4 planes,
// before with 32 pieces: 10.2 -> 6.5 us; 2629 x 4681, 4 23.3 -> 15.0; 7182 x 558, 4 8.4 -> 6.5; 4096^2 as before).
template <int NT, int WPR, int TAIL>
__global__ __launch_bounds__(kQuantThreads) void quantize_wave_kernel(const float* __restrict__ W,
                                                                      uint32_t* __restrict__ K,
                                                                      float* __restrict__ alpha, int m,
                                                                      int n, int q, int stride_dw) {
    constexpr int NG = (NT + 7) / 8;   // groups of up to 8 pieces = 32 sign bits
    __shared__ float wave_sums[2][4];   // WPR = 4: the waves' partial sums, double buffered over the planes
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (the row's buffer lies in scalar registers)
    const int wsub = wave % WPR;
    const int row = blockIdx.x * (kQuantThreads / 64 / WPR) + wave / WPR;
    if (row >= m) return;   // WPR = 4: whole workgroup
    // all loads in flight together; a buffer of the row's n elements: past its end they read as 0
    const __amdgpu_buffer_rsrc_t src =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(W + (size_t)row * n), 0, n * 4, 0x00020000);
    typedef uint32_t u32x4q __attribute__((ext_vector_type(4)));
    float r[NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const u32x4q v = __builtin_bit_cast(u32x4q, __builtin_amdgcn_raw_buffer_load_b128(
            src, (t * WPR + wsub) * 1024 + 16 * lane, 0, 0));
#pragma unroll
        for (int c = 0; c < 4; ++c) r[t][c] = __uint_as_float(v[c]);
    }
    __builtin_amdgcn_sched_barrier(0);
    // (+ 0.0f turns a weight of -0.0 into +0.0 and changes nothing else; a residual is never -0.0
    // afterwards (x - x = +0.0 under round-to-nearest), so the sign bit of r is exactly "r < 0" and
    // sign(0) = +1 as in Eq. 1's reading: the code and the residual update below agree)
    float s4[4] = {};
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            r[t][c] += 0.0f;
            s4[c] += fabsf(r[t][c]);
        }
    // which of a lane's sign bits belong to elements (bit 4 t + c of group t / 8)
    uint32_t there[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        there[g] = 0;
#pragma unroll
        for (int t = 8 * g; t < 8 * g + 8 && t < NT; ++t) {
            const int left = n - ((t * WPR + wsub) * 256 + 4 * lane);    // elements from this piece on
            there[g] |= (left >= 4 ? 15u : left > 0 ? (1u << left) - 1u : 0u) << (4 * (t & 7));
        }
    }
    // 8 x 8 nibbles: selectors of this lane's part of the three exchanges
    const uint32_t sel4 = lane & 4 ? 0x07060302u : 0x01000504u;      // (own, partner): halves
    const uint32_t sel2 = lane & 2 ? 0x07030501u : 0x02060004u;      // bytes
    const uint32_t rot1 = lane & 1 ? 4u : 28u;                       // nibbles
    const uint32_t keep1 = lane & 1 ? 0xf0f0f0f0u : 0x0f0f0f0fu;
    for (int i = 0; i < q; ++i) {
        float s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
        if constexpr (WPR > 1) {
            if (lane == 0) wave_sums[i & 1][wave] = s;
            __syncthreads();
            s = ((wave_sums[i & 1][0] + wave_sums[i & 1][1]) + wave_sums[i & 1][2]) + wave_sums[i & 1][3];
        }
        const float a = s / (float)n;
        if (lane == 0 && wsub == 0) alpha[(size_t)i * m + row] = a;
        uint32_t* krow = K + ((size_t)i * m + row) * stride_dw;
        // sign bits, highest element first, so that element (t, c) ends at bit 4 t + c
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            uint32_t neg = 0;
#pragma unroll
            for (int u = 31; u >= 0; --u)
                if (8 * g + (u >> 2) < NT)
                    neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(r[8 * g + (u >> 2)][u & 3]), 31);
            uint32_t w = ~neg & there[g];
            w = __builtin_amdgcn_perm(w, quant_xor4(w), sel4);
            w = __builtin_amdgcn_perm(w, quant_xor2(w), sel2);
            const uint32_t o = quant_xor1(w);
            w = (w & keep1) | (__builtin_amdgcn_alignbit(o, o, rot1) & ~keep1);
            // lane 8 h + l now holds piece t = 8 g + l of lanes 8 h .. 8 h + 7: 32 consecutive elements
            const int t = 8 * g + (lane & 7);
            const int dw = (t * WPR + wsub) * 8 + (lane >> 3);
            if (t < NT && dw < stride_dw) krow[dw] = w;
        }
        if (i + 1 == q) break;
        // r -= copysign(a, r), and the next plane's sum; elements past n stay 0
#pragma unroll
        for (int c = 0; c < 4; ++c) s4[c] = 0.0f;
        uint32_t valid[NG];
        if constexpr (TAIL > 0) {
#pragma unroll
            for (int g = (NT - TAIL) / 8; g < NG; ++g) {
                valid[g] = there[g];
                // (kept from being turned into one condition per element in scalar registers, outside the loop)
                asm volatile("" : "+v"(valid[g]));
            }
        }
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t b = __float_as_uint(r[t][c]);
                float x = r[t][c] - __uint_as_float((b & 0x80000000u) | (__float_as_uint(a) & 0x7fffffffu));
                if (t >= NT - TAIL)     // all ones or zero from the element's bit
                    x = __uint_as_float(__float_as_uint(x) &
                                        (uint32_t)__builtin_amdgcn_sbfe((int)valid[t >> 3], 4 * (t & 7) + c, 1));
                r[t][c] = x;
                s4[c] += fabsf(x);
            }
    }
}

}  // namespace biq
