// Many input vectors on the block-scaled matrix instructions (unpack_mfma plans with row_mode 1).
//
// The same contraction as biq_unpack_mfma.h - sign bits expanded to +-1 in registers, C = B_i . X on
// the matrix cores - with operands that cost a quarter of the matrix cycles per term: the weights are
// 4-bit floats (E2M1, +-1.0), the inputs 6-bit floats (E2M3) with one power-of-two scale per 32
// elements of an input vector.  v_mfma_scale_f32_32x32x64_f8f6f4 takes 33 clk here, as
// v_mfma_f32_32x32x16_bf16 does, for 64 instead of 16 elements of the contraction.
//
// Inputs.  A block of 32 elements is scaled so that its largest magnitude lies in [2, 4) and split
// into five digits, each rounded to nearest E2M3 (step 1/8 up to 2, 1/4 up to 4), digit j at scale
// 2^-5j: what a digit leaves is at most 1/8 of its scale = 4 of the next digit's, so the sum of the
// five misses the element by at most 2^-23 where the block's largest magnitude is at least 2:
// |error| <= 2^-24 of the block's largest magnitude - half a unit in the last place of that element,
// what adding the element to any fp32 sum that already holds the largest one would round off - and
// none for elements whose lowest set bit lies above that (the largest itself, integers, a one-hot
// vector).  The digits' scales are the instruction's scale operands.
// Two accumulators per tile, the first digits' and the others': a first digit is an integer below 2^5
// times its block's scale, so its sum is exact unless the blocks' scales differ widely, and
// the others' sum is 2^-5 of it, so its fp32 roundings weigh as little.  (One accumulator for all
// five: error 2.1e-7 instead of 5.8e-8 at 16384 x 4096; six digits: the same errors.)
// Relative 2-norm error against fp64, normal inputs, three bf16 terms -> digits: 16384 x 4096, 2
// planes, 128 vectors 4.2e-7 -> 5.8e-8; 4096 x 16384 5.9e-7 -> 6.6e-8; 4096^2, 3 planes, 32 vectors
// 2.2e-7 -> 7.4e-8 (the table kernels: 1.1e-7).
// Time, same order (us per call): 77 -> 43-46; 86 -> 50; 17.2 -> 13.3-13.9.  Bound by the power the matrix
// cores may draw: the instruction issues at 33 clk, but in a loop of nothing else the clock falls to
// 1.3-1.5 GHz, 5.1-5.8 PFLOP/s (bf16: 1.3-1.7 PFLOP/s), so fewer and cheaper instructions are what helps.
// The whole range of fp32 is covered: a block's scale byte stands for its exponent alone, and what the
// digits add to it - 2^-5j, which the byte could not hold for blocks below 2^-101 - is the scale of the
// WEIGHT operand, one constant per digit.  The first digits are summed at half their size: an element next
// to the largest fp32 rounds up to 2^128.  (The instruction keeps subnormal products and sums.)  A
// block that holds Inf or NaN gets the scale NaN, and the vector's results are NaN.
//
// Inputs that hold bf16 values (all elements of a key group - 256 - of all vectors of a column
// group) keep the one-term bf16 form: 16 elements per instruction, but one term instead of five digits
// (16384 x 4096, 2 planes, 128 vectors 33 us, 4096 x 16384 36-39: of 63 thousand clocks the vector ALU, which expands the
// weights, issues 40 and the matrix pipe is busy 33; what keeps the two from overlapping is not known).  Values of fp16 take all five digits.
// The form is chosen per (column group, key group) by the kernel that prepares the operands; the
// main kernel walks first the key groups of one form, then those of the other.
//
// Operand layout (32x32x64, lane = 32*h + r): A: row r, the 32 elements of key dword 8g + 4h + s
// of key group g at step s (0..3) - position 8i + j of the lane's 32 4-bit values is bit 4j + i of
// the dword: one shift and one v_and_or_b32 per 8 weights.  B: column r, the same 32 elements in
// the same order.  C as for 32x32x16.
//   Xd[column group][key group][column tile]: kDigitGroupBytes, holding either
//     [step 0..3][digit 0..4]: 64 lanes x 16 bytes, then 64 lanes x 8 bytes (dwords 0-3 and 4-5 of the
//     lane's 32 six-bit values), and behind the four steps 64 lanes x 4 scale bytes (one per step), or
//     [step 0..15]: 64 lanes x 16 bytes (bf16, the order of biq_unpack_mfma.h).
#pragma once

#include "biq_unpack_mfma.h"

namespace biq {

typedef int mfma_i32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t mfma_u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t mfma_u32x6 __attribute__((ext_vector_type(6)));
typedef float f32x32 __attribute__((ext_vector_type(32)));

constexpr int kDigits = 5;
constexpr int kDigitBytes = 64 * 24;                             // one digit of one step and column tile
constexpr int kDigitStepBytes = kDigits * kDigitBytes;
constexpr int kDigitScaleOffset = 4 * kDigitStepBytes;
constexpr int kDigitGroupBytes = kDigitScaleOffset + 64 * 4;     // 37120; the bf16 form takes 16384 of it
constexpr int kDigitMaxTiles = 8;                               // row x column tiles of a wave: 2 x 8 x 16 accumulator registers
constexpr int kFormDigits = 0, kFormBf16 = 1;                    // what a (column group, key group) holds
static_assert(kDigitGroupBytes <= 16 * 3 * 1024, "fits the area of the three-term fragments");

struct DigitParams {
    const uint8_t* K;        // [q][m][stride]
    const float* alpha;      // [q][m]
    const uint8_t* Xd;       // prepared B operands (see above)
    const int* form;         // [column group][key group]: kFormDigits or kFormBf16
    float* out;              // Y [batch][m], or partials [splits][batch][m]
    int m, batch;
    uint32_t stride_bytes;
    int groups;              // key groups per row = ceil(stride / 32)
    int gps;                 // key groups per split
    int splits;
    int row_blocks, col_groups;
    int ntasks, tasks_per_xcd;
};

// A block of 32 elements -> digits, handed to emit(d, 32 six-bit values in operand order) one after the
// other; returns the block's scale byte (digit d counts 2^-5d of it), 255 (NaN) for a block with Inf or NaN.
template <int UNROLL, typename Emit>
__device__ __forceinline__ uint32_t digit_split(const float (&x)[32], Emit&& emit) {
    // (the maximum that NaN passes on: two elements an instruction)
    float mx = 0.0f;
#pragma unroll
    for (int i = 0; i < 32; ++i) mx = __builtin_elementwise_maximum(mx, __builtin_fabsf(x[i]));
    const uint32_t mb = __float_as_uint(mx) & 0x7fffffffu;
    const bool finite = mb < 0x7f800000u;
    const int ex = max((int)(mb >> 23), 1);          // (subnormal elements: exponent as 1)
    const float norm = __uint_as_float((uint32_t)max(255 - ex, 1) << 23);   // 2^(128 - ex)
    f32x16 lo, hi;                                   // the 32 elements in operand order, even and odd positions
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int e = 8 * (u & 3) + (u >> 2);
        lo[u] = x[e] * norm;
        hi[u] = x[e + 4] * norm;
    }
    float scale = 1.0f;
#pragma unroll UNROLL
    for (int d = 0; d < kDigits; ++d) {
        const mfma_u32x6 p = __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(lo, hi, scale);
        emit(d, p);
        const f32x32 back = __builtin_amdgcn_cvt_scalef32_pk32_f32_fp6(p, scale);
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            lo[u] -= back[2 * u];
            hi[u] -= back[2 * u + 1];
        }
        scale *= 0.03125f;
    }
    return finite ? (uint32_t)(ex - 1) : 255u;
}

// One workgroup per (column tile, key group): 32 input vectors x 256 elements go through LDS (read along
// the vectors in whole KiB); thread = one block of 32 elements = one lane of one step's B operand.  Bound by
// latency (one load, ~350 instructions, one store), not by its 8.5 bytes per element.  Vectors past the
// batch and elements past n are zero.  The form holds for a column group: where that is two tiles, each
// workgroup looks at the other tile's elements too rather than being twice as large, with two waves on a
// SIMD (16384 x 4096, 2 planes, 128 vectors: the whole call 47.1 -> 46.3 us).
constexpr int kXdigitsPitch = 260;       // floats per vector in LDS: 16-byte rows, spread over the banks
template <int CT>
__global__ __launch_bounds__(256) void xdigits_kernel(const float* __restrict__ X, uint8_t* __restrict__ Xd,
                                                      int* __restrict__ form, int n, int batch, int groups) {
    __shared__ __align__(16) float xs[32 * kXdigitsPitch];
    __shared__ uint32_t votes[4];                    // one per wave
    const int g = (int)blockIdx.x % groups, tile = (int)blockIdx.x / groups;
    const int cg = tile / CT, c = tile % CT;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    {
        // wave w reads vectors 8w .. 8w + 7, all requests in flight together
        // (a buffer per vector: elements past n, and all of a vector past the batch, read as 0.  Reads behind
        // conditions were waited for one by one: odd n 5.1 -> 3.5 us)
        mfma_u32x4 v[8], u[8] = {};
        auto load = [&](int t, mfma_u32x4 (&to)[8]) {
            const int col0 = t * 32 + wave * 8;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int col = min(col0 + i, batch - 1);
                const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<float*>(X + (size_t)col * n), 0, col0 + i < batch ? n * 4 : 0, 0x00020000);
                to[i] = __builtin_bit_cast(mfma_u32x4, __builtin_amdgcn_raw_buffer_load_b128(src, 1024 * g + 16 * lane, 0, 0));
            }
        };
        load(tile, v);
        if constexpr (CT == 2) load(tile ^ 1, u);
        uint32_t low = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            *reinterpret_cast<mfma_u32x4*>(xs + (wave * 8 + i) * kXdigitsPitch + 4 * lane) = v[i];
            low |= v[i].x | v[i].y | v[i].z | v[i].w;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) low |= u[i].x | u[i].y | u[i].z | u[i].w;
        bool wave_bf16 = __builtin_amdgcn_ballot_w64((low & 0xffffu) != 0u) == 0ull;
        if (wave_bf16) {                             // ... unless there is Inf or NaN
            uint32_t mb = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int k = 0; k < 4; ++k) mb = max(mb, max(v[i][k] & 0x7fffffffu, u[i][k] & 0x7fffffffu));
            wave_bf16 = __builtin_amdgcn_ballot_w64(mb >= 0x7f800000u) == 0ull;
        }
        if (lane == 0) votes[wave] = wave_bf16;
    }
    __syncthreads();
    const int s = wave;                              // step within the key group
    const int h = lane >> 5, r = lane & 31;
    float x[32];
    {
        const float* src = xs + r * kXdigitsPitch + 32 * (4 * h + s);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float4 v = *reinterpret_cast<const float4*>(src + 4 * i);
            x[4 * i] = v.x; x[4 * i + 1] = v.y; x[4 * i + 2] = v.z; x[4 * i + 3] = v.w;
        }
    }
    const bool all_bf16 = votes[0] && votes[1] && votes[2] && votes[3];
    uint8_t* const area = Xd + ((size_t)(cg * groups + g) * CT + c) * kDigitGroupBytes;
    if (tid == 0 && c == 0) form[cg * groups + g] = all_bf16 ? kFormBf16 : kFormDigits;
    if (all_bf16) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            mfma_u32x4 d;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                d[i] = (__float_as_uint(x[4 * ks + i]) >> 16) | (__float_as_uint(x[4 * ks + i + 16]) & 0xffff0000u);
            *reinterpret_cast<mfma_u32x4*>(area + (4 * s + ks) * 1024 + lane * 16) = d;
        }
        return;
    }
    area[kDigitScaleOffset + lane * 4 + s] = (uint8_t)digit_split<kDigits>(x, [&](int d, const mfma_u32x6& p) {
        uint8_t* dst = area + s * kDigitStepBytes + d * kDigitBytes;
        mfma_u32x4 p0;
        p0.x = p[0]; p0.y = p[1]; p0.z = p[2]; p0.w = p[3];
        mfma_u32x2 p1;
        p1.x = p[4]; p1.y = p[5];
        *reinterpret_cast<mfma_u32x4*>(dst + lane * 16) = p0;
        *reinterpret_cast<mfma_u32x2*>(dst + 1024 + lane * 8) = p1;
    });
}

// Key dword -> the lane's 32 A values +-1.0 (E2M1: 0x2 / 0xa), with the OPPOSITE sign as in
// unpack_step: 4 dwords, value j of dword i is bit 4j + i.
__device__ __forceinline__ mfma_u32x4 unpack_nibbles(uint32_t w, uint32_t one8) {
    mfma_u32x4 d;
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = ((w << (3 - i)) & 0x88888888u) | one8;
    return d;
}

// Scale bytes of the weights for the digits 0-3 and for digit 4 (see the top of the file).
constexpr uint32_t kDigitWeightScales = 126u | (127u - 5u) << 8 | (127u - 10u) << 16 | (127u - 15u) << 24;
constexpr uint32_t kDigitWeightScale4 = 127u - 20u;

// 64 k of one row tile x one column tile: E2M1 weights (scale byte A of `wscale`) x one E2M3 digit (byte B of `scale`).
template <int A, int B>
__device__ __forceinline__ f32x16 digit_mfma(const mfma_u32x4& a, const mfma_u32x6& b, f32x16 c, uint32_t wscale,
                                             uint32_t scale) {
    mfma_i32x8 av = {}, bv = {};
#pragma unroll
    for (int i = 0; i < 4; ++i) av[i] = (int)a[i];
#pragma unroll
    for (int i = 0; i < 6; ++i) bv[i] = (int)b[i];
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, c, 4, 2, A, (int)wscale, B, (int)scale);
}

// Workgroup = 4 waves; WS of them share a row block along the contraction (each its own part of the
// key groups), 4 / WS stand side by side along the rows.  A wave owns RT = Q * RPW row tiles (all
// planes of its 32 * RPW output rows) x CT column tiles, at most 8: two accumulators of 16 registers
// each, 256 in all.  (16 tiles with one accumulator each were never the fastest mapping.)
template <int RPW, int CT, int WS>
struct DigitGeom {
    static constexpr int WROWS = 4 / WS;
    static constexpr int NOUT = RPW * CT;                          // output tiles of a wave
    static constexpr int RED_FLOATS = WS == 1 ? 0 : WROWS * NOUT * (WS - 1) * 1024;
    static constexpr int TP = 36;                                  // pitch of a transpose patch in floats
    static constexpr int LDS_BYTES = (RED_FLOATS + 4 * 32 * TP + 4 * 256) * 4;   // ... and the scales of 8 row tiles per wave
};

template <int Q, int RPW, int CT, int WS>
__global__ __launch_bounds__(kUnpackThreads, 1) void digit_mfma_kernel(const DigitParams p) {
    using G = DigitGeom<RPW, CT, WS>;
    constexpr int RT = Q * RPW, WROWS = G::WROWS, NOUT = G::NOUT;
    extern __shared__ __align__(16) mfma_u32x4 stage_buf[];

    const int wg = blockIdx.x;
    const int task = (wg & 7) * p.tasks_per_xcd + (wg >> 3);
    if (task >= p.ntasks) return;
    const int cg = task % p.col_groups;
    const int rest = task / p.col_groups;
    const int sp = rest % p.splits;
    const int rb = rest / p.splits;
    const int g0 = sp * p.gps;
    const int g1 = min(p.groups, g0 + p.gps);
    const int per = (g1 - g0 + WS - 1) / WS;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = wave / WROWS;
    const int wrow = wave % WROWS;
    const int h = lane >> 5;
    const int lr = lane & 31;
    const int ga = g0 + kg * per;                     // this wave's key groups [ga, gb)
    const int gb = min(g1, ga + per);

    const int rbase = rb * (WROWS * 32 * RPW) + wrow * (32 * RPW);
    // Unconditional, from clamped addresses (see biq_unpack_mfma.h); rows past m read the last row and
    // are never stored, keys past the row meet zeros.  Wave-uniform base + 32-bit lane offset: 64-bit
    // pointers per row tile would not fit beside 16 accumulators.
    auto load_keys = [&](int g, mfma_u32x4 (&k)[RT]) {
        const uint32_t want = (uint32_t)(32 * g + 16 * h);
        const uint32_t off = want < p.stride_bytes ? want : 0u;
#pragma unroll
        for (int i = 0; i < Q; ++i)
#pragma unroll
            for (int rp = 0; rp < RPW; ++rp) {
                const int row0 = min(rbase + rp * 32, p.m - 1);
                const uint8_t* base = p.K + ((size_t)i * p.m + row0) * p.stride_bytes;
                const uint32_t lane_off = (uint32_t)min(lr, p.m - 1 - row0) * p.stride_bytes + off;
                k[i * RPW + rp] = *reinterpret_cast<const mfma_u32x4*>(base + lane_off);
            }
    };

    // first digits at half their size, other digits: see the top of the file (bf16 terms: even and odd steps)
    f32x16 acc[RT][CT], acl[RT][CT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][c][v] = acl[t][c][v] = 0.0f;

    // the scales of the wave's RT * 32 key rows: requested here, in LDS from the form votes on
    constexpr int NA = (RT * 32 + 63) / 64;
    float av[NA];
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        const int t = min((64 * j + lane) >> 5, RT - 1);
        const int row = min(rbase + (t % RPW) * 32 + lr, p.m - 1);
        av[j] = p.alpha[(size_t)(t / RPW) * p.m + row];
    }

    const uint8_t* const xw = p.Xd + (size_t)cg * p.groups * CT * kDigitGroupBytes;   // wave-uniform
    mfma_u32x4 key[RT], keyn[RT];

    // ---- digits: the key groups ga + i for the bits i of `todo`.
    // Order of a step: digit by digit over all tiles (the same accumulator comes up again RT * CT
    // instructions later).  A digit's registers are requested again for the next step as soon as
    // its last instruction is issued, four digits ahead of their use: one set of B registers is enough
    // (two sets, requested two steps ahead, where up to 4 tiles leave room: no faster on 30 shapes).  The
    // next step's A operands replace a tile's during the last digit.  The fences
    // keep this order: left alone, the compiler clumps the expansions and drains the loads.
    auto walk_digits = [&](unsigned long long todo, bool have_keys) {
        uint32_t one8 = 0x22222222u, wsc = kDigitWeightScales, wsc4 = kDigitWeightScale4;
        asm volatile("" : "+v"(one8), "+v"(wsc), "+v"(wsc4));
        mfma_u32x6 b[kDigits][CT];
        uint32_t sc[CT], scn[CT];
        auto area = [&](int g, int c) { return xw + (size_t)(g * CT + c) * kDigitGroupBytes; };
        auto load_digit = [&](int g, int s, int d) {
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const uint8_t* src = area(g, c) + s * kDigitStepBytes + d * kDigitBytes;
                const mfma_u32x4 p0 = *reinterpret_cast<const mfma_u32x4*>(src + lane * 16);
                const mfma_u32x2 p1 = *reinterpret_cast<const mfma_u32x2*>(src + 1024 + lane * 8);
#pragma unroll
                for (int i = 0; i < 4; ++i) b[d][c][i] = p0[i];
                b[d][c][4] = p1[0];
                b[d][c][5] = p1[1];
            }
        };
        auto load_scales = [&](int g, uint32_t (&v)[CT]) {
#pragma unroll
            for (int c = 0; c < CT; ++c) v[c] = *reinterpret_cast<const uint32_t*>(area(g, c) + kDigitScaleOffset + lane * 4);
        };
        int g = ga + __builtin_ctzll(todo);
        if (!have_keys) load_keys(g, key);
        load_scales(g, sc);
#pragma unroll
        for (int d = 0; d < kDigits; ++d) load_digit(g, 0, d);
        mfma_u32x4 a[RT];
#pragma unroll
        for (int t = 0; t < RT; ++t) a[t] = unpack_nibbles(key[t][0], one8);
        do {
            todo &= todo - 1;
            const int gn = todo ? ga + __builtin_ctzll(todo) : g;    // after the last group: that group again, unused
            __builtin_amdgcn_sched_barrier(0);
            load_keys(gn, keyn);
            load_scales(gn, scn);
            __builtin_amdgcn_sched_barrier(0);
            auto step = [&](auto st) {
                constexpr int S = decltype(st)::value;
                auto digit = [&](auto dc) {
                    constexpr int D = decltype(dc)::value;
#pragma unroll
                    for (int t = 0; t < RT; ++t) {
#pragma unroll
                        for (int c = 0; c < CT; ++c) {
                            f32x16& sum = D == 0 ? acc[t][c] : acl[t][c];
                            sum = digit_mfma<D & 3, S>(a[t], b[D][c], sum, D < 4 ? wsc : wsc4, sc[c]);
                        }
                        if constexpr (D == kDigits - 1) a[t] = unpack_nibbles(S < 3 ? key[t][(S + 1) & 3] : keyn[t][0], one8);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    load_digit(S < 3 ? g : gn, (S + 1) & 3, D);
                    __builtin_amdgcn_sched_barrier(0);
                };
                digit(std::integral_constant<int, 0>{});
                digit(std::integral_constant<int, 1>{});
                digit(std::integral_constant<int, 2>{});
                digit(std::integral_constant<int, 3>{});
                digit(std::integral_constant<int, 4>{});
            };
            step(std::integral_constant<int, 0>{});
            step(std::integral_constant<int, 1>{});
            step(std::integral_constant<int, 2>{});
            step(std::integral_constant<int, 3>{});
#pragma unroll
            for (int t = 0; t < RT; ++t) key[t] = keyn[t];
#pragma unroll
            for (int c = 0; c < CT; ++c) sc[c] = scn[c];
            g = gn;
        } while (todo);
    };

    // ---- bf16 values (key groups as above): one term, 16 steps of 16 elements per key group, fragments seven steps ahead in
    // a ring of eight (see biq_unpack_mfma.h).
    auto walk_bf16 = [&](unsigned long long todo, bool have_keys) {
        uint32_t one2 = 0x3f803f80u, half2 = 0x3f003f00u;    // odd steps; even steps, whose sums count twice
        asm volatile("" : "+v"(one2), "+v"(half2));
        constexpr int R = 8;
        bf16x8 ring[R][CT];
        bf16x8 a[RT];
        auto load_b = [&](int g, int st, bf16x8 (&b)[CT]) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
                b[c] = *reinterpret_cast<const bf16x8*>(xw + (size_t)(g * CT + c) * kDigitGroupBytes + st * 1024 + lane * 16);
        };
        auto expand = [&](const mfma_u32x4& k, int st) {
            const uint32_t w = k[(st >> 2) & 3];
            const int ks = st & 3;
            return ks == 0 ? unpack_step<0, bf16x8>(w, half2) : ks == 1 ? unpack_step<1, bf16x8>(w, one2)
                 : ks == 2 ? unpack_step<2, bf16x8>(w, half2) : unpack_step<3, bf16x8>(w, one2);
        };
        int g = ga + __builtin_ctzll(todo);
        if (!have_keys) load_keys(g, key);
#pragma unroll
        for (int j = 0; j + 1 < R; ++j) load_b(g, j, ring[j]);
#pragma unroll
        for (int t = 0; t < RT; ++t) a[t] = expand(key[t], 0);
        do {
            todo &= todo - 1;
            const int gn = todo ? ga + __builtin_ctzll(todo) : g;    // after the last group: that group again, unused
            __builtin_amdgcn_sched_barrier(0);
            load_keys(gn, keyn);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int st = 0; st < 16; ++st) {
                load_b(st + R - 1 < 16 ? g : gn, (st + R - 1) & 15, ring[(st + R - 1) & (R - 1)]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < RT; ++t) {
#pragma unroll
                    for (int c = 0; c < CT; ++c) {
                        f32x16& sum = st & 1 ? acl[t][c] : acc[t][c];      // shorter sums: fewer roundings each
                        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t], ring[st & (R - 1)][c], sum, 0, 0, 0);
                    }
                    a[t] = st < 15 ? expand(key[t], st + 1) : expand(keyn[t], 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int t = 0; t < RT; ++t) key[t] = keyn[t];
            g = gn;
        } while (todo);
    };

    float* const red = reinterpret_cast<float*>(stage_buf);
    float* const patch = red + G::RED_FLOATS + wave * (32 * G::TP);
    float* const scales = red + G::RED_FLOATS + 4 * 32 * G::TP + wave * (RT * 32);   // -alpha of the wave's rows
    auto store_scales = [&] {
#pragma unroll
        for (int j = 0; j < NA; ++j)
            if (64 * j + lane < RT * 32) scales[64 * j + lane] = -av[j];
    };
    // the wave's key groups (at most 64) by form: first those in digits, then those in bf16
    if (ga < gb) {
        const int cnt = gb - ga;
        const int f = p.form[(size_t)cg * p.groups + ga + min(lane, cnt - 1)];
        load_keys(ga, key);    // the first group's keys do not wait for the forms, which mostly are one form anyway
        __builtin_amdgcn_sched_barrier(0);
        const unsigned long long all = cnt < 64 ? (1ull << cnt) - 1 : ~0ull;
        const unsigned long long bf = __builtin_amdgcn_ballot_w64(f == kFormBf16) & all;
        store_scales();    // they came before the forms, so nothing waits here (held in registers, they spilled)
        if (bf != all) walk_digits(all & ~bf, !(bf & 1));
        if (bf) walk_bf16(bf, bf == all);
    } else {
        store_scales();
    }

    // ---- epilogue: -alpha scale and plane sum (Eq. 2) on the wave's part of the contraction, then the
    // WS parts are added through LDS - output tile o by wave group o % WS, so that all waves take a
    // share of it - and each tile leaves through a transpose patch in 128-byte runs.
    // (lane numbers counted anew: kept, they would be spilled over the loops)
    const int elane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const int eh = elane >> 5, elr = elane & 31;
    const bool vec_ok = ((p.m & 3) == 0) && ((reinterpret_cast<uintptr_t>(p.out) & 15) == 0);
#pragma unroll
    for (int rp = 0; rp < RPW; ++rp)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                float v = 0.0f;
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    const int t = i * RPW + rp;
                    v = fmaf(scales[t * 32 + 8 * (j >> 2) + 4 * eh + (j & 3)], fmaf(2.0f, acc[t][c][j], acl[t][c][j]), v);
                }
                acc[rp][c][j] = v;                    // plane 0's accumulator takes the sum
            }
            // tile by tile, scales read and sums finished: the registers are full (left to itself, the compiler reads
            // all scales first and finishes the sums where they are used)
            asm volatile("" : "+v"(acc[rp][c]) : : "memory");
        }
    if constexpr (WS > 1) {
#pragma unroll
        for (int o = 0; o < NOUT; ++o) {
            const int owner = o % WS;
            if (kg != owner) {
                const int slot = ((wrow * NOUT + o) * (WS - 1)) + (kg > owner ? kg - 1 : kg);
                float4* dst = reinterpret_cast<float4*>(red + (size_t)slot * 1024) + elane;
                const f32x16& v = acc[o / CT][o % CT];
#pragma unroll
                for (int vq = 0; vq < 4; ++vq) dst[vq * 64] = make_float4(v[4 * vq], v[4 * vq + 1], v[4 * vq + 2], v[4 * vq + 3]);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int o = 0; o < NOUT; ++o) {
        if (kg != o % WS) continue;
        const int rp = o / CT, c = o % CT;
        f32x16& y = acc[rp][c];
        if constexpr (WS > 1) {
#pragma unroll
            for (int j = 0; j < WS - 1; ++j) {
                const int slot = ((wrow * NOUT + o) * (WS - 1)) + j;
                const float4* src = reinterpret_cast<const float4*>(red + (size_t)slot * 1024) + elane;
#pragma unroll
                for (int vq = 0; vq < 4; ++vq) {
                    const float4 v = src[vq * 64];
                    y[4 * vq] += v.x; y[4 * vq + 1] += v.y; y[4 * vq + 2] += v.z; y[4 * vq + 3] += v.w;
                }
            }
        }
#pragma unroll
        for (int vq = 0; vq < 4; ++vq)
            *reinterpret_cast<float4*>(patch + elr * G::TP + 8 * vq + 4 * eh) =
                make_float4(y[4 * vq], y[4 * vq + 1], y[4 * vq + 2], y[4 * vq + 3]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int pc = 8 * i + (elane >> 3);
            const int pr = 4 * (elane & 7);
            const float4 v = *reinterpret_cast<const float4*>(patch + pc * G::TP + pr);
            const int col = (cg * CT + c) * 32 + pc;
            const int row = rbase + rp * 32 + pr;
            if (col < p.batch && row < p.m) {
                float* dst = p.out + ((size_t)sp * p.batch + col) * p.m + row;
                if (vec_ok && p.splits == 1) {
                    // (written through: 8 MB left in the L2s for the end of the kernel took 0.5-1 us more)
                    typedef float f32x4o __attribute__((ext_vector_type(4)));
                    __builtin_nontemporal_store(f32x4o{v.x, v.y, v.z, v.w}, reinterpret_cast<f32x4o*>(dst));
                } else if (vec_ok) {
                    *reinterpret_cast<float4*>(dst) = v;
                } else {
                    dst[0] = v.x;
                    if (row + 1 < p.m) dst[1] = v.y;
                    if (row + 2 < p.m) dst[2] = v.z;
                    if (row + 3 < p.m) dst[3] = v.w;
                }
            }
        }
    }
}

}  // namespace biq
