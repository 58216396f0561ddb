// Few input vectors on the block-scaled matrix instructions, one dispatch, no tables.
//
// A workgroup turns its input vectors into the operands of v_mfma_scale_f32_16x16x128_f8f6f4 once - for
// all of the row, in LDS - and then streams keys: a key dword is 32 weights of one row and becomes 32
// 4-bit floats +-1.0 in 8 instructions (see unpack_nibbles), which one matrix instruction multiplies
// with 16 columns.  Where a 128 KiB set of tables costs a workgroup 1.3 us (half) to 3 us (full) per
// 2048 / 1024 columns and vector - a pair of vectors at half that width - the operands of a vector are
// 3.75 bytes per element, and one walk over the keys serves up to 16 vectors.
//
// Columns = digits of vectors.  An input element is the sum of five 6-bit floats (digit_split below):
// the five digits of a vector are five columns, three vectors fill a 16-column tile (the last column is
// idle), and every column has an accumulator of its own.  A digit is a small integer times its
// block's scale, so a column's sum is exact unless the magnitudes of its blocks differ by more
// than about 2^12; the five sums of a vector meet at the very end, smallest first.  Error against fp64:
// the input rounding (2^-24 of the largest of 32 elements) and a handful of fp32 roundings.
// All digits of a block share its scale byte, which covers every fp32 exponent; a column's own 2^-5j is
// put on its finished sums.  The later digits' sums, 2^5j too large until then, are kept from
// overflowing by weights of +-2^-6: a digit is at most 4, twice the block's largest element at
// most, so 32 of them are at most 2^6 times that one.  (Inputs below 2^-120: sums rounded to 2^-143.)
//
// Bounds.  Matrix pipe: 16 clk per 16 rows x 128 columns x 3 vectors; VALU: 8 instructions per key
// dword, 32 clk for the 64 lanes' 256 bytes of keys on each of 1024 SIMDs = 17 TB/s of keys, above what
// memory delivers; LDS: 24 bytes per lane and column tile and step, shared by the wave's RT row tiles.
// What a call takes is mostly latency: X, the split (about 300 instructions per block of 32
// elements), one barrier, keys and LDS reads behind each other: 3.5 us and up.  us per call, keys from memory,
// before -> here: 5003 x 3001, 3 planes, 7 vectors at mu = 6 13.1 (three bf16 terms 16.3) -> 9.2; 5000 x 3001, 3, 1
// 11.9 -> 6.4; 10240 x 1216, 2, 12 17.6 -> 8.6; 32000 x 1024, 3, 6 18.6 -> 7.0; 1790 x 316, 3, 5 at mu = 7 18.6 -> 4.7.
// With 4 planes and 10-15 vectors, keys on chip: 20000 x 700 9.3, 10000 x 2000 10.3.
// Errors 4-9e-8 instead of 0.8-1.3e-7 (tables).  One vector, 2 planes, tables / direct: 4096 x 4096 6.6 / 5.0, 16384 x 4096
// 8.6 / 7.7 (keys on chip 7.2 / 5.4).  Not taken for one vector where a table workgroup covers the row (2048 x 2048, 2:
// 3.9 / 4.6).  Small layers with several vectors go either way (tables / direct: 919 x 832, 3, 9 4.6 / 6.5; 1024 x 512, 2, 3 4.5 / 3.9).
// (Two chunks requested together with one row tile per wave, several groups of waves: 16384 x 4096 8.3 -> 7.7 us, but
// 5000 x 3001 6.4 -> 7.8, both with one row step per workgroup: a mapping for more than 256 row tiles, where it is
// estimated faster.)
//
// Layout.  Operand lane 16 * kg + r: row / column r, the 32 elements of one key dword.  A lane loads
// 16 key bytes, [64 j + 16 kg, +16) of its row ("chunk" j = 512 elements): four lanes cover 64
// contiguous bytes, and dword s of the 16 bytes is step s = elements [32 (16 j + 4 kg + s), +32).
// LDS: digits [vector][block of 32][digit] 24 bytes, scale bytes [vector][block].  A vector's digits end
// with 8 bytes of padding: the 15 columns of a tile then read 64-bit pieces at dwords 6 d + 2 v (+ 0, 1) of
// the 32 banks, all different, and consecutive blocks, written by consecutive lanes, lie 30 dwords apart.
#pragma once

#include "biq_digit_mfma.h"
#include "biq_direct_rule.h"

namespace biq {

static_assert(kDirectDigits == kDigits && kDirectWaves * 64 == kDirectThreads, "as the rule counts them");

struct DirectParams {
    const uint8_t* K;        // [q][m][stride]
    const float* alpha;      // [q][m]
    const float* X;          // [batch][n]
    float* out;              // Y [batch][m]
    int m, n, batch;
    uint32_t stride_bytes;
    int chunks;              // chunks of 512 elements per row
    uint32_t chunks_inv;     // ceil(2^32 / chunks), chunks > 1: g / chunks = (g * chunks_inv) >> 32 for g * chunks < 2^32
    int vecs;                // vectors per workgroup (grid: x = row blocks, y = batch tiles)
    int log_ksplit;          // 2^log_ksplit groups of waves along the row
    int units_per_group;     // units (UC chunks) of a group
    int steps;               // row steps of a workgroup; a step = (8 / ksplit) * RPW * 16 rows
};

typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));   // 128-bit access, any float address
typedef float f32x4v __attribute__((ext_vector_type(4)));

constexpr int kDirectWeightShift = 6;                // the weights are +-2^-6 (see the top of the file)

// 16 rows x 128 elements x 16 columns; scale byte S of `scale`.
template <int S>
__device__ __forceinline__ f32x4v direct_mfma(const mfma_u32x4& a, const mfma_u32x6& b, f32x4v c, uint32_t scale) {
    mfma_i32x8 av = {}, bv = {};
#pragma unroll
    for (int i = 0; i < 4; ++i) av[i] = (int)a[i];
#pragma unroll
    for (int i = 0; i < 6; ++i) bv[i] = (int)b[i];
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(av, bv, c, 4, 2, 0, 127 - kDirectWeightShift, S, (int)scale);
}

// Lanes 32-63 of a <-> lanes 0-31 of b; odd rows of 16 lanes of a <-> even rows of b.
__device__ __forceinline__ void swap_lanes32(float& a, float& b) {
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(t[0]);
    b = __uint_as_float(t[1]);
}
__device__ __forceinline__ void swap_lanes16(float& a, float& b) {
    const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(t[0]);
    b = __uint_as_float(t[1]);
}

// Lane i of a row of 16 gets lane i + N's value.
template <int N>
__device__ __forceinline__ float dpp_shl(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x100 + N, 0xf, 0xf, true));
}

// RPW row tiles of 16 rows (all Q planes of each) per wave, NT column tiles, keys of UC chunks (of
// 64 bytes per row) requested together.  Groups of waves along the row (RPW = 1) meet in LDS at the end
// of a row step.
template <int Q, int RPW, int NT, int UC>
__global__ __launch_bounds__(kDirectThreads, 1) void direct_kernel(const DirectParams p) {
    constexpr int RT = Q * RPW;
    extern __shared__ __align__(16) uint8_t direct_lds[];

    // (no divisions by run-time values on the way in: a small call is a chain of latencies)
    const int v0 = (int)blockIdx.y * p.vecs;
    const int nv = min(p.vecs, p.batch - v0);                 // vectors of this workgroup
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, kg = lane >> 4;
    const int ksplit = 1 << p.log_ksplit;
    const int kgroup = wave & (ksplit - 1), rgroup = wave >> p.log_ksplit;
    const int rgroups = kDirectWaves >> p.log_ksplit;
    const int blocks = p.chunks * 16;
    uint8_t* const digits = direct_lds;
    const int vec_bytes = blocks * (kDigits * 24) + 8;
    uint8_t* const scales = digits + vec_bytes * p.vecs;
    float* const red = reinterpret_cast<float*>(scales + blocks * p.vecs);

    // this wave's units (UC chunks each) of a row
    const int units = (p.chunks + UC - 1) / UC;
    const int u0 = kgroup * p.units_per_group, u1 = min(units, u0 + p.units_per_group);
    // first row of tile rp at row step rs
    const int step_rows = rgroups * RPW * 16;
    const int base0 = (int)blockIdx.x * p.steps * step_rows;
    auto tile_row = [&](int rs, int rp) { return base0 + rs * step_rows + (rgroup * RPW + rp) * 16; };
    const size_t plane_bytes = (size_t)p.m * p.stride_bytes;
    // unconditional loads from clamped addresses: rows past the end read the last row and are not
    // stored, keys past the row meet zero digits
    auto load_keys = [&](int rs, int u, mfma_u32x4 (&k)[RT][UC]) {
#pragma unroll
        for (int rp = 0; rp < RPW; ++rp) {
            const int row0 = min(tile_row(rs, rp), p.m - 1);
            const uint8_t* base = p.K + (size_t)row0 * p.stride_bytes;
            const uint32_t row_off = (uint32_t)min(r, p.m - 1 - row0) * p.stride_bytes;
#pragma unroll
            for (int i = 0; i < Q; ++i)
#pragma unroll
                for (int c = 0; c < UC; ++c) {
                    const uint32_t want = (uint32_t)((u * UC + c) * 64 + kg * 16);
                    const uint32_t lane_off = row_off + (want < p.stride_bytes ? want : 0u);
                    k[i * RPW + rp][c] = __builtin_nontemporal_load(
                        reinterpret_cast<const mfma_u32x4*>(base + i * plane_bytes + lane_off));
                }
        }
    };
    // rows 4 * kg .. + 3 of tile rp, plane i; rows past the end read as 0
    auto load_alpha = [&](int rs, float (&al)[RT][4]) {
#pragma unroll
        for (int rp = 0; rp < RPW; ++rp) {
            const int row0 = min(tile_row(rs, rp), p.m);
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<float*>(p.alpha + ((size_t)i * p.m + row0)), 0, min(p.m - row0, 16) * 4, 0x00020000);
                const mfma_u32x4 v =
                    __builtin_bit_cast(mfma_u32x4, __builtin_amdgcn_raw_buffer_load_b128(src, 16 * kg, 0, 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) al[i * RPW + rp][e] = __uint_as_float(v[e]);
            }
        }
    };

    mfma_u32x4 k[RT][UC], kn[RT][UC];
    float al[RT][4];
    // What the loop needs is computed while the inputs are on their way, not between the barrier and the first step.  With this,
    // the keys behind the inputs, and the partial sums of a row read at once: 4 % less over 282 shapes of 1 to 6 vectors (4.5 to
    // 17 us; eight groups of waves 5 %, one 2 %), 4096 x 4096, 2 planes, one vector, keys on chip 4.97 -> 4.75 us.
    // This lane's column of column tile nt: digit r % 5 of vector 3 nt + r / 5 (columns without a vector
    // repeat vector 0; their sums are not used)
    uint32_t col_off[NT], sc_off[NT];
    float digit_scale;
    uint32_t one8;
    int steps;                                                // row steps that have a row (the last row block may have fewer)
    auto prepare = [&] {
        digit_scale = __uint_as_float((uint32_t)(127 + kDirectWeightShift - 5 * (r % 5)) << 23);
        one8 = 0x22222222u;
        asm volatile("" : "+v"(digit_scale), "+v"(one8));
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int v = r < 15 && 3 * nt + r / 5 < nv ? 3 * nt + r / 5 : 0;
            col_off[nt] = (uint32_t)(v * vec_bytes + 4 * kg * (kDigits * 24) + (r % 5) * 24);
            sc_off[nt] = (uint32_t)(v * blocks + 4 * kg);
            asm volatile("" : "+v"(col_off[nt]), "+v"(sc_off[nt]));
        }
        steps = p.steps;
        while (steps > 1 && base0 + (steps - 1) * step_rows >= p.m) --steps;
        asm volatile("" : "+s"(steps));
    };
    // ---- inputs -> digits.  A wave takes 64 blocks at a time, four groups of 16 consecutive blocks of one
    // vector (a chunk); lane 16 g + w ends with block w of group g.  The four lanes w of a load take 64
    // contiguous bytes of one block and a 4 x 4 transpose over lane bits 4, 5 sorts them.  Buffer loads:
    // elements past the end of the vector read as 0.  The first keys and scales are requested behind the
    // inputs, so that the split waits for the inputs alone (again in every further round: a request behind
    // a condition would have to be waited for).
    const int ngroups = p.chunks * nv;
    auto vector_of = [&](int grp) { return p.chunks == 1 ? grp : (int)__umulhi((uint32_t)grp, p.chunks_inv); };
    int first = 4 * wave;
    if (first >= ngroups) {                                   // nothing to split
        prepare();                                            // (ahead of the keys: the other waves' inputs go first)
        load_keys(0, u0 < u1 ? u0 : 0, k);
        load_alpha(0, al);
    } else do {
        float t[4][8];                                        // [group][half and element of the piece]
        auto load_group = [&](int a, int v, int ch) {
            __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<float*>(p.X + (size_t)(v0 + v) * p.n), 0, p.n * 4, 0x00020000);
            const int off = 2048 * ch + 128 * r + 16 * kg;    // this lane's pieces: 16 bytes here and 64 further on
            const mfma_u32x4 lo = __builtin_bit_cast(mfma_u32x4, __builtin_amdgcn_raw_buffer_load_b128(src, off, 0, 0));
            const mfma_u32x4 hi = __builtin_bit_cast(mfma_u32x4, __builtin_amdgcn_raw_buffer_load_b128(src, off + 64, 0, 0));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                t[a][i] = __uint_as_float(lo[i]);
                t[a][4 + i] = __uint_as_float(hi[i]);
            }
        };
        if (nv == 1) {                                        // (one vector: its groups are its chunks)
#pragma unroll
            for (int a = 0; a < 4; ++a) load_group(a, 0, min(first + a, ngroups - 1));
        } else {
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const int grp = min(first + a, ngroups - 1);  // wave-uniform
                const int v = vector_of(grp);
                load_group(a, v, grp - v * p.chunks);
            }
        }
        load_keys(0, u0 < u1 ? u0 : 0, k);
        load_alpha(0, al);
        prepare();
        __builtin_amdgcn_sched_barrier(0);
        {
            float x[32];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                swap_lanes32(t[0][i], t[2][i]);
                swap_lanes32(t[1][i], t[3][i]);
                swap_lanes16(t[0][i], t[1][i]);
                swap_lanes16(t[2][i], t[3][i]);
            }
            // register a now holds piece a (and 4 + a) of this lane's block
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int i = 0; i < 8; ++i) x[16 * (i >> 2) + 4 * a + (i & 3)] = t[a][i];
            const int grp = min(first + kg, ngroups - 1);     // past the end: the last group again
            const int v = vector_of(grp), b = 16 * (grp - v * p.chunks) + r;
            uint8_t* dst = digits + v * vec_bytes + b * (kDigits * 24);
            const uint32_t sc = digit_split<kDigits>(x, [&](int d, const mfma_u32x6& pk) {
                mfma_u32x2* o = reinterpret_cast<mfma_u32x2*>(dst + d * 24);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    mfma_u32x2 w;
                    w.x = pk[2 * i]; w.y = pk[2 * i + 1];
                    o[i] = w;
                }
            });
            scales[v * blocks + b] = (uint8_t)sc;
        }
        first += 4 * kDirectWaves;
    } while (first < ngroups);
    __syncthreads();

    for (int rs = 0; rs < steps; ++rs) {
        f32x4v acc[RT][NT];
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[t][nt] = f32x4v{0.0f, 0.0f, 0.0f, 0.0f};
        if (rs > 0) load_alpha(rs, al);
        for (int u = u0; u < u1; ++u) {
            // the next unit, of this row step or the next one (none: nothing is requested, since the copy
            // below would wait for it)
            const bool last = u + 1 >= u1;
            const bool more = !last || rs + 1 < steps;
            if (more) load_keys(last ? rs + 1 : rs, last ? u0 : u + 1, kn);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int c = 0; c < UC; ++c) {
                // (UC = 2 and an odd number of chunks: the second one is past the row; nothing to add)
                if (UC > 1 && c > 0 && u * UC + c >= p.chunks) break;
                const uint32_t blk0 = (uint32_t)(u * UC + c) * 16;
                uint32_t sc[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    sc[nt] = *reinterpret_cast<const uint32_t*>(scales + sc_off[nt] + blk0);
                const uint8_t* dig = digits + blk0 * (kDigits * 24);
                auto load_b = [&](int st, int nt, mfma_u32x6& b) {
                    const mfma_u32x2* src = reinterpret_cast<const mfma_u32x2*>(dig + st * (kDigits * 24) + col_off[nt]);
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const mfma_u32x2 t = src[i];
                        b[2 * i] = t.x;
                        b[2 * i + 1] = t.y;
                    }
                };
                // the next step's operands are read while this one's instructions issue (a step is as
                // short as the latency of LDS: 16384 x 4096, 2 planes 6.3 -> 6.1 us; steps in a loop that is
                // not unrolled: 7.4)
                constexpr bool WHOLE = RT * NT <= 12;         // (what the registers hold)
                // ... otherwise column tile by column tile, two ahead (a whole step at once, spilled keys: 10-15 vectors,
                // 4 planes)
                mfma_u32x6 b[WHOLE ? 2 : 1][WHOLE ? NT : 3];
                if constexpr (WHOLE) {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) load_b(0, nt, b[0][nt]);
                } else {
                    load_b(0, 0, b[0][0]);
                    load_b(0, 1, b[0][1]);
                }
                auto step = [&](auto sc_t) {
                    constexpr int S = decltype(sc_t)::value;
                    if constexpr (WHOLE && S < 3) {
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) load_b(S + 1, nt, b[(S + 1) & 1][nt]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    mfma_u32x4 a[RT];
#pragma unroll
                    for (int t = 0; t < RT; ++t) a[t] = unpack_nibbles(k[t][c][S], one8);
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        const int next = S * NT + nt + 2;
                        if constexpr (!WHOLE) {
                            if (next < 4 * NT) load_b(next / NT, next % NT, b[0][next % 3]);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        const mfma_u32x6& bn = WHOLE ? b[S & 1][nt] : b[0][(next + 1) % 3];
#pragma unroll
                        for (int t = 0; t < RT; ++t) acc[t][nt] = direct_mfma<S>(a[t], bn, acc[t][nt], sc[nt]);
                    }
                };
                step(std::integral_constant<int, 0>{});
                step(std::integral_constant<int, 1>{});
                step(std::integral_constant<int, 2>{});
                step(std::integral_constant<int, 3>{});
                if constexpr (!WHOLE) {
                    // (the sums belong here: the compiler would move them behind the condition below, and with them the
                    // wait for this unit's operands behind the one for the next keys)
#pragma unroll
                    for (int t = 0; t < RT; ++t)
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) asm volatile("" : "+v"(acc[t][nt]));
                }
            }
            if (more)
#pragma unroll
                for (int t = 0; t < RT; ++t)
#pragma unroll
                    for (int c = 0; c < UC; ++c) k[t][c] = kn[t][c];
        }
        // ---- scale, planes, digits: lanes r = 0, 5, 10 end with vectors 3 nt + r / 5
        float y[RPW][NT][4];
#pragma unroll
        for (int rp = 0; rp < RPW; ++rp)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float s = 0.0f;
#pragma unroll
                    for (int i = 0; i < Q; ++i) s = fmaf(-al[i * RPW + rp][e], acc[i * RPW + rp][nt][e], s);
                    y[rp][nt][e] = s * digit_scale;
                }
        // (digit by digit over all sums: an exchange has to wait for an operand just written)
        float part[RPW][NT][4];
        auto gather_digit = [&](auto tap) {
            constexpr int N = decltype(tap)::value;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int rp = 0; rp < RPW; ++rp)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float d = N > 0 ? dpp_shl<N>(y[rp][nt][e]) : y[rp][nt][e];
                        part[rp][nt][e] = N == kDigits - 1 ? d : part[rp][nt][e] + d;
                    }
        };
        gather_digit(std::integral_constant<int, 4>{});
        gather_digit(std::integral_constant<int, 3>{});
        gather_digit(std::integral_constant<int, 2>{});
        gather_digit(std::integral_constant<int, 1>{});
        gather_digit(std::integral_constant<int, 0>{});
        // (where the accumulators leave few registers: lane numbers the compiler cannot compute addresses from
        // ahead of the loop, which it would spill)
        int er = r, ekg = kg;
        if constexpr (RT * NT >= 16 || (RPW == 4 && NT > 1)) asm volatile("" : "+v"(er), "+v"(ekg));
        const bool holder = er == 0 || er == 5 || er == 10;
        if (ksplit == 1) {
#pragma unroll
            for (int rp = 0; rp < RPW; ++rp) {
                const int row = tile_row(rs, rp) + 4 * ekg;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const int v = 3 * nt + er / 5;
                    if (holder && v < nv && row < p.m) {
                        float* dst = p.out + (size_t)(v0 + v) * p.m + row;
                        if (row + 3 < p.m) {
                            f32x4_a4 t;
                            t.x = part[rp][nt][0]; t.y = part[rp][nt][1]; t.z = part[rp][nt][2]; t.w = part[rp][nt][3];
                            *reinterpret_cast<f32x4_a4*>(dst) = t;
                        } else {
#pragma unroll
                            for (int e = 0; e < 3; ++e)
                                if (row + e < p.m) dst[e] = part[rp][nt][e];
                        }
                    }
                }
            }
        } else if constexpr (RPW == 1) {
            // red[buffer][wave][vector][16 rows]; two buffers, so one barrier per step: a wave writes a
            // buffer again only after the barrier of the step between, which follows its readers
            float* const buf = red + (rs & 1) * (kDirectWaves * NT * 3 * 16);
            if (holder) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    float* dst = buf + ((wave * NT + nt) * 3 + er / 5) * 16 + 4 * ekg;
#pragma unroll
                    for (int e = 0; e < 4; ++e) dst[e] = part[0][nt][e];
                }
            }
            __syncthreads();
            const int log_rows = 7 - p.log_ksplit;                // rows of a step: 128 / ksplit
            for (int o = tid; o < nv << log_rows; o += kDirectThreads) {
                const int v = o >> log_rows, rr = o & ((1 << log_rows) - 1);
                const int row = base0 + rs * step_rows + rr;
                // (all parts requested before the first is added: eight reads of LDS behind each other are 0.4 us)
                const float* src = buf + ((rr >> 4 << p.log_ksplit) * NT * 3 + v) * 16 + (rr & 15);
                auto add = [&](auto parts) {
                    constexpr int N = decltype(parts)::value;
                    float t[N];
#pragma unroll
                    for (int j = 0; j < N; ++j) t[j] = src[j * (NT * 3 * 16)];
                    float s = t[0];
#pragma unroll
                    for (int j = 1; j < N; ++j) s += t[j];
                    return s;
                };
                const float s = ksplit == 8 ? add(std::integral_constant<int, 8>{})
                              : ksplit == 4 ? add(std::integral_constant<int, 4>{}) : add(std::integral_constant<int, 2>{});
                if (row < p.m) p.out[(size_t)(v0 + v) * p.m + row] = s;
            }
        }
    }
}

}  // namespace biq
