// Tables given in device memory (biq_query), few lookups: no copy of the tables in LDS.
//
// Copying a tile of tables costs a workgroup 128 KiB of scattered reads whatever its rows - 17 us for
// 1024 x 1024, 2 planes, 8 vectors, of whose entries each is then used a few times.  Here every lookup
// reads its entry where it lies; the tables stay in L2.  Bound by the address unit: one cache line per
// lane and lookup, up to four input vectors of an entry in one read.  Same lookups in the same order of the sums as
// the kernel that copies (and as the fused one): the same bits.  Time, copy -> here: 1024 x 1024, 2 planes, 8
// vectors 17.8 -> 3.4 us, 4096 x 1000, 4, 5: 34 -> 11, one vector: 2000 x 1800, 2 planes 16.8 -> 5.1.  (Reads behind
// conditions on the last chunk and the last vectors were waited for one by one: 7.3 us for the first.)
#pragma once

#include <type_traits>
#include <utility>

#include "biq_gather_rule.h"
#include "biq_kernels.h"

namespace biq {

typedef uint32_t gather_u32x4 __attribute__((ext_vector_type(4)));
// The tables as a buffer: reads past their end, that is of chunks past the last one, return 0, and no
// condition keeps the reads of a lane from being in flight together.  (The host admits only calls in which the
// offsets of a whole last tile stay below 2^32.)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t gather_tables_of(const QueryParams& p) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.LUT), 0, p.C * 1024 * p.batch, 0x00020000);
}

// One input vector: entry `key` of chunk `chunk` (the kernels of biq_gemv8.h and biq_gemv8h.h with p.table_fill).
__device__ __forceinline__ float gather_entry(const QueryParams& p, uint32_t chunk, uint32_t key) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(gather_tables_of(p), (int)(chunk * 1024u + key * 4u), 0, 0));
}

// f(integral_constant 0), ..., f(integral_constant N - 1)
template <typename F, int... I>
__device__ __forceinline__ void for_each_index(std::integer_sequence<int, I...>, F&& f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void for_each_index(F&& f) {
    for_each_index(std::make_integer_sequence<int, N>{}, f);
}

// The value of lane `lane ^ OFF`: inside a row of 16 lanes without a pass through LDS.
template <int CTRL>
__device__ __forceinline__ float lane_dpp(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int OFF>
__device__ __forceinline__ float lane_xor(float v) {
    if constexpr (OFF == 1) return lane_dpp<0xB1>(v);                     // quad_perm [1,0,3,2]
    else if constexpr (OFF == 2) return lane_dpp<0x4E>(v);                // quad_perm [2,3,0,1]
    else if constexpr (OFF == 4) return lane_dpp<0x1B>(lane_dpp<0x141>(v));   // row_half_mirror, quad_perm [3,2,1,0]
    else if constexpr (OFF == 8) return lane_dpp<0x128>(v);               // row_ror:8
    else return __shfl_xor(v, OFF, kWave);
}

// This lane's first vector.  From 4 vectors on every slice is whole: the last one starts earlier and computes some
// vectors again (fewer vectors: the read goes on into the next entry, what it brings is not stored).
__device__ __forceinline__ int gather_first_vector(const QueryParams& p, int slice) {
    return max(0, min(slice * kGatherVec, p.batch - kGatherVec));
}

// MULTI: the splits of a row go to the waves of a workgroup (wave w: splits w, w + waves, ...), which leave their sums in
// LDS, [split][slot of the row and slice][VEC], to be added in the order of reduce_splits_kernel: a dispatch less
// than the copying kernels need.
template <bool MULTI, int VEC>
__device__ __forceinline__ void gather_finish(const QueryParams& p, float* red, int slots, int slot, bool holder, int row,
                                              int b0, float (&y)[VEC], float* out) {
    if (MULTI) {
        __syncthreads();
        if (threadIdx.x >= 64) return;
#pragma unroll
        for (int c = 0; c < VEC; ++c) y[c] = red[slot * VEC + c];
        for (int s = 1; s < p.splits; ++s)
#pragma unroll
            for (int c = 0; c < VEC; ++c) y[c] += red[(s * slots + slot) * VEC + c];
    }
    if (!holder || row >= p.m) return;
#pragma unroll
    for (int c = 0; c < VEC; ++c)
        if (b0 + c < p.batch) out[(size_t)(b0 + c) * p.m + row] = y[c];
}

// HALF (the order of gemm8x2h): 8 lanes of 16 chunks per row, tiles of 128 chunks; otherwise (gemm8x2, latency
// mode) 4 lanes, tiles of 64.
// MULTI: rows of several splits in the waves of a workgroup; otherwise the grid's z is the split, and p.out takes the
// splits' sums one after the other.
template <int Q, bool HALF, int LOG_SLICES, bool MULTI>
__global__ __launch_bounds__(MULTI ? 64 * kGatherWaves : 64) void gather8_kernel(const QueryParams p) {
    constexpr int LANES = HALF ? 8 : 4, SL = 1 << LOG_SLICES, ROWS = 64 / (LANES * SL);
    extern __shared__ __align__(16) float gather_lds[];
    const int row0 = (int)blockIdx.x * ROWS;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b0 = gather_first_vector(p, (int)blockIdx.y * SL + (lane & (SL - 1)));
    const __amdgpu_buffer_rsrc_t tables = gather_tables_of(p);
    const int L = (lane >> LOG_SLICES) & (LANES - 1), rsub = lane / (LANES * SL);
    const int crow = (row0 + rsub) & (64 / LANES - 1);   // the row's place in a step of the copying kernel
    const int rho = crow & 3;                        // ... whose rotation of the bytes of a dword it takes
    const int swap = !HALF && (crow & 4) ? 1 : 0;    // ... and, with 4 lanes per row, of its dwords
    const int row = min(row0 + rsub, p.m - 1);       // rows past the end: not stored
    const int slot = rsub * SL + (lane & (SL - 1));
    const uint32_t stride_bytes = (uint32_t)p.stride_dw * 4u;
    float y[kGatherVec];
    // (bounds from which the compiler sees a single turn: otherwise it keeps the addresses of all reads in registers, 94-132
    // instead of 69-110, and 183 x 90112, 1 plane, 3 vectors took 52.3 us instead of 49.3)
    for (int at = MULTI ? wave : 0; at < (MULTI ? p.splits : 1); at += MULTI ? (int)blockDim.x >> 6 : 1) {
    const int sp = MULTI ? at : (int)blockIdx.z;
    const uint32_t want = (uint32_t)(sp * LANES * 16 + 16 * L);
    const uint32_t seg = want < stride_bytes ? want : 0u;      // past the row: keys of chunks that count as 0
    gather_u32x4 k[Q];
    float al[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const size_t kr = (size_t)i * p.m + row;
        k[i] = *reinterpret_cast<const gather_u32x4*>(reinterpret_cast<const char*>(p.K) + kr * stride_bytes + seg);
        al[i] = p.alpha[kr];
    }
#pragma unroll
    for (int c = 0; c < kGatherVec; ++c) y[c] = 0.0f;
    // (planes in a loop, the next one's keys moved to the front: a call runs its code once, from a cold
    // instruction cache, and the 16 reads in flight of one plane keep the address unit busy)
#pragma unroll 1
    for (int plane = 0; plane < Q; ++plane) {
        constexpr int i = 0;
        float v[16][kGatherVec];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int td = (j >> 2) ^ swap, e = (j + rho) & 3;
            const uint32_t w = HALF ? k[i][j >> 2] : swap ? k[i][(j >> 2) ^ 1] : k[i][j >> 2];
            const uint32_t chunk = (uint32_t)(sp * LANES * 16 + 16 * L + 4 * td + e);
            const uint32_t key = (w >> (8 * e)) & 255u;
            const gather_u32x4 t = __builtin_bit_cast(gather_u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                tables, (int)(((chunk * 256u + key) * (uint32_t)p.batch + (uint32_t)b0) * 4u), 0, 0));
#pragma unroll
            for (int c = 0; c < kGatherVec; ++c) v[j][c] = __uint_as_float(t[c]);
        }
        __builtin_amdgcn_sched_barrier(0);           // all 16 reads before the first use
#pragma unroll
        for (int c = 0; c < kGatherVec; ++c) {
            // (the copying kernels start from 0 and from the first two values)
            float a0 = HALF ? 0.0f + v[0][c] : v[0][c], a1 = HALF ? 0.0f + v[1][c] : v[1][c];
#pragma unroll
            for (int j = 2; j < 16; ++j) {
                if (j & 1) a1 += v[j][c];
                else a0 += v[j][c];
            }
            y[c] = fmaf(al[i], a0 + a1, y[c]);
        }
#pragma unroll
        for (int n = 0; n + 1 < Q; ++n) { k[n] = k[n + 1]; al[n] = al[n + 1]; }
    }
    // the order of reduce8 / reduce4
#pragma unroll
    for (int c = 0; c < kGatherVec; ++c) y[c] += lane_xor<SL>(y[c]);
#pragma unroll
    for (int c = 0; c < kGatherVec; ++c) y[c] += lane_xor<2 * SL>(y[c]);
    if constexpr (HALF)
#pragma unroll
        for (int c = 0; c < kGatherVec; ++c) y[c] += lane_xor<4 * SL>(y[c]);
    if (MULTI && L == 0)
#pragma unroll
        for (int c = 0; c < kGatherVec; ++c) gather_lds[(sp * ROWS * SL + slot) * kGatherVec + c] = y[c];
    }
    gather_finish<MULTI>(p, gather_lds, ROWS * SL, slot, L == 0, row0 + rsub, b0, y,
                         MULTI ? p.out : p.out + (size_t)blockIdx.z * p.batch * p.m);
}

// Any mu, for the plans of query_kernel and (ascending) query_wide_kernel: G lanes of one key unit each per row,
// the workgroup's tiles one after the other, the same order of the sums.  Those kernels'
// copies cost 12-25 us: 163 x 223, 4 planes, 14 vectors, mu = 4 12.5 -> 5.2 us, 2404 x 737, 4, 11, mu = 5 30 -> 10.6.
// VEC = 1 for one input vector.
template <int MU, int VEC>
__global__ __launch_bounds__(64 * kGatherWaves) void gather_units_kernel(const QueryParams p, int log_slices, int log_splits,
                                                                         int ascending) {
    constexpr int E = 1 << MU, UD = KeyUnit<MU>::UD, UK = KeyUnit<MU>::UK;
    constexpr int NB = UK < 16 ? UK : 16;            // reads in flight
    extern __shared__ __align__(16) float gather_lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int slice = VEC == 1 ? 0 : ((int)blockIdx.y << log_slices) + (lane & ((1 << log_slices) - 1));
    const int b0 = VEC == 1 ? 0 : gather_first_vector(p, slice);
    const int L = (lane >> log_slices) & (p.G - 1);
    // 2^log_splits splits of a row side by side in a wave (gather_units_shape)
    const int lane_split = (lane >> (log_slices + p.log2G)) & ((1 << log_splits) - 1);
    const int log_lanes = p.log2G + log_slices + log_splits;      // lanes of a row: at most 64
    const int row_want = (int)(blockIdx.x << (6 - log_lanes)) + (lane >> log_lanes);
    const int row = min(row_want, p.m - 1);          // rows past the end: not stored
    const __amdgpu_buffer_rsrc_t tables =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.LUT), 0, p.C * (E * 4) * p.batch, 0x00020000);
    const int slots = 64 >> (p.log2G + log_splits), slot = ((lane >> log_lanes) << log_slices) + (lane & ((1 << log_slices) - 1));
    // dwords past the row hold no key of a chunk that exists, or the zero bits behind its last element
    auto load_keys = [&](int tile, int plane, uint32_t (&w)[UD], float& al) {
        const size_t kr = (size_t)plane * p.m + row;
        const uint32_t* src = p.K + kr * p.stride_dw;
        const int dw0 = (tile * p.CT / UK + L) * UD;
        if constexpr (UD == 4) {
            const gather_u32x4 v = *reinterpret_cast<const gather_u32x4*>(src + (dw0 < p.stride_dw ? dw0 : 0));
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = v[i];
        } else {
#pragma unroll
            for (int i = 0; i < UD; ++i) w[i] = src[min(dw0 + i, p.stride_dw - 1)];
        }
        al = p.alpha[kr];
    };
    float total[VEC];
    for (int sp0 = wave << log_splits; sp0 < p.splits; sp0 += ((int)blockDim.x >> 6) << log_splits) {
    const int sp = min(sp0 + lane_split, p.splits - 1);          // past the end: the last one again
    const int tile0 = sp * p.tps, tile1 = min(p.tiles, tile0 + p.tps);
    uint32_t w[UD], wn[UD];
    float al, aln;
    load_keys(tile0, 0, w, al);
#pragma unroll
    for (int c = 0; c < VEC; ++c) total[c] = 0.0f;
    for (int tile = tile0; tile < tile1; ++tile) {
        const uint32_t chunk0 = (uint32_t)(tile * p.CT + L * UK);
        const int dw0 = (tile * p.CT / UK + L) * UD;
        float y[VEC] = {};
#pragma unroll 1
        for (int plane = 0; plane < p.q; ++plane) {
            const bool last = plane + 1 == p.q;
            load_keys(last ? min(tile + 1, tile1 - 1) : tile, last ? 0 : plane + 1, wn, aln);
            if constexpr (UD != 4) {
#pragma unroll
                for (int i = 0; i < UD; ++i) w[i] = dw0 + i < p.stride_dw ? w[i] : 0u;
            }
            float acc[VEC] = {};
            auto batch_of = [&](auto first) {
                constexpr int T0 = decltype(first)::value;
                float v[NB][VEC];
                auto read = [&](auto tc) {
                    constexpr int T = T0 + decltype(tc)::value;
                    const uint32_t key = unit_key<MU, T>(w);
                    const uint32_t at = (((chunk0 + T) * (uint32_t)E + key) * (uint32_t)p.batch + (uint32_t)b0) * 4u;
                    if constexpr (VEC == 1) {
                        v[T - T0][0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(tables, (int)at, 0, 0));
                    } else {
                        const gather_u32x4 t =
                            __builtin_bit_cast(gather_u32x4, __builtin_amdgcn_raw_buffer_load_b128(tables, (int)at, 0, 0));
#pragma unroll
                        for (int c = 0; c < VEC; ++c) v[T - T0][c] = __uint_as_float(t[c]);
                    }
                };
                for_each_index<NB>(read);
                __builtin_amdgcn_sched_barrier(0);   // all reads before the first use
#pragma unroll
                for (int t = 0; t < NB; ++t)
#pragma unroll
                    for (int c = 0; c < VEC; ++c) acc[c] += v[t][c];
            };
            for_each_index<UK / NB>([&](auto b) { batch_of(std::integral_constant<int, decltype(b)::value * NB>{}); });
#pragma unroll
            for (int c = 0; c < VEC; ++c) y[c] = fmaf(al, acc[c], y[c]);
#pragma unroll
            for (int i = 0; i < UD; ++i) w[i] = wn[i];
            al = aln;
        }
        if (ascending) {
            for (int off = 1; off < p.G; off *= 2)
#pragma unroll
                for (int c = 0; c < VEC; ++c) y[c] += __shfl_xor(y[c], off << log_slices, kWave);
        } else {
            for (int off = p.G >> 1; off > 0; off >>= 1)
#pragma unroll
                for (int c = 0; c < VEC; ++c) y[c] += __shfl_xor(y[c], off << log_slices, kWave);
        }
#pragma unroll
        for (int c = 0; c < VEC; ++c) total[c] += y[c];
    }
    if (p.splits > 1 && L == 0)
#pragma unroll
        for (int c = 0; c < VEC; ++c) gather_lds[(sp * slots + slot) * VEC + c] = total[c];
    }
    if (p.splits > 1) gather_finish<true>(p, gather_lds, slots, slot, L == 0, row_want, b0, total, p.out);
    else gather_finish<false>(p, gather_lds, slots, slot, L == 0, row_want, b0, total, p.out);
}

}  // namespace biq
