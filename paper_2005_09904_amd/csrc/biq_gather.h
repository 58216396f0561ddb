// mu = 8, tables given in device memory (biq_query), few lookups: no copy of the tables in LDS.
//
// Copying a tile of tables costs a workgroup 128 KiB of scattered reads whatever its rows - 17 us for
// 1024 x 1024, 2 planes, 8 vectors, of whose entries each is then used a few times.  Here every lookup
// reads its entry where it lies; the tables stay in L2.  Bound by the address unit: one cache line per
// lane and lookup, up to four input vectors of an entry in one read.  Same lookups in the same order of the sums as
// the kernel that copies (and as the fused one): the same bits.  Time, copy -> here: 1024 x 1024, 2 planes, 8
// vectors 17.8 -> 4.2 us, 4096 x 1000, 4, 5: 34 -> 18, one vector: 2000 x 1800, 2 planes 16.8 -> 5.3.  (Reads behind
// conditions on the last chunk and the last vectors were waited for one by one: 7.3 us for the first.)
#pragma once

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

constexpr int kGatherVec = 4;      // input vectors per wave

// One wave per workgroup: HALF (the order of gemm8x2h): 8 rows x 8 lanes of 16 chunks, tiles of 128 chunks;
// otherwise (gemm8x2, latency mode) 16 rows x 4 lanes, tiles of 64.  Tiles of a row go to workgroups of their own
// (p.splits), their sums are added by reduce_splits_kernel as for the copying kernels.
template <int Q, bool HALF>
__global__ __launch_bounds__(64) void gather8_kernel(const QueryParams p) {
    constexpr int LANES = HALF ? 8 : 4, ROWS = 64 / LANES;
    const int row0 = (int)blockIdx.x * ROWS, sp = (int)blockIdx.y;
    // from 4 vectors on every slice is whole: the last one starts earlier and computes some vectors again
    // (fewer vectors: the read goes on into the next entry, what it brings is not stored)
    const int b0 = max(0, min((int)blockIdx.z * kGatherVec, p.batch - kGatherVec));
    const __amdgpu_buffer_rsrc_t tables = gather_tables_of(p);
    const int lane = threadIdx.x;
    const int L = lane & (LANES - 1), rsub = lane / LANES;
    const int rho = rsub & 3;                        // the copying kernel's rotation of the bytes of a dword
    const int swap = !HALF && (rsub & 4) ? 1 : 0;    // ... and, with 4 lanes per row, of its dwords
    const int row = min(row0 + rsub, p.m - 1);       // rows past the end: not stored
    const uint32_t stride_bytes = (uint32_t)p.stride_dw * 4u;
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
    float y[kGatherVec] = {};
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
#pragma unroll
    for (int c = 0; c < kGatherVec; ++c) {
        // the butterflies of reduce8 / reduce4
        y[c] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(y[c]), 0xB1, 0xf, 0xf, true));
        y[c] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(y[c]), 0x4E, 0xf, 0xf, true));
        if (HALF) y[c] += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(y[c]), 0x141, 0xf, 0xf, true));
        if (L == 0 && row0 + rsub < p.m && b0 + c < p.batch)
            p.out[((size_t)sp * p.batch + b0 + c) * p.m + row0 + rsub] = y[c];
    }
}

}  // namespace biq
