// C ABI of libbiq (see include/biq.h): argument checks, launch planning, launches.
#include "biq.h"

#include <hip/hip_runtime.h>

#include "biq_launch.h"
// kernel headers: only their geometry constants are used here (no kernel is instantiated in this file)
#include "biq_gemv8.h"
#include "biq_gemm8x2.h"
#include "biq_gemv8h.h"
#include "biq_gemm8x2h.h"
#include "biq_query_wide.h"
#include "biq_quantize.h"
#include "biq_grouped.h"
#include "biq_digit_mfma.h"
#include "biq_direct.h"
#include "biq_direct_rule.h"
#include "biq_gather.h"

namespace {

using namespace biq;

// gfx950 (MI355X) limits the planner is written for.
constexpr int kLdsTableBudget = 128 * 1024;  // tables of one tile (leaves room for 1 WG/CU extras)
constexpr int kNumCu = 256;
static_assert(kDirectCus == kNumCu && kDirectLds == kLdsPerCu, "as biq_direct_rule.h counts them");
constexpr int kNumXcd = 8;

enum KernelId { KERNEL_GENERIC = 0, KERNEL_GEMV8 = 1, KERNEL_GEMM8X2 = 2, KERNEL_UNPACK_MFMA = 3, KERNEL_GEMV8H = 4, KERNEL_GEMM8X2H = 5, KERNEL_WIDE = 6, KERNEL_COUNT };

inline bool shape_ok(int m, int n, int q, int batch, int mu) {
    if (m < 1 || n < 1 || q < 1 || batch < 1) return false;
    if (mu < 1 || mu > kMaxMu) return false;
    if ((long long)m * q >= (1ll << 31)) return false;
    return true;
}

inline int unit_keys(int mu) {
    switch (mu) {
        case 10: return KeyUnit<10>::UK; case 9: return KeyUnit<9>::UK;
        case 8: return KeyUnit<8>::UK; case 7: return KeyUnit<7>::UK; case 6: return KeyUnit<6>::UK;
        case 5: return KeyUnit<5>::UK; case 4: return KeyUnit<4>::UK; case 3: return KeyUnit<3>::UK;
        case 2: return KeyUnit<2>::UK; default: return KeyUnit<1>::UK;
    }
}

inline int ceil_div(int a, int b) { return (int)(((unsigned)a + (unsigned)b - 1u) / (unsigned)b); }   // a >= 0, b >= 1
inline long long ceil_div_ll(long long a, long long b) { return (a + b - 1) / b; }
// a * b * c of counts up to 2^31 each, 2^61 where it is more (comparisons and quotients stay meaningful)
inline long long product(long long a, long long b, long long c) {
    const __int128 p = (__int128)a * b * c;
    return p < ((__int128)1 << 61) ? (long long)p : 1ll << 61;
}
// rows per workgroup from a 64-bit estimate: rounded up to a multiple of `step`, at least `lo`, and
// never beyond what the 32-bit plan field holds (more rows than m are pointless anyway)
inline int rows_from(long long want, int step, int lo, int m) {
    long long r = ceil_div_ll(want, step) * step;
    const long long cap = ceil_div_ll(m, step) * step;
    if (r > cap) r = cap;
    if (r < lo) r = lo;
    return (int)r;
}
// ... with `each` workgroups per block of rows (splits of a row, tiles of input vectors): no more workgroups than CUs where
// that is possible.  A few more of them are a second round, which builds tables again, on a few CUs (rows shared out as
// m * each / cus: 7 % of the table plans; 150 of those, table kernels 30 % less with this: 10240 x 11353, 4 planes, 1 vector
// 33.0 -> 21.6 us, 356 x 4141, 3, 24 13.9 -> 9.4, 384 x 519, 4, 51 9.4 -> 5.6).
inline int rows_one_round(int m, long long each, int cus, int step, int lo) {
    return rows_from(each <= cus ? ceil_div_ll(m, cus / each) : ceil_div_ll(product(m, each, 1), cus), step, lo, m);
}
inline int ilog2(int v) { int l = 0; while ((1 << (l + 1)) <= v) ++l; return l; }

// 16-byte pieces of prepared input per key group (16 MFMA steps): column tiles x terms x 64 lanes
inline long long unpack_group_pieces(int batch_tile, int terms) { return 16ll * (batch_tile / 32) * terms * 64; }

// Unpack-MFMA plans: workgroups of 4 waves, key groups (32 key bytes of a row) instead of LUT tiles.
bool plan_finish_unpack(biq_plan& pl, int m, int n, int q, int batch) {
    if (q > 4 || pl.threads != kUnpackThreads) return false;
    if (pl.batch_tile != 32 && pl.batch_tile != 64) return false;
    if (pl.chunks_per_tile != kUnpackGroupBytes) return false;
    if (pl.wave_splits == 0) pl.wave_splits = 1;
    if (pl.input_terms == 0) pl.input_terms = 3;     // exact split unless the caller asks for two terms
    if (pl.input_terms != 2 && pl.input_terms != 3) return false;
    const int ws = pl.wave_splits;
    if (ws != 1 && ws != 2 && ws != 4) return false;
    // (4 / ws) waves side by side x r row tiles of 32 rows per plane, at most 4 row tiles per wave
    // (with block-scaled digits, row_mode 1: 8 row x column tiles)
    const bool digits = pl.row_mode == 1;
    const int per_r = (4 / ws) * 32;
    if (pl.rows_per_wg < 1 || pl.rows_per_wg % per_r) return false;
    const int r = pl.rows_per_wg / per_r;
    if (r != 1 && r != 2 && r != 4) return false;
    if (digits ? q * r * (pl.batch_tile / 32) > kDigitMaxTiles : q * r > 4) return false;
    if (!digits && ws == 4 && q * r * (pl.batch_tile / 32) == 8) return false;  // would not fit the register file
    if ((pl.row_mode != 0 && !digits) || pl.xcd_skew != 0 || pl.tiles_per_split < 1) return false;
    const int groups = (int)((biq_key_row_stride(n) + kUnpackGroupBytes - 1) / kUnpackGroupBytes);
    if (pl.tiles_per_split > groups) pl.tiles_per_split = groups;
    if (digits) {
        if (pl.input_terms != 3) return false;
        // a wave looks at the forms of its key groups with one load; 32-bit lane offsets over 32 rows
        if (ceil_div(pl.tiles_per_split, ws) > 64 || biq_key_row_stride(n) > (1u << 26)) return false;
    }
    pl.chunk_splits = (groups + pl.tiles_per_split - 1) / pl.tiles_per_split;
    pl.row_blocks = ceil_div(m, pl.rows_per_wg);
    pl.batch_tiles = ceil_div(batch, pl.batch_tile);
    pl.lds_bytes = ws == 1 ? 24 * 1024 : 96 * 1024;   // partial sums of the wave groups, transpose patches (UnpackGeom::LDS_BYTES)
    if (digits) {                                     // DigitGeom::LDS_BYTES
        const int nout = r * (pl.batch_tile / 32);
        pl.lds_bytes = ((4 / ws) * nout * (ws - 1) * 1024 + 4 * 32 * 36 + 4 * 256) * 4;
    }
    const long long tasks = product(pl.row_blocks, pl.chunk_splits, pl.batch_tiles);
    if (tasks > (1ll << 30)) return false;
    // prepared input: 2 bytes per term and (padded column, padded element)
    const long long xf = product(pl.batch_tiles, (long long)pl.chunk_splits * pl.tiles_per_split,
                                 unpack_group_pieces(pl.batch_tile, pl.input_terms) * 16);
    if (xf > (1ll << 40)) return false;
    return true;
}

inline int plan_lds_bytes(const biq_plan& pl, int mu) {
    if (pl.kernel == KERNEL_GEMV8)
        return kGemvTileBytes +
               (pl.tiles_per_split > 1 ? ((pl.rows_per_wg + pl.xcd_skew + 63) / 64) * 64 * 4 : 0);
    if (pl.kernel == KERNEL_GEMV8H)
        return kGemvHalfTileBytes + (pl.tiles_per_split > 1 ? ((pl.rows_per_wg + 3) / 4) * 16 : 0);
    if (pl.kernel == KERNEL_GEMM8X2H) return kGemmHalfTileBytes;
    if (pl.kernel == KERNEL_WIDE) return 128 * 1024;
    if (pl.kernel == KERNEL_GEMM8X2)
        return kGemmTileBytes + (pl.tiles_per_split > 1 ? ((pl.rows_per_wg + 63) / 64) * 64 * 8 : 0);
    long long b = (long long)pl.chunks_per_tile * (1 << mu) * pl.batch_tile * 4;
    if (pl.tiles_per_split > 1) b += (long long)pl.rows_per_wg * pl.batch_tile * 4;
    return b > (1ll << 30) ? (1 << 30) : (int)b;
}

// Completes the derived fields and checks a plan against the shape and device limits.
bool plan_finish(biq_plan& pl, int m, int n, int q, int batch, int mu) {
    const int UK = unit_keys(mu);
    const int C = ceil_div(n, mu);
    if (pl.kernel < 0 || pl.kernel >= KERNEL_COUNT) return false;
    if (pl.kernel == KERNEL_UNPACK_MFMA) return plan_finish_unpack(pl, m, n, q, batch);
    if (pl.wave_splits != 0 || pl.input_terms != 0) return false;  // unpack_mfma only
    if (pl.table_fill == 2) {
        DirectGeom g;
        if (!direct_geometry(g, m, n, q, batch)) return false;
    } else if (pl.table_fill != 0 && !(pl.table_fill == 1 && pl.kernel == KERNEL_GEMV8 && pl.row_mode == 0)) {
        return false;
    }
    if (pl.threads < 64 || pl.threads > 1024 || pl.threads % 64) return false;
    if (pl.kernel == KERNEL_GEMV8) {
        // mu = 8, one input vector, at most 4 planes; one 128-chunk tile per workgroup
        if (mu != 8 || batch != 1 || q > 4) return false;
        if (pl.chunks_per_tile != kGemvTileChunks || pl.batch_tile != 1) return false;
        // 32-bit byte offsets inside a workgroup's row block
        if ((long long)pl.rows_per_wg * (long long)biq_key_row_stride(n) >= (1ll << 31)) return false;
    }
    if (pl.kernel == KERNEL_GEMV8H) {
        // mu = 8, one input vector, at most 4 planes; 256-chunk tiles of half tables, latency mode
        // only; row_mode 1 can walk several tiles (row sums carried in LDS beside the tables)
        if (mu != 8 || batch != 1 || q > 4) return false;
        if (pl.chunks_per_tile != kGemvHalfTileChunks || pl.batch_tile != 1) return false;
        if (pl.row_mode != 1 && pl.row_mode != 2) return false;
        if (pl.tiles_per_split != 1 && (pl.row_mode != 1 || pl.rows_per_wg > 4096)) return false;
    }
    if (pl.kernel == KERNEL_WIDE) {
        // mu <= 6; one tile of 32 key units per workgroup, batch tile fixed by mu (tables fill 128 KiB)
        if (mu > 6 || pl.chunks_per_tile != 32 * UK) return false;
        if (pl.batch_tile != (128 * 1024) / (32 * UK * (1 << mu) * 4)) return false;
        if (pl.row_mode != 0 || pl.tiles_per_split != 1) return false;
    }
    if (pl.kernel == KERNEL_GEMM8X2H) {
        // mu = 8, at most 4 planes; one 128-chunk tile of half tables for two input vectors per
        // workgroup, latency mode only
        if (mu != 8 || q > 4) return false;
        if (pl.chunks_per_tile != kGemmHalfTileChunks || pl.batch_tile != 2) return false;
        if (pl.row_mode != 1 || pl.tiles_per_split != 1) return false;
    }
    if (pl.kernel == KERNEL_GEMM8X2) {
        // mu = 8, at most 4 planes; 64-chunk tiles of two input vectors
        if (mu != 8 || q > 4) return false;
        if (pl.chunks_per_tile != kGemmTileChunks || pl.batch_tile != kGemmBT) return false;
        if ((long long)pl.rows_per_wg * (long long)biq_key_row_stride(n) >= (1ll << 31)) return false;
    }
    if (pl.batch_tile != 1 && pl.batch_tile != 2 && pl.batch_tile != 4 && pl.batch_tile != 8) return false;
    if (pl.chunks_per_tile < UK || pl.chunks_per_tile % UK) return false;
    const int G = pl.chunks_per_tile / UK;
    if (G > 64 || (G & (G - 1))) return false;
    if (pl.rows_per_wg < 1 || pl.tiles_per_split < 1) return false;
    const int tiles = ceil_div(C, pl.chunks_per_tile);
    if (pl.tiles_per_split > tiles) pl.tiles_per_split = tiles;
    if (pl.row_mode != 0 &&
        !(pl.row_mode == 1 && pl.kernel != KERNEL_GENERIC && (pl.tiles_per_split == 1 || pl.kernel == KERNEL_GEMV8H)) &&
        !(pl.row_mode == 2 && pl.kernel == KERNEL_GEMV8H))
        return false;
    if (pl.xcd_skew != 0) {
        // only the GEMV kernel's throughput mode, whole grid = 8 equal XCD shares, no chunk split
        if (pl.kernel != KERNEL_GEMV8 || pl.row_mode != 0 || pl.xcd_skew < 0) return false;
        if (pl.xcd_skew >= pl.rows_per_wg || ceil_div(m, pl.rows_per_wg) % kNumXcd != 0) return false;
        if (ceil_div(tiles, pl.tiles_per_split) != 1) return false;
        // (even XCDs hold rows_per_wg + xcd_skew rows in LDS: counted in lds_bytes below)
    }
    pl.chunk_splits = ceil_div(tiles, pl.tiles_per_split);
    pl.row_blocks = ceil_div(m, pl.rows_per_wg);
    pl.batch_tiles = ceil_div(batch, pl.batch_tile);
    pl.lds_bytes = plan_lds_bytes(pl, mu);
    if (pl.lds_bytes > kLdsPerCu) return false;
    const long long tasks = product(pl.row_blocks, pl.chunk_splits, pl.batch_tiles);
    if (tasks > (1ll << 30)) return false;
    return true;
}

// Estimated time (us) of the lookup-table plan `pl`, from rates measured on MI355X: where the tables
// stop paying off (the crossover of Sec. IV-B / Fig. 10).  The batched mu = 8 kernels, fitted to 330 shapes, 7 % rms (half
// tables 5 %): per round of workgroups over the CUs and tile the lookups of its rows and two input vectors, more where rows
// of the input are not read 16 bytes at a time, keys at 4.5 TB/s, a second kernel with 0.24 us per split, half of it
// for up to ten results.  (Estimated /
// measured: 17856 x 14656, 3 planes, 2 vectors 38.3 / 38.3; 7360 x 1884, 2, 53 26.4 / 25.6; 960 x 14438, 2, 11 16.6 / 16.0.)
// Narrow keys, fitted to 319 shapes, 9 % rms: 5.1 us per round and the lookups of
// a whole tile, 2.9 (mu = 5) and 4.1 times (mu = 6) the time where a pass serves one vector only; a second kernel
// 3.3 us and 9 us per million partial results.  One vector in half tables, fitted to 275 shapes, 7 % rms: 0.8 us and a row's
// planes at 11 ns per tile, 2.4 us more where rows of the input are not read 16 bytes at a time, keys at 6.7 TB/s, a second
// kernel 1 us, 0.27 us per split and 13 us per million partial results.  The generic kernel: 6.5e12 lookups/s, keys at no more than 0.25 TB/s,
// and 0.4 us per partial result a second kernel adds (320 x 12288, mu = 7, 4, 24: 38 / 33) - but one vector on rows of
// up to four key units, the fewer lanes of a row the better: 0.1 to 0.3 ps per lookup of a row's whole units, more
// where the workgroups are fewer than the CUs (310460 x 192, mu = 4, 1 plane 7.3 / 6.8 us; the general rule says 35.8).
double tables_estimate(const biq_plan& pl, int m, int n, int q, int batch, int mu) {
    const double wgs = (double)pl.row_blocks * pl.chunk_splits * pl.batch_tiles;
    const double rounds = (double)(long long)((wgs + kNumCu - 1) / kNumCu);
    const double rows = pl.rows_per_wg < m ? pl.rows_per_wg : m;
    const double mem = (double)q * m * biq_key_row_stride(n);
    if (pl.kernel == KERNEL_GEMM8X2 || pl.kernel == KERNEL_GEMM8X2H) {   // (a short row still takes its lanes' time)
        const bool half = pl.kernel == KERNEL_GEMM8X2H;
        const double lookups = rows * q * pl.chunks_per_tile * 2;
        const double tile = half ? 26.8e-6 * lookups + (n % 4 ? 1.0 : 0.0) : 0.51 + 18.6e-6 * lookups + (n % 4 ? 0.4 : 0.0);
        const double turns = rounds * pl.tiles_per_split;    // (the first one's tables are built beside the dispatch)
        return (half ? 3.65 : 2.8) + together(turns * tile + (turns - 1) * (half ? 1.3 : 1.5), mem / 4.5e6) +
               (pl.chunk_splits > 1 ? (half ? 1.5 : 3.1) + pl.chunk_splits * (((long long)m * batch <= 10 ? 0.11 : 0.24) +
                                                                              (half ? 1.7e-6 : 0.9e-6) * m * batch) : 0.0);
    }
    if (pl.kernel == KERNEL_WIDE) {
        const double slower = mu == 6 ? 4.1 : mu == 5 ? 2.9 : mu == 4 ? 1.14 : 1.0;
        return rounds * (5.1 + slower * rows * q * pl.chunks_per_tile * pl.batch_tile / 65e3) +
               (pl.chunk_splits > 1 ? 3.3 + 8.7e-6 * pl.chunk_splits * (double)m * batch : 0.0);
    }
    if (pl.kernel == KERNEL_GEMV8H) {
        const double rq = rows * q, tiles = pl.tiles_per_split;
        const double walk = rounds * (pl.row_mode == 2 ? 0.011 * rq + (n % 4 ? 2.7 : 0.0)
                                                       : tiles * (0.8 + 0.011 * rq + (n % 4 ? 2.4 : 0.0)) +
                                                             (tiles > 1 ? 0.42 * q : 0.0) + (tiles > 2 ? 0.5 * q : 0.0));
        return 3.3 + together(walk, mem / 6.7e6) +
               (pl.chunk_splits > 1 ? 1.06 + pl.chunk_splits * (0.27 + 13e-6 * m) : 0.0);
    }
    const int units = pl.chunks_per_tile / unit_keys(mu);
    if (batch == 1 && units <= 4 && pl.chunk_splits == 1 && mu <= 7) {
        const double ps = mu <= 4   ? (units == 1 ? 0.107 : units == 2 ? 0.152 : 0.25)
                          : mu == 5 ? 0.18
                          : mu == 6 ? (units <= 2 ? 0.23 : 0.27)
                                    : (units == 1 ? 0.20 : 0.30);
        return 4.2 + ps * 1e-6 * m * q * pl.chunks_per_tile * (wgs < kNumCu ? kNumCu / wgs : 1.0);
    }
    const double weights = (double)q * m * n;
    double t = weights / mu * batch / 6.5e6;
    if (t < weights / 8 / 0.25e6) t = weights / 8 / 0.25e6;
    return 6.0 + t + (pl.chunk_splits > 1 ? 2.0 + 0.4 * pl.chunk_splits : 0.0);
}

// The mapping of the unpack + MFMA kernel - column tile (32 or 64 input vectors), row tiles per
// wave and plane (r), wave groups along the contraction inside a workgroup (ws; partial sums
// added in LDS) and workgroups along the contraction (S; partial sums through the workspace and
// a second kernel) - is the candidate with the lowest estimated time.  The estimate: MFMAs per
// wave x 33 clk at 2.1 GHz (measured rate of back-to-back MFMAs under load) x an issue-overhead
// factor per accumulator shape (smallest for 4 x 2 tiles, more for fewer, where key expansion
// and fragment loads are shared by fewer MFMAs) x rounds of workgroups over the 256 CUs, plus
// fixed costs per launch, accumulator tile and round, the input split (per byte of padded X)
// and the second kernel.  The constants (one set per number of input terms) are least-squares
// fits to sweeps of 16 layer shapes x all valid mappings, on which the estimate's choice was the
// fastest or within 5 % of it.
struct UnpackCost {
    double shape8, shape6, shape4x1, shape3x1, shape2x2, shape2x1, shape1x2, shape1x1;
    double fix, per_tile, per_round, split_per_mb, second_kernel, second_per_mb, per_wave_group;
};
const UnpackCost kUnpackCost3 = {1.13, 1.16, 1.19, 1.22, 1.22, 1.30, 1.45, 1.65, 9.0, 0.25, 0.0, 0.0, 3.5, 0.4, 0.6};
const UnpackCost kUnpackCost2 = {1.20, 1.20, 1.36, 1.29, 1.42, 1.67, 2.10, 2.27, 5.3, 1.0, 1.1, 1.65, 2.45, 0.1, 0.0};

bool plan_unpack(biq_plan& pl, int m, int n, int q, int batch, int mu, int terms) {
    if (q > 4 || (terms != 2 && terms != 3)) return false;
    const UnpackCost& c = terms == 3 ? kUnpackCost3 : kUnpackCost2;
    pl = biq_plan{};
    pl.kernel = KERNEL_UNPACK_MFMA;
    pl.threads = kUnpackThreads;
    pl.chunks_per_tile = kUnpackGroupBytes;
    pl.input_terms = terms;
    const int groups = (int)((biq_key_row_stride(n) + kUnpackGroupBytes - 1) / kUnpackGroupBytes);
    double best = 1e30;
    for (int bt = 32; bt <= 64; bt += 32)
        for (int ws = 1; ws <= 4; ws *= 2)
            for (int r = 1; r <= 4; r *= 2)
                for (int S = 1; S <= 16; S *= 2) {
                    const int ct = bt / 32, rt = q * r;
                    if (rt > 4 || S * ws > groups) continue;
                    if (ws == 4 && rt * ct == 8) continue;   // would not fit the register file
                    const int rows = (4 / ws) * 32 * r;
                    const long long wgs = (long long)ceil_div(m, rows) * ceil_div(batch, bt) * S;
                    if (wgs > 4ll * kNumCu && S > 1) continue;
                    const int gpw = ceil_div(ceil_div(groups, S), ws);   // key groups per wave
                    const double shape = rt * ct == 8 ? c.shape8 : rt * ct == 6 ? c.shape6 : rt == 4 ? c.shape4x1
                                       : rt == 3 ? c.shape3x1 : (rt == 2 && ct == 2) ? c.shape2x2
                                       : rt == 2 ? c.shape2x1 : ct == 2 ? c.shape1x2 : c.shape1x1;
                    const double rounds = (double)ceil_div_ll(wgs, kNumCu);
                    const double bpad_mb = (double)ceil_div(batch, bt) * bt * 4 / 1e6;   // MB per element of a vector
                    double t = (double)terms * rt * ct * gpw * 16 * 33 * shape / 2100.0 * rounds;
                    t += c.fix + c.per_tile * rt * ct * rounds + c.per_round * (rounds - 1.0) + c.split_per_mb * bpad_mb * n;
                    if (S > 1) t += c.second_kernel + c.second_per_mb * (S + 1.0) * bpad_mb * m;
                    if (ws > 1) t += c.per_wave_group * (ws - 1) * rt * ct / 4;
                    if (t < best) {
                        best = t;
                        pl.batch_tile = bt;
                        pl.wave_splits = ws;
                        pl.rows_per_wg = rows;
                        pl.tiles_per_split = ceil_div(groups, S);
                    }
                }
    return plan_finish(pl, m, n, q, batch, mu);
}

// The mapping of the block-scaled matrix-core kernel (row_mode 1): the same candidates, and the same
// kind of estimate (us; left in `est`).  MFMAs per wave: 5 digits x 4 steps per key group and tile, at
// 33 clk and an overhead that falls with the tiles of a wave, but no less than 564 clk per step (the keys
// are requested one key group ahead); 7.7 us for the two dispatches, 1 us per MB of padded X, 0.1 per MB of results.
// What the inputs hold is not known here.  For bf16 values, whose 16-bit weights are expanded per column tile, two
// column tiles are faster (16384 x 4096, 2 planes, 128 vectors 37.6 us instead of 40.0, three bf16 terms 38.1), for others slower
// (50.0 instead of 48.1; with fewer than eight tiles per wave 10-25 %): they are chosen for eight tiles and long rows.
// On 90 shapes (128 .. 16384 columns, 14 .. 256 vectors) the choice is 2.3 % (fp32) and 2.5 % (bf16 values) slower
// than the fastest of up to 36 mappings on average, 19 % at most (one row step more or less of a short row).
// The estimate handed on has constants of its own, for keys from memory and the 6.7 MB of padded X from which the split is
// bound by bandwidth, fitted to 2600 shapes of 1 .. 1000000 rows near the crossovers: 7 % rms (with the constants that
// rank the mappings 17 %: half the time for sixteen key groups per wave, twice for 50 MB of X).
bool plan_digits(biq_plan& pl, int m, int n, int q, int batch, double& est) {
    double best = 1e30;
    est = 1e30;
    if (q > 4) return false;
    pl = biq_plan{};
    pl.kernel = KERNEL_UNPACK_MFMA;
    pl.threads = kUnpackThreads;
    pl.chunks_per_tile = kUnpackGroupBytes;
    pl.input_terms = 3;
    pl.row_mode = 1;
    const int groups = (int)((biq_key_row_stride(n) + kUnpackGroupBytes - 1) / kUnpackGroupBytes);
    for (int bt = 32; bt <= 64; bt += 32)
        for (int ws = 1; ws <= 4; ws *= 2)
            for (int r = 1; r <= 4; r *= 2)
                for (int S = 1; S <= 16; S *= 2) {
                    const int ct = bt / 32, tiles = q * r * ct;
                    if (tiles > kDigitMaxTiles || (S > 1 && S * ws > groups)) continue;
                    const int rows = (4 / ws) * 32 * r;
                    const long long wgs = (long long)ceil_div(m, rows) * ceil_div(batch, bt) * S;
                    if (wgs > 4ll * kNumCu && S > 1) continue;
                    const int gpw = ceil_div(ceil_div(groups, S), ws);   // key groups per wave
                    if (gpw > 64) continue;
                    // workgroups of up to 4 tiles per wave share a CU
                    double rounds = (double)ceil_div_ll(wgs, kNumCu);
                    if (tiles <= 4) rounds = 1.0 + (rounds - 1.0) * (tiles <= 2 && groups == 1 ? 0.6 : 0.95);
                    const double bpad_mb = (double)ceil_div(batch, bt) * bt * 4 / 1e6;   // MB per element of a vector
                    double step = 165.0 * (1.043 * tiles + 1.011);
                    if (step < 564.0) step = 564.0;
                    double t = 7.7 + 0.99 * bpad_mb * n + rounds * (4.0 * gpw * step / 2100.0 + 0.5 * tiles) +
                               0.4e-6 * m * (double)batch;
                    if (S > 1) t += 1.5 + 0.304 * (S + 1.0) * bpad_mb * m;
                    const double rank = ct == 1 ? t : tiles < kDigitMaxTiles ? 1.05 * t : gpw >= 6 ? 0.99 * t : t;
                    if (rank < best) {
                        best = rank;
                        // (what a call takes with its keys from memory)
                        const double cold = step < 622.0 ? 622.0 : step, x_mb = bpad_mb * n;
                        est = 5.5 + (x_mb < 6.7 ? 0.96 * x_mb : 4.82 + 0.24 * x_mb) + rounds * (4.0 * gpw * cold / 1420.0 + 0.3 * tiles) +
                              0.86e-6 * m * (double)batch + (S > 1 ? 2.3 + 0.71 * (S + 1.0) * bpad_mb * m : 0.0);
                        pl.batch_tile = bt;
                        pl.wave_splits = ws;
                        pl.rows_per_wg = rows;
                        pl.tiles_per_split = ceil_div(groups, S);
                    }
                }
    return best < 1e30 && plan_finish(pl, m, n, q, batch, 8);
}

// Estimated time (us) of a matrix product in three 16-bit terms: 2 * 3 flop per weight and padded input vector at 1.45e9
// flop/us.
double three_terms_estimate(int m, int n, int q, int batch) {
    return 10.0 + 6.0 * ((double)q * m * n) * (ceil_div(batch, 32) * 32.0) / 1.45e9;
}

// Default mapping.  Algorithm 2 leaves the tile sizes open; the choices here are:
//  - batch tile: as many input vectors as one lookup can serve with a single wide LDS read
//  - tile width: the largest power-of-two number of key units whose tables fit the LDS budget
//  - chunk splits: bounded so that the partial sums written stay below about twice the
//    bytes the method has to move anyway
//  - rows per workgroup: enough workgroups to fill the 256 CUs several times over
bool plan_generic(biq_plan& pl, int m, int n, int q, int batch, int mu);

bool plan_tables(biq_plan& pl, int m, int n, int q, int batch, int mu) {
    const int UK = unit_keys(mu);
    const int C = ceil_div(n, mu);
    const int E = 1 << mu;
    pl = biq_plan{};
    if (mu == 8 && batch == 1 && q <= 4) {
        // GEMV: workgroups of 1024 threads, 128-chunk tiles, one workgroup per CU when the
        // rows allow it (every further round of workgroups pays the table build again).  With
        // >= 512 rows per CU a workgroup walks all tiles of its rows (no partial sums: measured
        // equal to or faster than a split from there on); otherwise the tiles are split over
        // workgroups as well and the partials are summed by a second small kernel.
        pl.kernel = KERNEL_GEMV8;
        pl.threads = 1024;
        pl.chunks_per_tile = kGemvTileChunks;
        pl.batch_tile = 1;
        const int tiles = ceil_div(C, kGemvTileChunks);
        if (ceil_div(m, 512) >= kNumCu) {
            pl.tiles_per_split = tiles;
            int rows = ceil_div(ceil_div(m, kNumCu), 64) * 64;
            pl.rows_per_wg = rows > 8192 ? 8192 : rows;
            // Odd XCDs stream slower than even ones, by an amount that differs from box to box and
            // grows with the run time (in-kernel time stamps, back-to-back launches, equal shares:
            // workgroups on odd XCDs end 6 % later on one box and 13 % on another with 4096 rows
            // each, 0-7 % with 1024 rows): rows are moved from the odd to the even XCDs, 4.5 % of a
            // workgroup's share from 4096 rows on, 3 % from 2048, in units of 32 rows.
            if (ceil_div(m, pl.rows_per_wg) % kNumXcd == 0 && pl.rows_per_wg >= 2048) {
                const int permille = pl.rows_per_wg >= 4096 ? 45 : 30;
                pl.xcd_skew = ((pl.rows_per_wg * permille / 1000 + 16) / 32) * 32;
                if (tiles > 1 && pl.rows_per_wg + pl.xcd_skew > 8192) pl.xcd_skew = 0;
            }
        } else if (C > kGemvTileChunks && (long long)m * ceil_div(C, kGemvHalfTileChunks) <= 512ll * kNumCu) {
            // small and mid-size (up to where a workgroup of the full-table kernel gets 512 rows and
            // walks all its tiles), wider than one full-table tile: half tables (256 chunks per
            // workgroup), so that rows up to n = 2048 need no split and no second kernel.  One workgroup per CU if the
            // rows allow it (a second round of workgroups pays the table build again), at least
            // 8 rows each; 4 rows per wave step, up to 9 steps per wave (few blocks of many splits: 6896 x 36882, 3 planes).
            pl.kernel = KERNEL_GEMV8H;
            pl.chunks_per_tile = kGemvHalfTileChunks;
            pl.tiles_per_split = 1;
            pl.row_mode = 1;
            const int tiles_h = ceil_div(C, kGemvHalfTileChunks);
            if (tiles_h == 2 || tiles_h == 3) {
                // two or three tiles: a workgroup walks them (a table build of 1.3 us each) rather
                // than sharing the row with other workgroups, which costs a second dispatch (2.5 us
                // and more) for the sum of the partial results
                pl.tiles_per_split = tiles_h;
                pl.rows_per_wg = rows_from(ceil_div(m, kNumCu), 4, 8, m);
            } else {
                pl.rows_per_wg = rows_one_round(m, tiles_h, kNumCu, 4, 8);
                // up to one row per wave: 64 lanes per row instead of 16 (4 lookups per lane and plane)
                if (pl.rows_per_wg <= 16) pl.row_mode = 2;
            }
        } else if ((long long)m * tiles <= 4ll * 128 * kNumCu) {
            // small: latency mode, 8 rows per wave step, at most 4 steps per wave
            pl.tiles_per_split = 1;
            pl.row_mode = 1;
            pl.rows_per_wg = rows_one_round(m, tiles, kNumCu, 8, 8);
        } else {
            pl.tiles_per_split = 1;
            const int rows = rows_one_round(m, tiles, kNumCu, 64, 64);
            pl.rows_per_wg = rows > 8192 ? 8192 : rows;
        }
        return plan_finish(pl, m, n, q, batch, mu);
    }
    if (mu == 8 && batch >= 2 && q <= 4 && C > kGemmTileChunks &&
        product(m, ceil_div(C, kGemmHalfTileChunks), ceil_div(batch, 2)) <= 512ll * kNumCu) {
        // Small batched calls wider than one full-table tile: half tables (128 chunks x 2 input
        // vectors per workgroup) halve the number of row splits; up to n = 1024 there is none and
        // no second kernel.  One workgroup per CU if the rows allow it, at least 8 rows each;
        // 8 rows per wave step, up to 8 steps per wave (one block of all rows: 992 x 10379, 1 plane, 24 vectors).
        pl.kernel = KERNEL_GEMM8X2H;
        pl.threads = 1024;
        pl.chunks_per_tile = kGemmHalfTileChunks;
        pl.batch_tile = 2;
        pl.tiles_per_split = 1;
        pl.row_mode = 1;
        pl.rows_per_wg = rows_one_round(m, product(ceil_div(C, kGemmHalfTileChunks), ceil_div(batch, 2), 1), kNumCu, 8, 8);
        return plan_finish(pl, m, n, q, batch, mu);
    }
    if (mu == 8 && batch >= 2 && q <= 4) {
        // Batched: workgroups of 1024 threads over (row block, chunk split, pair of input
        // vectors).  Rows per workgroup as many as the LDS row accumulators hold (4096), so that
        // a table build is amortised over many lookups; tiles are split over workgroups only as
        // far as needed to give every CU a workgroup; if that is still not enough, rows shrink.
        pl.kernel = KERNEL_GEMM8X2;
        pl.threads = 1024;
        pl.chunks_per_tile = kGemmTileChunks;
        pl.batch_tile = kGemmBT;
        const int tiles = ceil_div(C, kGemmTileChunks);
        const int T = ceil_div(batch, kGemmBT);
        int rows = m > 4096 ? 4096 : ceil_div(m, 64) * 64;
        const long long RT = (long long)ceil_div(m, rows) * T;
        int S = 1;
        if (RT < kNumCu) {
            S = (int)ceil_div_ll(kNumCu, RT);
            if (S > tiles) S = tiles;
        }
        pl.tiles_per_split = ceil_div(tiles, S);
        S = ceil_div(tiles, pl.tiles_per_split);
        // (one tile per workgroup: no accumulators in LDS, a few rows more than 4096 for one round of workgroups)
        if (RT * S < kNumCu || (pl.tiles_per_split == 1 && RT * S > kNumCu && (long long)T * S <= kNumCu)) {
            const int r2 = rows_one_round(m, (long long)T * S, kNumCu, 64, 64);
            if (r2 < rows || (RT * S > kNumCu && r2 <= 8192 && r2 * (long long)biq_key_row_stride(n) < (1ll << 31))) rows = r2;
        }
        if (pl.tiles_per_split == 1 && rows <= 4 * 256) {
            // few rows per workgroup: latency mode, 16 rows per wave step, at most 4 steps per wave
            pl.row_mode = 1;
            rows = ceil_div(rows, 256) * 256;
        }
        pl.rows_per_wg = rows;
        return plan_finish(pl, m, n, q, batch, mu);
    }
    if ((mu <= 5 || (mu == 6 && batch <= 4)) && C >= 16 * UK) {
        // Narrow keys, rows at least half a tile wide: 32 lanes per row, conflict-free gathers.
        // (mu = 6 holds one input vector per pass only and re-reads the keys per vector: measured
        // faster than the generic kernel up to 4 input vectors, slower from 16 on.)
        // One tile per workgroup (wider rows are split, partial sums through the workspace); one
        // workgroup per CU (the tables fill the LDS: a second round of workgroups would only
        // build tables again), at least 32 rows (one step of the 16 waves) each.
        pl.kernel = KERNEL_WIDE;
        pl.threads = 1024;
        pl.chunks_per_tile = 32 * UK;
        pl.batch_tile = (128 * 1024) / (32 * UK * E * 4);
        pl.tiles_per_split = 1;
        const int rows = rows_one_round(m, product(ceil_div(C, pl.chunks_per_tile), ceil_div(batch, pl.batch_tile), 1), kNumCu, 32, 32);
        pl.rows_per_wg = rows > (1 << 20) ? (1 << 20) : rows;
        return plan_finish(pl, m, n, q, batch, mu);
    }
    return plan_generic(pl, m, n, q, batch, mu);
}

// The generic kernel: any mu, any q.
bool plan_generic(biq_plan& pl, int m, int n, int q, int batch, int mu) {
    const int UK = unit_keys(mu);
    const int C = ceil_div(n, mu);
    const int E = 1 << mu;
    pl = biq_plan{};
    pl.kernel = KERNEL_GENERIC;
    pl.batch_tile = batch >= 5 ? 8 : batch >= 3 ? 4 : batch;
    // one key unit's tables must fit the LDS budget (mu = 9, 10: 64 KiB per unit and input vector)
    while (pl.batch_tile > 1 && (long long)UK * E * pl.batch_tile * 4 > kLdsTableBudget) pl.batch_tile /= 2;
    // widest tile: G units, G a power of two, tables within the budget, no wider than the row
    int G = 1;
    while (G < 64 && (long long)(2 * G) * UK * E * pl.batch_tile * 4 <= kLdsTableBudget &&
           G * UK < C)
        G *= 2;
    pl.chunks_per_tile = G * UK;
    const int tiles = ceil_div(C, pl.chunks_per_tile);
    pl.threads = 512;
    const int groups = pl.threads / G;
    const int batch_tiles = ceil_div(batch, pl.batch_tile);
    // chunk splits
    const __int128 result_bytes = (__int128)4 * m * batch;
    const __int128 algo_bytes = (__int128)q * m * ceil_div(n, 8) + 4ll * q * m + (__int128)4 * n * batch + result_bytes;
    long long max_splits = (long long)((2 * algo_bytes) / result_bytes);
    if (max_splits < 1) max_splits = 1;
    int splits = tiles < max_splits ? tiles : (int)max_splits;
    pl.tiles_per_split = ceil_div(tiles, splits);
    splits = ceil_div(tiles, pl.tiles_per_split);
    // rows per workgroup: aim at 2 workgroups per CU (every workgroup builds its own tables, and
    // with the tables filling most of the LDS only one is resident per CU anyway; measured: 8 per
    // CU was up to 2.7x slower on small-batch calls) while each keeps >= 1 row iteration
    const long long row_iters = ceil_div(m, groups);
    const long long want_wgs = 2ll * kNumCu;
    long long k = product(row_iters, splits, batch_tiles) / want_wgs;
    if (k < 1) k = 1;
    if (k > 64) k = 64;
    if (pl.tiles_per_split > 1) {
        // row accumulators share the LDS with the tables
        const long long table_bytes = (long long)pl.chunks_per_tile * E * pl.batch_tile * 4;
        const long long fit = (kLdsPerCu - table_bytes) / (4ll * pl.batch_tile * groups);
        if (k > fit) k = fit < 1 ? 1 : fit;
    }
    pl.rows_per_wg = (int)(k * groups);
    return plan_finish(pl, m, n, q, batch, mu);
}

// The library's plan for a shape.  Should the tuned choice not pass plan_finish (a shape outside
// what its kernel's 32-bit offsets cover), the generic kernel takes the call; false if that
// fails too (the caller reports BIQ_EUNSUPPORTED, sizes read as 0).
// Many input vectors: the contraction is compute bound and the matrix cores (block-scaled digits) beat
// the table lookups, from the estimated times of both.
bool plan_default(biq_plan& pl, int m, int n, int q, int batch, int mu, bool tables_given = false,
                  DirectGeom* geom = nullptr) {
    const bool ok = plan_tables(pl, m, n, q, batch, mu) || plan_generic(pl, m, n, q, batch, mu);
    if (tables_given || q > 4) return ok;
    // Few vectors, no tables: the plan stays the table kernel's (what biq_query runs for the shape), marked
    // by table_fill = 2.  Fewer than 128 rows (less than one row step of a workgroup) keep the tables, whose sums
    // biq_query repeats bit for bit.
    DirectGeom local{};
    DirectGeom& g = geom ? *geom : local;             // (a caller that launches the direct kernel has use for it)
    if (mu == 8 && batch == 1) {
        // One vector: rows beyond one half-table tile, i.e. where the tables take several builds or a second dispatch, if
        // direct, whose estimate is 7 to 12 % low, is estimated well below them (700 shapes, 128 .. 500000 rows, 2049 ..
        // 16384 columns, keys from memory: 0.7 % slower in the mean than the better of both).  Even widths: 0.865 of the tables'
        // (368 shapes: none takes 5 % longer than it would with tables; with 0.9 three do, for 0.1 % less in the mean).  Odd widths:
        // 0.95 (332 shapes; with 0.865 0.3 % more in the mean, and five go to the tables that took direct before the tables' side
        // was estimated here).  Tables / direct: 256 x 5952, 3 planes 8.6 / 5.6; 4096 x 4096, 2 6.6 / 5.0; 4096 x 11008, 2 9.5 / 8.2;
        // 16384 x 4096, 2 8.6 / 7.7; 5000 x 3001, 3 12.2 / 6.4; 11008 x 4096, 3 (tables) 9.6 / 8.9; but 1088 x 9288, 4 8.4 / 9.7;
        // 234 x 32722, 4 12.7 / 19.9; 36294 x 3136, 2 12.6 / 15.8.  The full-table kernel (33 MB of keys per plane and more) keeps its
        // calls: 47993 x 6847, 3 37 / 40.
        if (ok && m >= 128 && n > 2048 && pl.kernel == KERNEL_GEMV8H && direct_geometry(g, m, n, q, 1) &&
            g.est < (n % 4 ? 0.95 : 0.865) * tables_estimate(pl, m, n, q, 1, mu))
            pl.table_fill = 2;
        return ok;
    }
    const double tables = ok ? tables_estimate(pl, m, n, q, batch, mu) : 1e30;
    const double direct = ok && m >= 128 && direct_geometry(g, m, n, q, batch) ? g.est : 1e30;
    // The one estimated faster; direct's errors are also the smaller ones (5-8e-8 against 1.0-1.3e-7), so it has the ties.  The
    // generic kernel's estimate is the looser one, and misses on the low side: it keeps what it wins clearly, but one vector on rows
    // of up to 128 columns, where direct's is 20 % low (80000 x 128, mu = 7, 1 plane 4.4 us tables / 5.9 direct).  Not for one vector
    // on a few short rows (982 x 144, 2: 3.7 / 4.0; but 68544 x 206, 3, mu = 6: 13.6 / 6.5).  3200 shapes of 2 .. 256 vectors,
    // mu = 8: 0.6 % slower in the mean than the best of tables, direct and digits, 1.7 % of them by more than 10 % (up to 5e7
    // operations 0.3 and 0.6 %); 700 with other mu 0.6 and 2 %.  Tables / direct: 1145 x 7117, 4, 7 12.2 / 12.7;
    // 919 x 832, 3, 9 4.6 / 6.5; 1541 x 384, 2, 4 4.4 / 4.6; 512 x 512, 2, 2 4.3 / 3.8; 1024 x 512, 2, 3 4.5 / 3.9; 1536 x 128, 2, 3
    // 4.3 / 3.8; 2048 x 1024, 2, 4 4.3 / 5.4; 10240 x 1216, 2, 12 12.4 / 8.8; 1088 x 510, 2, 181 7.7 / 6.8; mu = 7: 1790 x 316, 3, 5
    // 18.6 / 4.7; mu = 4: 458 x 2061, 3, 15 7.9 / 11.5; 38243 x 14976, 1, 1 35.0 / 27.9.
    const bool brief = batch == 1 && n <= 512 && (long long)m * q < 4096;
    const double margin = pl.kernel != KERNEL_GENERIC ? 1.0 : batch > 1 ? 1.3 : n > 128 ? 1.05 : 0.8;
    const bool use_direct = !brief && direct < margin * tables;
    // (one vector padded to 32 is never the better use of the matrix cores where direct takes it: 310460 x 192, mu = 4
    // 17 us in digits, 6.8 with tables)
    if (batch == 1 && (brief || direct < 1e30)) {
        if (use_direct) pl.table_fill = 2;
        return ok;
    }
    const double few = use_direct ? direct : tables;
    // (no digit plan takes less than 8 us: small calls, where this search would show, skip it; the narrow-key kernel
    // keeps calls below 5e6 multiply-adds that direct does not take: 129 x 5000, 2 planes, 3 vectors at mu = 3 12.6 us
    // with tables, 12.5 with digits)
    if (few >= 8.3 && !(pl.kernel == KERNEL_WIDE && (double)q * m * n * batch < 5e6)) {
        biq_plan d;
        double est;
        if (!plan_digits(d, m, n, q, batch, est)) {
            // rows too long for those plans: the exact three-term split
            if (three_terms_estimate(m, n, q, batch) < few && plan_unpack(d, m, n, q, batch, mu, 3)) {
                pl = d;
                return true;
            }
        } else if (est < (use_direct ? 1.05 : 0.95) * few) {
            // (3900 shapes: one margin for both, or direct's 1.0 or 1.1, has more that take 10 % longer; digits instead of direct
            // at 14464 x 10824, 2 planes, 20 vectors 101 -> 36 us)
            pl = d;
            return true;
        }
    }
    if (use_direct) pl.table_fill = 2;
    return ok;
}

// Bytes of the prepared-input area at the start of the workspace (unpack-MFMA plans only): the
// B fragments, then one scaling exponent per padded input vector (two terms) or one count of
// non-zero terms per MFMA step and column tile (three).
size_t plan_xfrag_bytes(const biq_plan& pl) {
    const size_t b = (size_t)pl.batch_tiles * pl.chunk_splits * pl.tiles_per_split *
                     (size_t)unpack_group_pieces(pl.batch_tile, pl.input_terms) * 16;
    return (b + 255) & ~(size_t)255;
}
size_t plan_xf_bytes(const biq_plan& pl) {
    if (pl.kernel != KERNEL_UNPACK_MFMA) return 0;
    const size_t e = pl.input_terms == 2
                         ? (size_t)pl.batch_tiles * pl.batch_tile * sizeof(int)
                         : (size_t)pl.batch_tiles * pl.chunk_splits * pl.tiles_per_split * 16 * (pl.batch_tile / 32) *
                               sizeof(int);
    return plan_xfrag_bytes(pl) + ((e + 255) & ~(size_t)255);
}

size_t plan_workspace(const biq_plan& pl, int m, int batch) {
    return plan_xf_bytes(pl) +
           (pl.chunk_splits > 1 ? (size_t)pl.chunk_splits * batch * m * sizeof(float) : 0);
}

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// mu = 8, tables in device memory: lookups read the tables where they lie instead of from a copy in LDS
// (biq_gather.h) if there are few of them.  A copy costs 16-17 us per tile a workgroup walks and the second dispatch of
// a split row; the reads, counted per four input vectors, 3.7-5 us per million up to 4 vectors, 2.8 up to 8 and 1.8-2.6
// beyond, where neighbouring lanes share an entry's lines (gather_log_slices).  Copied / in place: 4071 x 1941, 2
// planes, 5 vectors (4.0 million) 20.1 / 11.0 us; 3345 x 4044, 2, 7 (6.8) 22.3 / 19.6; 2397 x 3767, 4, 7 (9.0) 23.2 / 25.1;
// 3970 x 2085, 2, 13 (8.3) 40 / 15; one vector, two tiles: 4096 x 4096, 4 planes (8.4) 32.8 / 30.0.  Tables of very long rows lie
// beyond the L2s, and shared lines save less: more than 64 splits: 64 x 131072, 1, 4 (1.0) 53 / 51; 183 x 90112, 1, 3 (2.1)
// 62 / 51; 30 x 174080, 3, 8 (3.9) 101 / 79; but up to 4 vectors 66 x 201728, 2, 4 (3.3) 93 / 102; 78 x 97113, 4, 4 (3.8)
// 66 / 83; and 66 x 120657, 3, 7 (6.0) 72 / 89.
constexpr long long kGatherLookups = 4200000;
bool gather_tables(const biq_plan& pl, int m, int q, int batch, int C) {
    if (pl.kernel != KERNEL_GEMV8 && pl.kernel != KERNEL_GEMV8H && pl.kernel != KERNEL_GEMM8X2 &&
        pl.kernel != KERNEL_GEMM8X2H)
        return false;
    // 32-bit offsets: at most 1 GiB of tables, and less than 4 GiB up to the end of the last tile, since lanes
    // address whole tiles and a chunk past the row counts as 0 only while its offset does not wrap (one chunk,
    // 131072 vectors: chunk 32 would be chunk 0 again); slices of 4 vectors are the grid's y, at most 65535
    const long long tile_end = (long long)ceil_div(C, pl.chunks_per_tile) * pl.chunks_per_tile;
    if (pl.row_mode == 0 || (long long)C * batch > (1ll << 20) || tile_end * batch >= (1ll << 22)) return false;
    if (ceil_div(batch, 4) > 65535) return false;
    const int log_slices = batch > 1 ? gather_log_slices(batch) : 0;
    const long long limit = batch > 1 && pl.chunk_splits > kGatherSplits
                                ? (log_slices ? kGatherLookups : kGatherLookups * 3 / 4)
                                : (kGatherLookups * pl.tiles_per_split * (2 + log_slices)) >> 1;
    return (long long)m * q * C * ceil_div(batch, 4) <= limit;
}

// The same for the plans of query_kernel, whose copies cost 12-25 us and whose lookups cost three times those of the
// other kernels, and of query_wide_kernel (13-15 us), any mu.  Copied / in place: 163 x 223, 4 planes, 14 vectors, mu = 4 12.5 /
// 5.2 us; 4080 x 1318, 3, 7, 4 (8.1 million) 27.5 / 12.8; 2783 x 3596, 4, 12, 6 (20.0) 45.6 / 37.9; query_wide:
// 3596 x 1817, 2, 4, 6 (2.2) 13.6 / 10.8; 1547 x 3857, 4, 2, 5 (4.8) 17.3 / 18.4; 2290 x 3782, 4, 3, 3 (11.6) 23.7 / 22.7;
// 2902 x 3374, 4, 8, 4 (19.6) 23.8 / 39.5.
constexpr long long kGatherUnitLookups = 20000000;
bool gather_units(const biq_plan& pl, int m, int q, int batch, int mu, int C) {
    if (pl.kernel != KERNEL_GENERIC && pl.kernel != KERNEL_WIDE) return false;
    const long long tile_end = (long long)ceil_div(C, pl.chunks_per_tile) * pl.chunks_per_tile;
    if (product((long long)C << mu, batch, 1) > (1ll << 28) || product(tile_end << mu, batch, 1) >= (1ll << 30)) return false;
    if (ceil_div(batch, 4) > 65535 || pl.chunk_splits > kGatherSplits) return false;
    const int keys = unit_keys(mu);
    if (gather_units_crowd(gather_units_shape(ilog2(pl.chunks_per_tile / keys), m, batch, pl.chunk_splits), batch, pl.chunk_splits,
                           pl.tiles_per_split, q, keys, ((long long)C << mu) * batch * 4))
        return false;
    return product((long long)m * q, C, ceil_div(batch, 4)) <= (pl.kernel == KERNEL_WIDE ? kGatherLookups : kGatherUnitLookups);
}

// Kernel parameters of a lookup-table plan.
void fill_query_params(QueryParams& qp, const biq_plan& pl, const uint8_t* K, const float* alpha, const float* X,
                       const float* LUT, float* out, int m, int n, int q, int batch, int mu) {
    qp.K = reinterpret_cast<const uint32_t*>(K);
    qp.alpha = alpha;
    qp.X = X;
    qp.LUT = LUT;
    qp.out = out;
    qp.m = m; qp.n = n; qp.q = q; qp.batch = batch;
    qp.stride_dw = (int)(biq_key_row_stride(n) / 4);
    qp.C = ceil_div(n, mu);
    qp.CT = pl.chunks_per_tile;
    qp.G = pl.chunks_per_tile / unit_keys(mu);
    qp.log2G = ilog2(qp.G);
    qp.tiles = ceil_div(qp.C, qp.CT);
    qp.tps = pl.tiles_per_split;
    qp.splits = pl.chunk_splits;
    qp.rows_per_wg = pl.rows_per_wg;
    qp.row_blocks = pl.row_blocks;
    qp.batch_tiles = pl.batch_tiles;
    qp.ntasks = pl.row_blocks * pl.chunk_splits * pl.batch_tiles;
    qp.tasks_per_xcd = ceil_div(qp.ntasks, kNumXcd);
    qp.row_mode = pl.row_mode;
    qp.xcd_skew = pl.xcd_skew;
    qp.table_fill = LUT ? (batch == 1 && gather_tables(pl, m, q, batch, qp.C)) : pl.table_fill;
}

// Plan of one problem of a grouped launch: mu = 8, at most 4 planes, a single dispatch without
// workspace (rows no wider than one tile), and only `cus` CUs' worth of workgroups, since the
// other problems of the group fill the rest of the chip.  false: the shape needs biq_gemm.
bool plan_grouped(biq_plan& pl, int& kind, int m, int n, int q, int batch, int mu, int cus) {
    if (mu != 8 || q > 4) return false;
    const int C = ceil_div(n, 8);
    pl = biq_plan{};
    pl.threads = 1024;
    pl.tiles_per_split = 1;
    pl.row_mode = 1;
    if (batch == 1 && C <= kGemvTileChunks) {
        kind = GROUP_GEMV8;
        pl.kernel = KERNEL_GEMV8;
        pl.chunks_per_tile = kGemvTileChunks;
        pl.batch_tile = 1;
        pl.rows_per_wg = rows_from(ceil_div_ll(m, cus), 8, 8, m);
    } else if (batch == 1 && C <= kGemvHalfTileChunks) {
        kind = GROUP_GEMV8H;
        pl.kernel = KERNEL_GEMV8H;
        pl.chunks_per_tile = kGemvHalfTileChunks;
        pl.batch_tile = 1;
        pl.rows_per_wg = rows_from(ceil_div_ll(m, cus), 4, 8, m);
    } else if (batch >= 2 && C <= kGemmHalfTileChunks) {
        kind = GROUP_GEMM8X2H;
        pl.kernel = KERNEL_GEMM8X2H;
        pl.chunks_per_tile = kGemmHalfTileChunks;
        pl.batch_tile = 2;
        pl.rows_per_wg = rows_one_round(m, ceil_div(batch, 2), cus, 8, 8);
    } else {
        return false;
    }
    return plan_finish(pl, m, n, q, batch, mu) && pl.chunk_splits == 1;
}

// Large-batch path: split X into 16-bit terms in MFMA operand order (workspace), contract, and
// sum the partial results when the key groups were split over workgroups.
biq_status run_unpack_mfma(const biq_plan& pl, const uint8_t* K, const float* alpha, const float* X,
                           float* Y, int m, int n, int q, int batch, void* workspace, hipStream_t s) {
    const int CT = pl.batch_tile / 32;
    const int groups = (int)((biq_key_row_stride(n) + kUnpackGroupBytes - 1) / kUnpackGroupBytes);
    const int steps = groups * 16;  // MFMA steps along a row
    mfma_u32x4* Xf = reinterpret_cast<mfma_u32x4*>(workspace);
    int* colexp = reinterpret_cast<int*>(reinterpret_cast<char*>(workspace) + plan_xfrag_bytes(pl));
    float* partial = reinterpret_cast<float*>(reinterpret_cast<char*>(workspace) + plan_xf_bytes(pl));

    if (pl.row_mode == 1) {
        uint8_t* Xd = reinterpret_cast<uint8_t*>(workspace);
        if (launch_xdigits(CT, X, Xd, colexp, n, batch, groups, pl.batch_tiles, s) != hipSuccess) return BIQ_EHIP;
        DigitParams dp{};
        dp.K = K;
        dp.alpha = alpha;
        dp.Xd = Xd;
        dp.form = colexp;
        dp.out = pl.chunk_splits > 1 ? partial : Y;
        dp.m = m;
        dp.batch = batch;
        dp.stride_bytes = (uint32_t)biq_key_row_stride(n);
        dp.groups = groups;
        dp.gps = pl.tiles_per_split;
        dp.splits = pl.chunk_splits;
        dp.row_blocks = pl.row_blocks;
        dp.col_groups = pl.batch_tiles;
        dp.ntasks = pl.row_blocks * pl.chunk_splits * pl.batch_tiles;
        dp.tasks_per_xcd = ceil_div(dp.ntasks, kNumXcd);
        const int grid = dp.tasks_per_xcd * kNumXcd;
        const int rpw = pl.rows_per_wg / ((4 / pl.wave_splits) * 32);
        const auto launch = pl.wave_splits == 1 ? launch_digits_ws1
                          : pl.wave_splits == 2 ? launch_digits_ws2 : launch_digits_ws4;
        if (launch(q, rpw, CT, dp, grid, pl.lds_bytes, s) != hipSuccess) return BIQ_EHIP;
        if (pl.chunk_splits > 1 &&
            launch_reduce_splits(partial, Y, (long long)batch * m, pl.chunk_splits, s) != hipSuccess)
            return BIQ_EHIP;
        return BIQ_OK;
    }
    if (launch_xsplit(pl.input_terms, CT, X, Xf, colexp, n, batch, steps, pl.batch_tiles * pl.batch_tile, s) !=
        hipSuccess)
        return BIQ_EHIP;

    UnpackParams up{};
    up.K = K;
    up.alpha = alpha;
    up.Xf = Xf;
    up.colexp = colexp;
    up.nterms = colexp;   // the same area: exponents (two terms) or term counts (three)
    up.out = pl.chunk_splits > 1 ? partial : Y;
    up.m = m;
    up.batch = batch;
    up.stride_bytes = (uint32_t)biq_key_row_stride(n);
    up.groups = groups;
    up.gps = pl.tiles_per_split;
    up.splits = pl.chunk_splits;
    up.row_blocks = pl.row_blocks;
    up.col_groups = pl.batch_tiles;
    up.ntasks = pl.row_blocks * pl.chunk_splits * pl.batch_tiles;
    up.tasks_per_xcd = ceil_div(up.ntasks, kNumXcd);
    const int grid = up.tasks_per_xcd * kNumXcd;
    const int rpw = pl.rows_per_wg / ((4 / pl.wave_splits) * 32);
    const hipError_t e = launch_unpack(pl.input_terms, q, rpw, CT, pl.wave_splits, up, grid, pl.lds_bytes, s);
    if (e != hipSuccess) return BIQ_EHIP;
    if (pl.chunk_splits > 1) {
        const long long count = (long long)batch * m;
        if (launch_reduce_splits(partial, Y, count, pl.chunk_splits, s) != hipSuccess) return BIQ_EHIP;
    }
    return BIQ_OK;
}

// Few input vectors, no tables (table_fill 2).  g: the geometry, or row_blocks = 0 if it is still to be found.
biq_status run_direct(DirectGeom& g, const uint8_t* K, const float* alpha, const float* X, float* out, int m, int n, int q,
                      int batch, hipStream_t s) {
    if (g.row_blocks == 0 && !direct_geometry(g, m, n, q, batch)) return BIQ_EUNSUPPORTED;
    DirectParams p{};
    p.K = K;
    p.alpha = alpha;
    p.X = X;
    p.out = out;
    p.m = m;
    p.n = n;
    p.batch = batch;
    p.stride_bytes = (uint32_t)biq_key_row_stride(n);
    p.chunks = g.chunks;
    p.chunks_inv = (uint32_t)((((uint64_t)1 << 32) + g.chunks - 1) / g.chunks);   // (not used for one chunk)
    p.vecs = g.vecs;
    p.log_ksplit = ilog2(g.ksplit);
    p.units_per_group = ceil_div(ceil_div(g.chunks, g.uc), g.ksplit);
    p.steps = g.steps;
    const auto launch = g.kind == DIRECT_MANY ? launch_direct_many : g.kind == DIRECT_LINES ? launch_direct_lines : launch_direct_few;
    return launch(q, ceil_div(g.vecs, 3), p, dim3(g.row_blocks, g.batch_tiles), g.lds, s) == hipSuccess ? BIQ_OK : BIQ_EHIP;
}

biq_status run_query(bool fused, const uint8_t* K, const float* alpha, const float* X,
                     const float* LUT, float* Y, int m, int n, int q, int batch, int mu,
                     const biq_plan* user_plan, void* workspace, size_t workspace_bytes,
                     void* stream) {
    if (!shape_ok(m, n, q, batch, mu)) return BIQ_EINVAL;
    if (!K || !alpha || !Y || (fused ? !X : !LUT)) return BIQ_EINVAL;
    if (!aligned(K, 16) || !aligned(alpha, 4) || !aligned(Y, 4) || !aligned(fused ? X : LUT, 4))
        return BIQ_EINVAL;
    biq_plan pl;
    DirectGeom geom{};
    if (user_plan) {
        pl = *user_plan;
        if (!plan_finish(pl, m, n, q, batch, mu)) return BIQ_EINVAL;
    } else {
        if (!plan_default(pl, m, n, q, batch, mu, !fused, &geom)) return BIQ_EUNSUPPORTED;
    }
    if (pl.kernel == KERNEL_UNPACK_MFMA && !fused) return BIQ_EINVAL;  // that kernel reads X, not tables
    if (pl.table_fill != 0 && !fused) return BIQ_EINVAL;               // a build method needs tables to build
    const size_t need = plan_workspace(pl, m, batch);
    if (need > 0) {
        if (!workspace || workspace_bytes < need) return BIQ_EWORKSPACE;
        if (!aligned(workspace, 16)) return BIQ_EINVAL;
    }
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (pl.kernel == KERNEL_UNPACK_MFMA)
        return run_unpack_mfma(pl, K, alpha, X, Y, m, n, q, batch, workspace, s);
    if (pl.table_fill == 2) return run_direct(geom, K, alpha, X, Y, m, n, q, batch, s);

    // (given tables, several input vectors or other than mu = 8: read in place, splits added in the same dispatch where
    // they don't need the chip's other CUs)
    const int C = ceil_div(n, mu);
    const bool units = !fused && gather_units(pl, m, q, batch, mu, C);
    const bool gather = !fused && batch > 1 && gather_tables(pl, m, q, batch, C);
    const bool waves = gather && gather_in_waves(pl.kernel == KERNEL_GEMM8X2H ? 8 : 4, m, q, batch, pl.chunk_splits);
    const bool parts = pl.chunk_splits > 1 && !units && !waves;
    QueryParams qp{};
    fill_query_params(qp, pl, K, alpha, X, LUT, parts ? reinterpret_cast<float*>(workspace) : Y, m, n, q,
                      batch, mu);
#ifdef BIQ_TRACE
    if (fused) qp.LUT = reinterpret_cast<const float*>(workspace);  // time stamps of a trace build go here
#endif
    const int grid = qp.tasks_per_xcd * kNumXcd;

    hipError_t e;
    if (units) e = launch_gather_units(mu, qp, pl.kernel == KERNEL_WIDE, s);
    else if (gather) e = launch_gather(pl.kernel == KERNEL_GEMM8X2H, q, qp, waves, s);
    else if (pl.kernel == KERNEL_GEMV8) e = launch_gemv8(fused, q, qp, grid, pl.threads, pl.lds_bytes, s);
    else if (pl.kernel == KERNEL_GEMV8H) e = launch_gemv8h(fused, q, qp, grid, pl.threads, pl.lds_bytes, s);
    else if (pl.kernel == KERNEL_WIDE) e = launch_wide(fused, mu, qp, grid, pl.threads, pl.lds_bytes, s);
    else if (pl.kernel == KERNEL_GEMM8X2H) e = launch_gemm8x2h(fused, q, qp, grid, pl.threads, pl.lds_bytes, s);
    else if (pl.kernel == KERNEL_GEMM8X2) e = launch_gemm8x2(fused, q, qp, grid, pl.threads, pl.lds_bytes, s);
    else e = launch_query_generic(fused, mu, pl.batch_tile, qp, grid, pl.threads, pl.lds_bytes, s);
    if (e != hipSuccess) return BIQ_EHIP;
    if (parts) {
        const long long count = (long long)batch * m;
        if (launch_reduce_splits(reinterpret_cast<const float*>(workspace), Y, count, pl.chunk_splits, s) !=
            hipSuccess)
            return BIQ_EHIP;
    }
    return BIQ_OK;
}

template <typename KEY>
biq_status unpack_keys_any(const uint8_t* K, KEY* keys, int m, int n, int q, int mu, void* stream) {
    if (!shape_ok(m, n, q, 1, mu) || !K || !keys) return BIQ_EINVAL;
    if (!aligned(K, 16) || !aligned(keys, sizeof(KEY))) return BIQ_EINVAL;
    if (mu > 8 * (int)sizeof(KEY)) return BIQ_EUNSUPPORTED;  // key does not fit the output type
    const long long key_rows = (long long)q * m;
    const int stride_dw = (int)(biq_key_row_stride(n) / 4);
    const int C = ceil_div(n, mu);
    const hipError_t e = launch_unpack_keys(mu, sizeof(KEY) == 2, reinterpret_cast<const uint32_t*>(K), keys,
                                            key_rows, C, stride_dw, reinterpret_cast<hipStream_t>(stream));
    return e == hipSuccess ? BIQ_OK : BIQ_EHIP;
}

// ---- the allocation-free entry point's scratch buffer -------------------------------------
// The plan of biq_gemm_noalloc where the digit plan does not fit its buffer (digits and partial sums of
// wide batches): the tables, or - where a three-term matrix product is faster than they are - that one, from
// lookups/s (13e12 for the conflict-free kernels, 6.5e12 and no more than 0.25 TB/s of keys for the generic
// one, plus 6 us).
bool plan_small_workspace(biq_plan& pl, int m, int n, int q, int batch, int mu) {
    const double weights = (double)q * m * n;
    const bool tuned = mu == 8 || mu <= 5 || (mu == 6 && batch <= 4);
    double t_lut = weights / mu * batch / (tuned ? 13e6 : 6.5e6);
    if (!tuned && t_lut < weights / 8 / 0.25e6) t_lut = weights / 8 / 0.25e6;
    if (q <= 4 && three_terms_estimate(m, n, q, batch) < t_lut + 6.0) return plan_unpack(pl, m, n, q, batch, mu, 3);
    return plan_default(pl, m, n, q, batch, mu, true);
}
// ... and where that one does not fit either: of the tables' plan (without tables, where direct is the faster one) and the
// matrix cores' (digits; three terms for rows too long for those) the one that fits, the faster one by the estimates if
// both do.  Many vectors on the tables, which often need no workspace at all, are left to the caller from kNoallocSlower
// times the matrix cores' time on: biq_gemm with a workspace is the better call, and BIQ_EWORKSPACE says so (16384 x 16384,
// 2 planes, 512 vectors: 4.4 times).  Few rows with many inputs, where the split of the inputs is most of a call, have 1 us
// per MB of them on top.
constexpr double kNoallocSlower = 4.0;
bool plan_fitting(biq_plan& pl, int m, int n, int q, int batch, int mu, size_t limit) {
    biq_plan lut, cores;
    double t_cores = 1e300;
    const bool have_lut = plan_default(lut, m, n, q, batch, mu, true);
    if (!plan_digits(cores, m, n, q, batch, t_cores))
        t_cores = plan_unpack(cores, m, n, q, batch, mu, 3) ? three_terms_estimate(m, n, q, batch) : 1e300;
    double t_lut = have_lut ? tables_estimate(lut, m, n, q, batch, mu) : 1e300;
    DirectGeom g;
    if (have_lut && m >= 128 && direct_geometry(g, m, n, q, batch) && g.est < t_lut) {
        t_lut = g.est;
        lut.table_fill = 2;
    }
    const bool cores_fit = t_cores < 1e300 && plan_workspace(cores, m, batch) <= limit;
    const bool lut_fits = have_lut && plan_workspace(lut, m, batch) <= limit && t_lut < kNoallocSlower * (t_cores + 4e-6 * n * (double)batch);
    pl = cores_fit && (!lut_fits || t_cores < t_lut) ? cores : lut;
    return cores_fit || lut_fits;
}

// Workspace of biq_gemm_noalloc: device memory that belongs to the library's code object, one
// copy per GPU, held until the process ends.  In host code the array's name is only a handle
// for hipGetSymbolAddress; the device address is looked up once per device and kept.
constexpr size_t kScratchBytes = (size_t)32 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
void* g_scratch_addr[kMaxDevices];  // device address of `scratch` on each device, 0 = not looked up yet

// Device address of the current device's copy of `scratch`.
hipError_t scratch_address(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    void* p = __atomic_load_n(&g_scratch_addr[dev], __ATOMIC_ACQUIRE);
    if (!p) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        __atomic_store_n(&g_scratch_addr[dev], p, __ATOMIC_RELEASE);  // racing first calls store the same value
    }
    *out = p;
    return hipSuccess;
}

}  // namespace

extern "C" {

const char* biq_status_str(biq_status status) {
    switch (status) {
        case BIQ_OK: return "ok";
        case BIQ_EINVAL: return "invalid argument";
        case BIQ_EUNSUPPORTED: return "unsupported request";
        case BIQ_EWORKSPACE: return "workspace too small";
        case BIQ_EHIP: return "HIP runtime error";
    }
    return "unknown status";
}

int biq_version(void) { return 100; }

size_t biq_key_row_stride(int n) { return n < 1 ? 0 : ((size_t)n + 127) / 128 * 16; }

size_t biq_packed_bytes(int m, int n, int q) {
    if (m < 1 || n < 1 || q < 1) return 0;
    return (size_t)q * m * biq_key_row_stride(n);
}

size_t biq_num_chunks(int n, int mu) {
    if (n < 1 || mu < 1 || mu > kMaxMu) return 0;
    return ((size_t)n + mu - 1) / mu;
}

size_t biq_lut_bytes(int n, int batch, int mu) {
    if (n < 1 || batch < 1 || mu < 1 || mu > kMaxMu) return 0;
    return biq_num_chunks(n, mu) * ((size_t)1 << mu) * batch * sizeof(float);
}

biq_status biq_plan_get(int m, int n, int q, int batch, int mu, biq_plan* plan) {
    if (!plan || !shape_ok(m, n, q, batch, mu)) return BIQ_EINVAL;
    return plan_default(*plan, m, n, q, batch, mu) ? BIQ_OK : BIQ_EUNSUPPORTED;
}

biq_status biq_plan_get_lut(int m, int n, int q, int batch, int mu, biq_plan* plan) {
    if (!plan || !shape_ok(m, n, q, batch, mu)) return BIQ_EINVAL;
    return plan_default(*plan, m, n, q, batch, mu, true) ? BIQ_OK : BIQ_EUNSUPPORTED;
}

biq_status biq_plan_get_mfma(int m, int n, int q, int batch, int mu, int input_terms, biq_plan* plan) {
    if (!plan || !shape_ok(m, n, q, batch, mu)) return BIQ_EINVAL;
    if (input_terms != 2 && input_terms != 3) return BIQ_EINVAL;
    if (q > 4) return BIQ_EUNSUPPORTED;
    return plan_unpack(*plan, m, n, q, batch, mu, input_terms) ? BIQ_OK : BIQ_EUNSUPPORTED;
}

biq_status biq_plan_check(int m, int n, int q, int batch, int mu, biq_plan* plan) {
    if (!plan || !shape_ok(m, n, q, batch, mu)) return BIQ_EINVAL;
    return plan_finish(*plan, m, n, q, batch, mu) ? BIQ_OK : BIQ_EINVAL;
}

size_t biq_plan_workspace_bytes(const biq_plan* plan, int m, int batch) {
    if (!plan || m < 1 || batch < 1) return 0;
    return plan_workspace(*plan, m, batch);
}

size_t biq_workspace_bytes(int m, int n, int q, int batch, int mu) {
    if (!shape_ok(m, n, q, batch, mu)) return 0;
    // the larger of what biq_gemm's and biq_query's default plans need
    biq_plan pl;
    if (!plan_default(pl, m, n, q, batch, mu, false)) return 0;
    const size_t a = plan_workspace(pl, m, batch);
    if (!plan_default(pl, m, n, q, batch, mu, true)) return 0;
    const size_t b = plan_workspace(pl, m, batch);
    return a > b ? a : b;
}

const char* biq_kernel_name(int kernel) {
    switch (kernel) {
        case KERNEL_GENERIC: return "query_generic";
        case KERNEL_GEMV8: return "gemv8";
        case KERNEL_GEMM8X2: return "gemm8x2";
        case KERNEL_UNPACK_MFMA: return "unpack_mfma";
        case KERNEL_GEMV8H: return "gemv8_half";
        case KERNEL_GEMM8X2H: return "gemm8x2_half";
        case KERNEL_WIDE: return "query_wide";
    }
    return "unknown";
}

biq_status biq_pack(const int8_t* B, uint8_t* K, int m, int n, int q, int mu, void* stream) {
    if (!shape_ok(m, n, q, 1, mu) || !B || !K) return BIQ_EINVAL;
    if (!aligned(K, 16)) return BIQ_EINVAL;
    const long long key_rows = (long long)q * m;
    const int stride_dw = (int)(biq_key_row_stride(n) / 4);
    const long long total = key_rows * stride_dw;
    if (total > (1ll << 38)) return BIQ_EUNSUPPORTED;
    const hipError_t e = launch_pack(B, reinterpret_cast<uint32_t*>(K), key_rows, n, stride_dw,
                                     reinterpret_cast<hipStream_t>(stream));
    return e == hipSuccess ? BIQ_OK : BIQ_EHIP;
}

biq_status biq_quantize(const float* W, uint8_t* K, float* alpha, int m, int n, int q, void* stream) {
    if (!shape_ok(m, n, q, 1, 8) || !W || !K || !alpha) return BIQ_EINVAL;
    if (!aligned(K, 16) || !aligned(W, 4) || !aligned(alpha, 4)) return BIQ_EINVAL;
    if (n > kQuantMaxN) return BIQ_EUNSUPPORTED;  // a row's residual is kept in the registers of one workgroup
    const int stride_dw = (int)(biq_key_row_stride(n) / 4);
    const hipError_t e = launch_quantize(W, reinterpret_cast<uint32_t*>(K), alpha, m, n, q, stride_dw,
                                         reinterpret_cast<hipStream_t>(stream));
    return e == hipSuccess ? BIQ_OK : BIQ_EHIP;
}

biq_status biq_unpack_keys(const uint8_t* K, uint8_t* keys, int m, int n, int q, int mu, void* stream) {
    return unpack_keys_any<uint8_t>(K, keys, m, n, q, mu, stream);
}

biq_status biq_unpack_keys16(const uint8_t* K, uint16_t* keys, int m, int n, int q, int mu, void* stream) {
    return unpack_keys_any<uint16_t>(K, keys, m, n, q, mu, stream);
}

biq_status biq_build_lut(const float* X, float* LUT, int n, int batch, int mu, void* stream) {
    if (!shape_ok(1, n, 1, batch, mu) || !X || !LUT) return BIQ_EINVAL;
    if (!aligned(X, 4) || !aligned(LUT, 4)) return BIQ_EINVAL;
    const hipError_t e = launch_build_lut(mu, X, LUT, n, batch, ceil_div(n, mu),
                                          reinterpret_cast<hipStream_t>(stream));
    return e == hipSuccess ? BIQ_OK : BIQ_EHIP;
}

biq_status biq_query(const uint8_t* K, const float* alpha, const float* LUT, float* Y, int m, int n,
                     int q, int batch, int mu, void* workspace, size_t workspace_bytes, void* stream) {
    return run_query(false, K, alpha, nullptr, LUT, Y, m, n, q, batch, mu, nullptr, workspace,
                     workspace_bytes, stream);
}

biq_status biq_gemm(const uint8_t* K, const float* alpha, const float* X, float* Y, int m, int n,
                    int q, int batch, int mu, void* workspace, size_t workspace_bytes, void* stream) {
    return run_query(true, K, alpha, X, nullptr, Y, m, n, q, batch, mu, nullptr, workspace,
                     workspace_bytes, stream);
}

biq_status biq_gemm_ex(const uint8_t* K, const float* alpha, const float* X, float* Y, int m, int n,
                       int q, int batch, int mu, const biq_plan* plan, void* workspace,
                       size_t workspace_bytes, void* stream) {
    if (!plan) return BIQ_EINVAL;
    return run_query(true, K, alpha, X, nullptr, Y, m, n, q, batch, mu, plan, workspace,
                     workspace_bytes, stream);
}

biq_status biq_init(void) {
    void* p = nullptr;
    return scratch_address(&p) == hipSuccess ? BIQ_OK : BIQ_EHIP;
}

size_t biq_noalloc_scratch_bytes(void) { return kScratchBytes; }

biq_status biq_gemm_noalloc(const uint8_t* K, const float* alpha, const float* X, float* Y, int m, int n,
                            int q, int batch, int mu, void* stream) {
    if (!shape_ok(m, n, q, batch, mu)) return BIQ_EINVAL;
    biq_plan pl;
    if (!plan_default(pl, m, n, q, batch, mu, false)) return BIQ_EUNSUPPORTED;
    size_t need = plan_workspace(pl, m, batch);
    if (need > kScratchBytes) {
        if ((!plan_small_workspace(pl, m, n, q, batch, mu) || plan_workspace(pl, m, batch) > kScratchBytes) &&
            !plan_fitting(pl, m, n, q, batch, mu, kScratchBytes))
            return BIQ_EWORKSPACE;                        // use biq_gemm with a workspace
        need = plan_workspace(pl, m, batch);
    }
    void* ws = nullptr;
    if (need > 0 && scratch_address(&ws) != hipSuccess) return BIQ_EHIP;
    // Every kernel writes the part of the workspace it later reads (split input, partial sums) in
    // full before reading it, so what an earlier call left there does not matter and nothing is
    // cleared.
    return run_query(true, K, alpha, X, nullptr, Y, m, n, q, batch, mu, &pl, ws, need, stream);
}

biq_status biq_gemm_grouped(const biq_problem* problems, int count, int mu, void* stream) {
    if (!problems || count < 1) return BIQ_EINVAL;
    for (int i = 0; i < count; ++i) {
        const biq_problem& pr = problems[i];
        if (!shape_ok(pr.m, pr.n, pr.q, pr.batch, mu)) return BIQ_EINVAL;
        if (!pr.K || !pr.alpha || !pr.X || !pr.Y) return BIQ_EINVAL;
        if (!aligned(pr.K, 16) || !aligned(pr.alpha, 4) || !aligned(pr.X, 4) || !aligned(pr.Y, 4)) return BIQ_EINVAL;
    }
    // every problem gets its share of the CUs; all are planned before anything is launched
    const int cus = count >= kNumCu ? 1 : kNumCu / count;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    // first pass (launch = false) only checks that every problem has a single-dispatch plan
    for (int pass = 0; pass < 2; ++pass) {
        int i = 0;
        while (i < count) {
            GroupParams g{};
            int kind = -1, q = 0, lds = 0, grid = 0;
            while (i < count && g.count < kGroupMax) {
                const biq_problem& pr = problems[i];
                biq_plan pl;
                int k = -1;
                if (!plan_grouped(pl, k, pr.m, pr.n, pr.q, pr.batch, mu, cus)) return BIQ_EUNSUPPORTED;
                if (g.count > 0 && (k != kind || pr.q != q)) break;  // next dispatch
                kind = k;
                q = pr.q;
                if (pl.lds_bytes > lds) lds = pl.lds_bytes;
                QueryParams& qp = g.p[g.count];
                fill_query_params(qp, pl, pr.K, pr.alpha, pr.X, nullptr, pr.Y, pr.m, pr.n, pr.q, pr.batch, mu);
                g.first_wg[g.count] = grid;
                grid += qp.tasks_per_xcd * kNumXcd;
                ++g.count;
                ++i;
            }
            g.first_wg[g.count] = grid;
            if (pass == 1 && launch_grouped(kind, q, g, grid, lds, s) != hipSuccess) return BIQ_EHIP;
        }
    }
    return BIQ_OK;
}

biq_status biq_lstm_cell(const uint8_t* K, const float* alpha, const float* bias, const float* X,
                         const float* C_prev, float* H_out, float* C_out, int hidden, int n, int q, int batch,
                         int mu, void* stream) {
    if (hidden < 1 || hidden > (1 << 28)) return BIQ_EINVAL;
    const int m = 4 * hidden;
    if (!shape_ok(m, n, q, batch, mu)) return BIQ_EINVAL;
    if (!K || !alpha || !bias || !X || !C_prev || !H_out || !C_out) return BIQ_EINVAL;
    if (!aligned(K, 16) || !aligned(alpha, 4) || !aligned(bias, 4) || !aligned(X, 4) || !aligned(C_prev, 4) ||
        !aligned(H_out, 4) || !aligned(C_out, 4))
        return BIQ_EINVAL;
    if (mu != 8 || q > 4) return BIQ_EUNSUPPORTED;
    const int C = ceil_div(n, 8);
    biq_plan pl{};
    pl.threads = 1024;
    pl.tiles_per_split = 1;
    pl.row_mode = 1;
    int units;  // hidden units per workgroup: one workgroup per CU if the units allow it
    if (batch == 1 && C <= kGemvHalfTileChunks) {
        pl.kernel = KERNEL_GEMV8H;
        pl.chunks_per_tile = kGemvHalfTileChunks;
        pl.batch_tile = 1;
        units = ceil_div(hidden, kNumCu);
    } else if (batch >= 2 && C <= kGemmHalfTileChunks) {
        pl.kernel = KERNEL_GEMM8X2H;
        pl.chunks_per_tile = kGemmHalfTileChunks;
        pl.batch_tile = 2;
        units = 2 * (int)ceil_div_ll((long long)hidden * ceil_div(batch, 2), 2ll * kNumCu);  // two per wave step
    } else {
        return BIQ_EUNSUPPORTED;  // rows wider than one half-table tile: biq_gemm, then the cell update by the caller
    }
    if (units < 1) units = 1;
    pl.rows_per_wg = 4 * units;
    if (!plan_finish(pl, m, n, q, batch, mu) || pl.chunk_splits != 1) return BIQ_EUNSUPPORTED;
    QueryParams qp{};
    fill_query_params(qp, pl, K, alpha, X, nullptr, H_out, m, n, q, batch, mu);
    // workgroups are laid out over hidden units, not gate rows
    qp.row_blocks = ceil_div(hidden, units);
    qp.ntasks = qp.row_blocks * qp.batch_tiles;
    qp.tasks_per_xcd = ceil_div(qp.ntasks, kNumXcd);
    qp.bias = bias;
    qp.c_prev = C_prev;
    qp.c_out = C_out;
    qp.hidden = hidden;
    const int grid = qp.tasks_per_xcd * kNumXcd;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const hipError_t e = pl.kernel == KERNEL_GEMV8H ? launch_lstm8h(q, qp, grid, pl.threads, pl.lds_bytes, s)
                                                    : launch_lstm8x2h(q, qp, grid, pl.threads, pl.lds_bytes, s);
    return e == hipSuccess ? BIQ_OK : BIQ_EHIP;
}

}  // extern "C"
