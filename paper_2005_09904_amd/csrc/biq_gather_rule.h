// How lookups that read the tables in place (biq_gather.h) are spread over the chip (plain C++: no kernel code).
#pragma once

namespace biq {

constexpr int kGatherVec = 4;      // input vectors of a lane's read
constexpr int kGatherWaves = 8;    // most waves of a workgroup
// Most splits of a row that a workgroup adds.  Their sums lie in LDS, 16 bytes for each of up to 64 rows and slices: with one
// lane per row 64 KiB, the most that a launch gets without asking for more.
constexpr int kGatherSplits = 64;
static_assert(kGatherSplits * 64 * kGatherVec * 4 <= 65536, "LDS of a workgroup");
constexpr int kGatherCus = 256;

// The slices of up to four vectors an entry is read in, of one lane each: 1, 2 or 4 of them (2^log_slices) on
// neighbouring lanes, which then share the entry's cache lines (a wave's reads cost the address unit a line each:
// 1024 x 1024, 2 planes, 8 vectors 3.8 -> 3.1 us on the GPU; 3317 x 480, 2, 15 9.3 -> 4.8), the rest in the grid's y.
constexpr int gather_log_slices(int batch) { return batch > 2 * kGatherVec ? 2 : batch > kGatherVec ? 1 : 0; }

// mu = 8: the splits of a row in the waves of one workgroup, which adds them, or in workgroups of their own and added by
// reduce_splits_kernel.  The former saves a dispatch (1-2 us) and costs what a CU then reads more than its share of the
// whole, counted in cache lines (1024 per split and plane, fewer where slices share them), 0.5-1.3 ns each.  Waves / own
// workgroups, us: 64 x 4096, 2 planes, 8 vectors (3072 lines) 4.1 / 4.7; 1024 x 4096, 2, 4 (4096) 7.2 / 8.2; 185 x 5795, 2, 8
// (4096, 6 splits) 8.2 / 6.7; 128 x 5120, 2, 4 (8192) 6.6 / 5.2; 64 x 16384, 2, 8 (15360) 22.0 / 9.0; 16 x 65536, 2, 4 (129024) 148 / 21.
// With more than 8 vectors the waves of a CU meet in the lines of the same entries; then, with one plane or a third
// of the chip busy, they are the better up to more: 277 x 15360, 3, 12 (4608) 27.0 / 34.2; 236 x 30720, 2, 16 (8192) 30 / 38;
// 58 x 51548, 1, 32 (9984) 22.5 / 30.6; but 60 x 6144, 4, 16 (5120) 9.0 / 6.7; 22 x 10240, 4, 16 (9216) 12.3 / 7.3.
// row_lanes: lanes that share a row.
constexpr bool gather_in_waves(int row_lanes, int m, int q, int batch, int splits) {
    if (splits == 1 || splits > kGatherSplits) return false;
    const int log_slices = gather_log_slices(batch);
    const long long rows = 64 / (row_lanes << log_slices), slices = (batch + kGatherVec - 1) / kGatherVec;
    const long long groups = ((m + rows - 1) / rows) * ((slices + (1 << log_slices) - 1) >> log_slices);
    const long long together = (groups + kGatherCus - 1) / kGatherCus * splits;
    const long long apart = (groups * splits + kGatherCus - 1) / kGatherCus;
    const long long lines = ((together - apart) * q * 1024) >> log_slices;
    return lines <= (log_slices == 2 && (q == 1 || groups >= 80) ? 10240 : splits <= 4 ? 4096 : 3584);
}

// Any mu: how gather_units_kernel lays out a call.  2^log_splits splits of a row sit side by side in a wave where rows are
// few (more workgroups: 187 x 2894, 4 planes, 15 vectors at mu = 7, where a row of a tile is one lane, 19.4 -> 7.2 us, copied 26.5).
struct GatherUnits { int log_slices, log_splits; long long blocks, slice_blocks; };
constexpr GatherUnits gather_units_shape(int log_lanes, int m, int batch, int splits) {
    GatherUnits g{gather_log_slices(batch), 0, 0, 0};
    if (g.log_slices + log_lanes > 6) g.log_slices = 6 - log_lanes;
    const long long slices = (batch + kGatherVec - 1) / kGatherVec;
    g.slice_blocks = (slices + (1 << g.log_slices) - 1) >> g.log_slices;
    while (log_lanes + g.log_slices + g.log_splits < 6 && (2 << g.log_splits) <= splits &&
           m * g.slice_blocks < (kGatherCus * 64ll) >> (log_lanes + g.log_slices + g.log_splits))
        ++g.log_splits;
    const int rows = 64 >> (log_lanes + g.log_slices + g.log_splits);
    g.blocks = ((long long)m + rows - 1) / rows;
    return g;
}

// Where reading in place takes longer than copying the tables to LDS (15-25 us): the splits of a row share the waves of a workgroup, so
// that few long rows leave most of the chip idle.  Counted in cache lines that a CU reads one after the other (keys_per_lane: of one
// tile and plane), a line costs 0.3-0.45 ns as long as the tables fit the 4 MB of an XCD's L2, 1.1-1.3 ns beyond.  Several vectors,
// copied / in place, us: 655 x 6055, 4 planes, 2 vectors, mu = 4 (32768 lines) 22 / 14; 4 x 37436, 2, 7, 2 (40960) 24 / 17;
// 26 x 79841, 2, 4, 3 (53248) 26 / 30; 13 x 66339, 4, 5, 3 (90112) 26 / 43; tables beyond the L2: 4 x 53398, 1, 3, 5 (12288) 19 / 8; 77 x
// 119417, 1, 3, 6 (20480) 28 / 32; 4 x 100000, 2, 4, 6 (34816) 22 / 41; 10 x 124685, 4, 5, 5 (102400) 24 / 138.  A full chip hides those
// reads, while its copies cost up to 50 us (2674 x 11220, 2, 4, 7 (57344) 48 / 40), but for one vector copies stay at 15-25 us, more where
// rows are many and have one plane: 7 x 46503, 2, 1, 3 (32768) 15 / 11; 587 x 13830, 5, 1, 8 (40960) 18 / 26; 1898 x 20280, 3, 1, 7
// (73728) 32 / 50; 2200 x 10761, 5, 1, 7 (143360) 19 / 48; 14328 x 4164, 1, 1, 7 (43008) 35 / 18.  Tables in a CU's own cache cost 0.1-0.2 ns a
// line: 2528 x 995, 5, 1, 1 (81920) 37 / 19; 11743 x 1463, 2, 1, 2 (98304) 21 / 25; 5389 x 1446, 5, 1, 2 (122880) 25 / 30.
constexpr bool gather_units_crowd(const GatherUnits& g, int batch, int splits, int tiles_per_split, int q, int keys_per_lane,
                                  long long table_bytes) {
    const long long groups = g.blocks * g.slice_blocks;
    if (groups >= kGatherCus && batch > 1) return false;
    const long long turns = (splits + (1 << g.log_splits) - 1) >> g.log_splits;
    const long long lines = ((groups + kGatherCus - 1) / kGatherCus * turns * tiles_per_split * q * keys_per_lane * 64) >> g.log_slices;
    if (table_bytes > 4000000) return lines > 16384;
    if (batch > 1) return lines > 40960;
    return lines > (table_bytes <= 16000 ? 98304 : q == 1 ? 49152 : 32768);
}

}  // namespace biq
