// How lookups that read the tables in place (biq_gather.h) are spread over the chip (plain C++: no kernel code).
#pragma once

namespace biq {

constexpr int kGatherVec = 4;      // input vectors of a lane's read
constexpr int kGatherWaves = 8;    // most waves of a workgroup
constexpr int kGatherSplits = 64;  // most splits of a row (32 KiB of LDS with 8 lanes per row)
constexpr int kGatherCus = 256;

// The slices of up to four vectors an entry is read in, of one lane each: 1, 2 or 4 of them (2^log_slices) on
// neighbouring lanes, which then share the entry's cache lines (a wave's reads cost the address unit a line each:
// 1024 x 1024, 2 planes, 8 vectors 3.8 -> 3.1 us on the GPU; 3317 x 480, 2, 15 9.3 -> 5.6), the rest in the grid's y.
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

}  // namespace biq
