// The mapping of the direct kernel (biq_direct.h) for a shape and its estimated time (plain C++: no kernel code).
#pragma once

#include <initializer_list>

namespace biq {

constexpr int kDirectThreads = 512;
constexpr int kDirectWaves = kDirectThreads / 64;
constexpr int kDirectDigits = 5;                  // of an input element
constexpr int kDirectCus = 256;
constexpr int kDirectLds = 160 * 1024;            // of a CU, the most a workgroup can ask for
constexpr int kDirectMaxVec = 15;                 // vectors of a workgroup: five column tiles
// The mappings: one row tile per wave and one chunk at a time (few rows); one row tile and two chunks requested
// together, 128 bytes per row: a whole line (lines); more row tiles per wave, which share a step's operands in LDS, and
// two chunks where the registers hold them beside RT x NT accumulators (many rows).
enum DirectKind { DIRECT_FEW, DIRECT_MANY, DIRECT_LINES };
constexpr int direct_rpw(int q, int nt) { return q == 1 ? (nt <= 2 ? 4 : 2) : q == 2 && nt <= 3 ? 2 : 1; }
constexpr int direct_uc(int nt) { return nt <= 2 ? 2 : 1; }
constexpr bool direct_has_kind(int kind, int q, int nt) {
    return kind == DIRECT_FEW || (kind == DIRECT_MANY ? direct_rpw(q, nt) > 1
                                                      : nt == 1 || (direct_rpw(q, nt) == 1 && direct_uc(nt) == 2));
}

// quotients rounded up (a >= 0, b >= 1)
inline int direct_div(int a, int b) { return (int)(((unsigned)a + (unsigned)b - 1u) / (unsigned)b); }
inline long long direct_div_ll(long long a, long long b) { return (a + b - 1) / b; }
inline unsigned direct_row_bytes(int n) { return (unsigned)direct_div(n, 128) * 16u; }   // keys of a row

// cbrt(a^3 + b^3) for a, b > 0, to 1.2e-5: of two costs that overlap, the larger one and some of the other.  (Polynomial for
// (1 + u)^(1/3) on [0, 1]; plans are made on every call, and the library's root takes 37 ns.)
inline double together(double a, double b) {
    const double most = a > b ? a : b, r = (a > b ? b : a) / most, u = r * r * r;
    return most * (1.0 + u * (0.3329064 + u * (-0.10635862 + u * (0.04417861 - 0.01081733 * u))));
}

inline long long direct_lds_bytes(long long chunks, int vecs, int rpw, bool exchange) {
    const long long blocks = chunks * 16;
    // digits, scale bytes, partial results of the waves (two buffers)
    return (blocks * kDirectDigits * 24 + 8) * vecs + blocks * vecs +
           (exchange ? 2 * kDirectWaves * rpw * ((vecs + 2) / 3) * 3 * 16 * 4 : 0);
}

// Mapping of the direct kernel (biq_direct.h) for a shape, with its estimated time (us); false if its
// operands do not fit the LDS.  Candidates: the many-rows instantiation, and one row tile per wave with 1 .. 8
// groups of waves along the row; as many row steps per workgroup as leave at most 256 workgroups.  A row step costs
// its chunks (matrix pipe, expansion or LDS of the two waves per SIMD, or the latency of the next keys) and an
// epilogue; keys stream at 3.5 TB/s, results and scales count 2.25 times; the split of the inputs 2.2 us per round of 512
// blocks over the eight waves, half of it in a last round of up to four waves (one per SIMD), a quarter for one.  Fitted to
// 3700 shapes of 2 .. 256 vectors (128 .. 32768 rows, 128 .. 16384 columns, every mapping of each, a replayed graph, keys
// from memory): 8 % rms where tables or digits are within a factor of two (without the last rounds, results and scales 12 %),
// the mapping chosen 0.9 % slower in the mean than the best.  One vector on more than 2048 columns has costs of its own,
// fitted to 2300 times of 298 shapes: 7 % rms, but 7 to 12 % below what a replayed graph takes with keys from memory; the mapping
// chosen is 0.2 % slower in the mean than the best.  The estimate handed on (not the choice of the mapping) has at least
// 0.81 us per row step where there are several: a step waits for its scales, and short rows have nothing else to do
// meanwhile (1025348 x 111, 1 plane, 1 vector: 16 us without, measured 34).
struct DirectGeom {
    int vecs, batch_tiles, chunks, ksplit, steps, row_blocks, lds;
    int uc;                  // chunks requested together
    int kind;                // DirectKind
    double est;
};
// Input vectors of one workgroup whose digits fit the LDS beside the exchange buffers.
inline int direct_max_vectors(int n) {
    const long long spare = kDirectLds - 2 * kDirectWaves * 15 * 16 * 4;
    const long long v = spare / direct_lds_bytes(direct_div(n, 512), 1, 1, false);
    return (int)(v < kDirectMaxVec ? v : kDirectMaxVec);
}
inline bool direct_geometry(DirectGeom& g, int m, int n, int q, int batch) {
    if (q > 4 || direct_row_bytes(n) > (1u << 26)) return false;
    if (m > (1 << 30)) return false;                 // rows past the end of the last workgroup's steps stay in 32 bits
    const int vmax = direct_max_vectors(n);
    if (vmax == 0) return false;
    g.chunks = direct_div(n, 512);
    g.batch_tiles = direct_div(batch, vmax);
    g.vecs = direct_div(batch, g.batch_tiles);
    g.batch_tiles = direct_div(batch, g.vecs);
    if (g.batch_tiles > 65535) return false;
    const int nt = direct_div(g.vecs, 3);
    // groups of 16 blocks of inputs, four to a wave at a time
    const int groups = g.chunks * g.vecs, last = groups % (4 * kDirectWaves);
    const double split_rounds = groups / (4 * kDirectWaves) + (last == 0 ? 0.0 : last <= 4 ? 0.25 : last <= 16 ? 0.47 : 1.0);
    double best = 1e30, least_work = 0.0, best_mem = 0.0;
    // (plans are made on every call: quotients by powers of two are shifts)
    for (int kind : {DIRECT_MANY, DIRECT_LINES, DIRECT_FEW}) {
        if (!direct_has_kind(kind, q, nt)) continue;
        const int rpw = kind == DIRECT_MANY ? direct_rpw(q, nt) : 1, uc = kind == DIRECT_FEW ? 1 : direct_uc(nt);
        // one vector on wide rows: costs of their own, and beyond 256 row tiles several groups of waves along whole lines,
        // too (332 shapes: up to there those take 1.01 to 1.2 times as long, 0.97 with four row steps and 0.84 with five
        // and more; with 2 to 6 vectors, 110 shapes, 1 % less at most)
        const bool one = batch == 1 && n > 2048 && kind != DIRECT_MANY;
        if (kind == DIRECT_LINES && (one ? m <= 16 * kDirectCus : direct_rpw(q, nt) > 1)) continue;
        const double keys = (double)q * m * direct_row_bytes(n) * g.batch_tiles;
        const double mem = one ? keys * (uc == 2 ? 1 / 4.35e6 : 1 / 3.72e6) : (keys + 9.0 * m * ((double)q * g.batch_tiles + batch)) * (1 / 3.5e6);
        const int units = uc == 2 ? (g.chunks + 1) >> 1 : g.chunks;
        const int rt = q * rpw;
        double clk, before;                              // a chunk; what comes ahead of the first row step
        if (one) {
            clk = 727.0 * q;
            const double least = uc == 2 ? 818.0 : 1132.0;
            if (clk < least) clk = least;
            before = 2.54 + 1.87 / (4 * kDirectWaves) * g.chunks;
        } else {
            clk = 17.5 * rt * (16 * nt > 32 ? 16 * nt : 32);
            if (clk < 680.0 * nt) clk = 680.0 * nt;
            if (clk < 850.0) clk = 850.0;
            before = 2.9 + 0.085 * (nt - 1);
        }
        const double unit = uc * clk * (1 / 2200.0);
        const int log_step_rows = 7 + (rpw >> 1);        // rows of a row step of the eight waves: rpw is 1, 2 or 4
        for (int log_ks = 0; log_ks <= (kind == DIRECT_FEW || (one && uc == 2) ? 3 : 0) && ((1 << log_ks) - 1) * uc < g.chunks; ++log_ks) {
            const int log_rows = log_step_rows - log_ks;
            const long long all_steps = ((long long)m + (1 << log_rows) - 1) >> log_rows;
            long long steps = direct_div_ll(all_steps * g.batch_tiles, kDirectCus);
            if (steps > all_steps) steps = all_steps;
            const long long blocks = steps == 1 ? all_steps : direct_div_ll(all_steps, steps);
            const double turns = (double)direct_div_ll(blocks * g.batch_tiles, kDirectCus);     // rounds of workgroups
            const int upg = (units + (1 << log_ks) - 1) >> log_ks;
            const double row_step = one ? (log_ks > 0 ? 0.57 : 0.53) : 0.008 * rt * nt + (log_ks > 0 ? 0.17 : 0.0);
            const double ahead = one ? before : before + 2.2 * turns * split_rounds;
            const double work = turns * steps * (upg * unit + row_step);
            // (both together: of two mappings that memory bounds, the one with less work)
            const double t = ahead + together(work, mem);
            if (t < best) {
                best = t;
                g.est = steps > 1 && work < 0.81 * turns * steps ? -ahead : t;
                g.kind = kind;
                g.ksplit = 1 << log_ks;
                g.uc = uc;
                g.steps = (int)steps;
                g.row_blocks = (int)blocks;
                least_work = 0.81 * turns * steps;
                best_mem = mem;
            }
        }
    }
    if (g.est < 0.0) g.est = together(least_work, best_mem) - g.est;
    g.lds = (int)direct_lds_bytes(g.chunks, g.vecs, 1, g.ksplit > 1);
    return best < 1e30;
}

}  // namespace biq
