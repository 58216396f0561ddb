"""csrc/biq_direct_rule.h: which mapping of the direct kernel a shape gets."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

FEW, MANY, LINES = 0, 1, 2
# One vector on rows of more than 2048 columns: m, n, q, and the mapping it is here for - kind, groups of waves along the row,
# whether a workgroup has several row steps (for each of these mappings one shape whose last workgroup has fewer).
WIDE_ROWS = [
    # whole lines of keys, every number of planes with every number of groups there is, one row step and several
    (16513, 2590, 1, LINES, 1, False), (8399, 2083, 1, LINES, 2, False), (4222, 3086, 1, LINES, 4, False),
    (33076, 2092, 1, LINES, 1, True), (32905, 3081, 1, LINES, 2, True), (16437, 7188, 1, LINES, 4, True), (8427, 15021, 1, LINES, 8, True),
    (8263, 14441, 1, LINES, 8, True),
    (16585, 2604, 2, LINES, 1, False), (8375, 3107, 2, LINES, 2, False), (4193, 3772, 2, LINES, 4, False),
    (49225, 2561, 2, LINES, 1, True), (40982, 3118, 2, LINES, 2, True), (16424, 3718, 2, LINES, 4, True), (8290, 7253, 2, LINES, 8, True), (8221, 7193, 2, LINES, 8, True),
    (16771, 2576, 3, LINES, 1, False), (13875, 9442, 3, LINES, 2, False), (7081, 3239, 3, LINES, 4, False),
    (57196, 2187, 3, LINES, 1, True), (41791, 3087, 3, LINES, 2, True), (16535, 3073, 3, LINES, 4, True), (8260, 7196, 3, LINES, 8, True),
    (16603, 2567, 4, LINES, 1, False), (11394, 3767, 4, LINES, 2, False), (6054, 7607, 4, LINES, 4, False),
    (16429, 3113, 4, LINES, 4, True), (8262, 7243, 4, LINES, 8, True),
    # one chunk at a time: more than 256 row tiles all the same, and fewer
    (16763, 2153, 3, FEW, 1, False), (8677, 2591, 4, FEW, 2, False), (4097, 2049, 3, FEW, 4, False),
    (4096, 2049, 1, FEW, 4, False), (4081, 4096, 2, FEW, 8, False), (257, 5951, 3, FEW, 8, False), (128, 2052, 4, FEW, 4, False)]


@pytest.fixture(scope="module")
def mapping(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("rule")
    (tmp / "main.cpp").write_text("""
#include <cstdio>
#include "biq_direct_rule.h"
int main() {
    int m, n, q, b;
    while (std::scanf("%d %d %d %d", &m, &n, &q, &b) == 4) {
        biq::DirectGeom g{};
        const bool ok = biq::direct_geometry(g, m, n, q, b);
        std::printf("%d %d %d %d %d %d %d %d %d\\n", ok, g.kind, g.ksplit, g.uc, g.steps, g.row_blocks, g.vecs, g.batch_tiles, g.lds);
    }
}
""")
    exe = str(tmp / "rule")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2005_09904_amd", "csrc"),
                    str(tmp / "main.cpp"), "-o", exe], check=True)

    def run(shapes):
        out = subprocess.run([exe], input="".join("%d %d %d %d\n" % s for s in shapes), check=True, capture_output=True, text=True).stdout
        return [tuple(map(int, l.split())) for l in out.splitlines()]

    return run


def test_wide_rows_reach_their_mappings(mapping):
    """The shapes of the GPU test run the instances they are listed for, whatever the estimates become."""
    several_mappings, uneven = set(), set()
    for (m, n, q, kind, groups, several), (ok, k, ks, uc, steps, blocks, _, _, _) in zip(WIDE_ROWS, mapping([(m, n, q, 1) for m, n, q, *_ in WIDE_ROWS])):
        assert (ok, k, ks, steps > 1) == (1, kind, groups, several), (m, n, q, k, ks, steps)
        assert uc == (2 if kind == LINES else 1)
        step_rows = 8 // groups * 16
        last = -(-(m - (blocks - 1) * steps * step_rows) // step_rows)       # row steps of the last workgroup
        if several:
            several_mappings.add((q, kind, groups))
            uneven |= {(q, kind, groups)} if 1 <= last < steps and m % 16 else set()
    assert several_mappings == uneven
    assert {(q, ks) for _, _, q, kind, ks, several in WIDE_ROWS if kind == LINES} == {(q, ks) for q in (1, 2, 3, 4) for ks in (1, 2, 4, 8)}


def test_every_row_has_a_place(mapping):
    shapes = [(m, n, q, b) for m in (1, 127, 128, 4096, 4097, 50000, 1 << 30) for n in (1, 512, 2048, 2049, 9000, 38000)
              for q in (1, 2, 3, 4) for b in (1, 2, 3, 7, 15, 16, 200)]
    for (m, n, q, b), (ok, kind, ks, uc, steps, blocks, vecs, tiles, lds) in zip(shapes, mapping(shapes)):
        assert ok and lds <= 160 * 1024 and vecs <= 15 and vecs * tiles >= b > vecs * (tiles - 1)
        rpw = 1 if kind != MANY else {1: 4 if vecs <= 6 else 2, 2: 2}[q]
        rows = steps * (8 // ks) * rpw * 16
        assert rows * blocks >= m > rows * (blocks - 1)
        assert (ks - 1) * uc < -(-n // 512)                                   # every group has a chunk


def test_together(tmp_path):
    """Costs of very different and of equal sizes, against the root itself."""
    (tmp_path / "main.cpp").write_text("""
#include <cmath>
#include <cstdio>
#include "biq_direct_rule.h"
int main() {
    double worst = 0.0;
    for (double a = 1e-3; a < 1e9; a *= 1.37)
        for (double b = 1e-3; b < 1e9; b *= 1.73) worst = std::fmax(worst, std::fabs(biq::together(a, b) / std::cbrt(a * a * a + b * b * b) - 1.0));
    std::printf("%g\\n", worst);
}
""")
    exe = str(tmp_path / "together")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-I" + os.path.join(ROOT, "paper_2005_09904_amd", "csrc"),
                    str(tmp_path / "main.cpp"), "-o", exe], check=True)
    assert float(subprocess.run([exe], check=True, capture_output=True, text=True).stdout) < 1.3e-5
