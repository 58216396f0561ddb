"""csrc/biq_gather_rule.h: rows whose splits would crowd a few CUs give them workgroups of their own
(mu = 8) or are copied (any mu)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, body):
    (tmp_path / "main.cpp").write_text('#include <cstdio>\n#include "biq_gather_rule.h"\nusing namespace biq;\nint main() {\n%s\n}\n' % body)
    exe = str(tmp_path / "rule")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-I" + os.path.join(ROOT, "paper_2005_09904_amd", "csrc"),
                    str(tmp_path / "main.cpp"), "-o", exe], check=True)
    return [tuple(map(int, l.split())) for l in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()]


def test_splits_in_waves_or_apart(tmp_path):
    rows = _run(tmp_path, """
    for (int lanes = 4; lanes <= 8; lanes *= 2)
        for (int m = 1; m <= 20000; m = m * 3 / 2 + 1)
            for (int q = 1; q <= 4; ++q)
                for (int b = 2; b <= 300; b = b * 2 + (b == 2))
                    for (int s = 1; s <= 200; s = s * 5 / 4 + 1)
                        std::printf("%d %d %d %d %d %d\\n", lanes, m, q, b, s, gather_in_waves(lanes, m, q, b, s));""")
    seen = set()
    for lanes, m, q, b, s, waves in rows:
        share = 1 if b <= 4 else 2 if b <= 8 else 4
        groups = -(-m // (64 // (lanes * share))) * -(-(-(-b // 4)) // share)
        assert not (waves and (s == 1 or s > 64))
        if waves:
            # cache lines that a CU reads beyond its share of the whole: 10 thousand or so, a few us
            assert (-(-groups // 256) * s - -(-groups * s // 256)) * q * 1024 // share <= 10240
        if 1 < s <= 64 and groups % 256 == 0:
            assert waves                              # the chip is full either way: a dispatch less
        seen.add((lanes, share, waves))
    assert len(seen) == 12


def test_units_of_few_long_rows(tmp_path):
    rows = _run(tmp_path, """
    for (int lanes = 0; lanes <= 6; ++lanes)
        for (int m = 1; m <= 20000; m = m * 3 / 2 + 1)
            for (int b = 1; b <= 300; b = b * 2 + (b == 2))
                for (int s = 1; s <= 64; s = s * 5 / 4 + 1) {
                    const GatherUnits g = gather_units_shape(lanes, m, b, s);
                    std::printf("%d %d %d %d %d %d %lld %lld %d %d %d\\n", lanes, m, b, s, g.log_slices, g.log_splits, g.blocks, g.slice_blocks,
                                gather_units_crowd(g, b, s, 1, 2, 32, 16000), gather_units_crowd(g, b, s, 1, 2, 32, 4000000),
                                gather_units_crowd(g, b, s, 1, 2, 32, 4000001));
                }""")
    for lanes, m, b, s, slices, splits, blocks, slice_blocks, crowd_l1, crowd_l2, crowd_beyond in rows:
        row = lanes + slices + splits
        assert row <= 6 and (1 << splits) <= s
        assert blocks * (64 >> row) >= m > (blocks - 1) * (64 >> row)
        assert slice_blocks << slices >= -(-b // 4) > (slice_blocks - 1) << slices
        # LDS: the sums of every split, 16 bytes each
        assert s * (64 >> (lanes + splits)) * 16 <= 65536
        groups = blocks * slice_blocks
        lines = -(-groups // 256) * -(-s // (1 << splits)) * 2 * 32 * 64 >> slices
        idle = groups < 256 or b == 1
        assert crowd_l1 == (idle and lines > (98304 if b == 1 else 40960)) and crowd_beyond == (idle and lines > 16384)
        assert crowd_l2 == (idle and lines > (32768 if b == 1 else 40960))
