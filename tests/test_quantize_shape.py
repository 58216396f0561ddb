"""csrc/biq_quantize_shape.h, every row length: the instance that biq_quantize takes holds the row, exists, and masks every
piece that is not wholly inside it."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAIN = """
#include <cstdio>
#include "biq_quantize_shape.h"
int main() {
    for (int n = 1; n <= biq::kQuantMaxN; ++n) {
        const biq::QuantShape g = biq::quant_shape(n);
        std::printf("%d %d %d %d %d\\n", n, g.pieces, g.waves, g.tail, biq::quant_tail(g.pieces));
    }
}
"""


def test_every_row_length(tmp_path):
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "shapes")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-I" + os.path.join(ROOT, "paper_2005_09904_amd", "csrc"),
                    str(tmp_path / "main.cpp"), "-o", exe], check=True)
    rows = [tuple(map(int, line.split())) for line in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()]
    assert [r[0] for r in rows] == list(range(1, 32769))
    for n, pieces, waves, tail, instance_tail in rows:
        assert 256 * waves * pieces >= n and waves == (1 if n <= 8192 else 4)
        assert (1 if waves == 1 else 9) <= pieces <= 32 and (pieces <= 16 or pieces % 2 == 0), "no such instance"
        assert tail in (0, instance_tail)
        # the end of the last piece that is not masked, of the last wave
        assert 256 * waves * (pieces - tail) <= n, "n = %d: pieces past the row are not masked" % n
