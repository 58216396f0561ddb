// Which instance of quantize_wave_kernel holds a row of n elements (plain C++: no kernel code).
#pragma once

namespace biq {

constexpr int kQuantMaxN = 32768;
constexpr int kQuantWaveN = 8192;     // longest row of one wave

// The pieces of a wave that are masked where the instance is not filled: instances of more than 16 pieces exist for even
// numbers of them only, so that their last two may be partial or lie past the row.
constexpr int quant_tail(int pieces) { return pieces > 16 ? 2 : 1; }

// `waves` waves with `pieces` pieces of 256 elements each; the last `tail` pieces of a wave are masked (0: the row
// fills all of them).  Whether it does is asked of the instance's pieces, not of the row's: a row of 17 whole pieces runs in the instance
// of 18, whose last one lies past the row.
struct QuantShape { int pieces, waves, tail; };
constexpr QuantShape quant_shape(int n) {
    const int waves = n <= kQuantWaveN ? 1 : 4;
    const int needed = ((n + 255) / 256 + waves - 1) / waves;
    const int pieces = needed > 16 ? (needed + 1) / 2 * 2 : needed;
    return {pieces, waves, n == 256 * waves * pieces ? 0 : quant_tail(pieces)};
}

}  // namespace biq
