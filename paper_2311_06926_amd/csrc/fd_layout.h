// Layout of the fast-diagonalisation kernels' LDS planes (fd.hip), in plain
// constexpr functions so that the host can check them against the reads.
#pragma once

#include <type_traits>

namespace hp {

// Row of the contraction tile that value i of lane group lk holds (the row map
// of the 16x16x4 MFMA results; it differs between FP64 and FP32, measured).
template <typename T>
constexpr int mfma_row(int lk, int i) {
    return std::is_same<T, double>::value ? lk + 4 * i : 4 * lk + i;
}

// MFMA steps of a 16-wide tile that holds `rem` contraction values: 0, 1, 2 or
// 4, what the kernels compile.
template <typename T>
constexpr int mfma_steps(int rem) {
    if (rem <= 0) return 0;
    if (std::is_same<T, double>::value) return rem > 8 ? 4 : (rem > 4 ? 2 : 1);
    return rem > 2 ? 4 : rem;
}

// Columns that the products read of a half of h values: its full tiles and the
// steps of its last one (FP32, where every step spreads over the tile, and
// split BF16 the whole tile).
template <typename T>
constexpr int half_width(int h) {
    const int full = h / 16 * 16, st = mfma_steps<T>(h - full);
    return full + (std::is_same<T, double>::value ? 4 * st : (st ? 16 : 0));
}

// Pitch of the folded plane in LDS: a row holds [even | odd] of n values and is
// read to the end of either half's last MFMA step, all of which the staging
// fills (zeros past the odd half); odd, so that the 16 rows of an operand fall
// in different banks.
template <typename T>
constexpr int plane_pitch(int n) {
    const int he = (n + 1) / 2, ho = n / 2;
    const int a = half_width<T>(he), b = he + half_width<T>(ho);
    return (a > b ? a : b) | 1;
}

}  // namespace hp
