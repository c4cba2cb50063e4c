// Where the copies of the products that walk their tiles (k_gemm_dma64_rounds) read: plain arithmetic, so that a program on the host can
// walk all of them.
#pragma once
#include <cstdint>

namespace faar {

// Copy u of a slice (64 lanes, 16 bytes each) fills LDS rows 8 u .. 8 u + 7 of the stacked [BM rows of A; rows of B]: lane / 8 -> row,
// lane % 8 -> slot.  LDS row p of a group of WN rows of B holds row TN * (p % 16) + p / 16 % TN of the group.
template <int BM, int WN, int TN>
struct RoundsCopy {
  static_assert(WN == 16 * TN && BM % 8 == 0, "a group of B's rows is one wavefront's columns");
  // row of the operand's tile
  static constexpr uint32_t row(int u, int lane) {
    const int ub = u - BM / 8;
    return static_cast<uint32_t>(u < BM / 8 ? 8 * u + lane / 8
                                            : TN * (8 * (ub & 1) + lane / 8) + ub % (WN / 8) / 2 + WN * (ub / (WN / 8)));
  }
  // 16-byte chunk of the slice: slot ^ (LDS row / 2) % 8
  static constexpr uint32_t chunk(int u, int lane) { return static_cast<uint32_t>((lane % 8) ^ (lane / 16) ^ (4 * (u & 1))); }
  // Byte offset from the tile's first row, to which 128 bytes a slice are added.  Rows that the matrix does not have are the last one that
  // it has: their products are not stored.  rows_left: rows from the tile's first to the end of the matrix, at least 1.
  static constexpr uint32_t offset(int u, int lane, uint32_t rows_left, uint32_t row_bytes) {
    const uint32_t r = row(u, lane);
    return (r < rows_left ? r : rows_left - 1) * row_bytes + chunk(u, lane) * 16;
  }
};

}  // namespace faar
