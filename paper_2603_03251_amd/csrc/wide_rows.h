// Which row of a wide pass a workgroup of the residual launch takes (plain C++: no HIP types).
#pragma once

namespace ssd {

// Workgroups go round-robin to the 8 dies (XCDs) by their index; rows go to them in pieces of 8, piece q to die q mod 8.  The
// 16-byte operand pieces of 8 consecutive rows are one aligned 128-byte line, which then meets in one L2, and no die has more than
// one piece above another whatever the number of rows.  Measured against single rows dealt round-robin, which send every line to
// memory in eight parts, and against an eighth of the rows, rounded up to whole 16-row tiles, per die, which leaves dies idle
// for most numbers of rows: see wide_resid_kernel.
constexpr int kRowPiece = 8;
constexpr int kRowDies = 8;
constexpr int wide_resid_grid(int rows) { return (rows + kRowDies * kRowPiece - 1) / (kRowDies * kRowPiece) * (kRowDies * kRowPiece); }
constexpr int wide_resid_row(int block) {
  const int die = block % kRowDies, slot = block / kRowDies;
  return (slot / kRowPiece * kRowDies + die) * kRowPiece + slot % kRowPiece;
}

}  // namespace ssd
