// Which row of a wide pass a workgroup of the residual launch takes (plain C++: no HIP types).
#pragma once

namespace ssd {

// Workgroups go round-robin to the 8 dies (XCDs) by their index; large launches deal the rows to them in pieces of 8, piece q to die
// q mod 8.  The 16-byte operand pieces of 8 consecutive rows are one aligned 128-byte line, which then meets in one L2, and no die
// has more than one piece above another whatever the number of rows.  Which launches: see launch_wide_resid.
constexpr unsigned kRowPiece = 8, kRowDies = 8;
constexpr unsigned wide_resid_grid(unsigned rows) { return (rows + kRowDies * kRowPiece - 1) / (kRowDies * kRowPiece) * (kRowDies * kRowPiece); }
constexpr unsigned wide_resid_row(unsigned block) {
  const unsigned die = block % kRowDies, slot = block / kRowDies;
  return (slot / kRowPiece * kRowDies + die) * kRowPiece + slot % kRowPiece;
}

}  // namespace ssd
