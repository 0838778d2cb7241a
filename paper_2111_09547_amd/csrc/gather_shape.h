// How the waves of the fused layer over neighbour lists (gather_kernel.h) divide a tile of 16 rows, and where a
// lane's part of its own row lies.  Compiled for the host as well.
#pragma once
#include <stdint.h>

namespace qgtc {

// The dimensions of an instance; PARTS = 2: codes of 9 to 16 bits, a low and a high byte each.
template <int LP, int WPT, int PARTS>
struct GatherShape {
  static constexpr int P = 1 << LP;
  static constexpr int PS = P < 16 ? P : 16;         // pieces of a unit: 16 slots
  static constexpr int RC = 16 / PS, HV = P / PS;    // rows of a unit; P > 16: parts of 256 columns
  static constexpr int UNITS = 16 / WPT / RC;        // units of a wave per part
  static constexpr int LR = LP < 4 ? LP : 4;         // lane ln has row ln >> LR of a unit, piece ln % PS
  static constexpr int W = UNITS * PARTS < 4 ? UNITS * PARTS : 4;   // sums at a time: parts of units
};

// The own row of lane (ln, g) of a unit, four columns, as the lane's and the unit's (scalar) offset of a buffer load
// on the rows of a tile that exist, `size` bytes.  The load compares the lane's offset with size - scalar offset, so
// that the scalar offset of a unit behind the last row is held to size: the difference must not wrap.
template <class Shape>
constexpr uint32_t own_lane_offset(int ln, int g, uint32_t ldx) {
  return (uint32_t)(ln >> Shape::LR) * ldx + 16u * (uint32_t)(ln & (Shape::PS - 1)) + 4u * (uint32_t)g;
}
constexpr uint32_t own_unit_offset(uint32_t row, uint32_t byte, uint32_t ldx, uint32_t size) {
  return row * ldx + byte < size ? row * ldx + byte : size;
}

}  // namespace qgtc
