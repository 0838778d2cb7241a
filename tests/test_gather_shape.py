"""Where the fused layer over neighbour lists reads its own rows (csrc/gather_shape.h), compiled with the host
compiler: a load that the unit's rule lets through stays inside the rows that exist."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2111_09547_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "gather_shape.h"
using namespace qgtc;
static long loads = 0, outside = 0, missed = 0;

template <int LP, int WPT, int PARTS>
void tile(uint32_t pieces, uint32_t rows) {
  using Sh = GatherShape<LP, WPT, PARTS>;
  const uint32_t part = 16u * pieces, ldx = part * PARTS, size = rows * ldx;
  for (int wave = 0; wave < WPT; ++wave)
    for (int hv = 0; hv < Sh::HV; ++hv)
      for (int unit = 0; unit < Sh::UNITS; ++unit)
        for (int which = 0; which < PARTS; ++which)
          for (int lane = 0; lane < 64; ++lane) {
            const int ln = lane & 15, g = lane >> 4;
            const uint32_t unit_row = (uint32_t)(wave * (16 / WPT) + unit * Sh::RC), byte = hv * 256u + which * part;
            const uint32_t voff = own_lane_offset<Sh>(ln, g, ldx), soff = own_unit_offset(unit_row, byte, ldx, size);
            // the load's rule: nothing is read where the lane's offset is size - scalar offset or more
            const bool read = voff < size - soff;
            ++loads;
            if (read && (uint64_t)voff + soff + 4 > size) ++outside;
            const uint32_t row = unit_row + (ln >> Sh::LR), col = 16u * ((ln & (Sh::PS - 1)) + 16 * hv) + 4u * g;
            if (row < rows && col < part && !(read && voff + soff == row * ldx + which * part + col)) ++missed;
          }
}
template <int LP>
void pieces_of() {
  for (uint32_t pieces = LP ? (1u << (LP - 1)) + 1 : 1; pieces <= 1u << LP; ++pieces)
    for (uint32_t rows = 1; rows <= 16; ++rows) {
      tile<LP, 1, 1>(pieces, rows);
      if (LP >= 2) tile<LP, 4, 1>(pieces, rows);
      if (LP <= 5) tile<LP, 1, 2>(pieces, rows);
      if (LP >= 2 && LP <= 5) tile<LP, 4, 2>(pieces, rows);
    }
}
int main() {
  pieces_of<0>(); pieces_of<1>(); pieces_of<2>(); pieces_of<3>(); pieces_of<4>(); pieces_of<5>(); pieces_of<6>();
  std::printf("%ld loads, %ld outside, %ld that a row lacks\n", loads, outside, missed);
  return loads > 0 && outside == 0 && missed == 0 ? 0 : 1;
}
"""


def test_own_rows_are_read_inside_the_rows_that_exist(tmp_path):
    src = tmp_path / "own.cpp"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(tmp_path / "own")], check=True)
    r = subprocess.run([str(tmp_path / "own")], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout
