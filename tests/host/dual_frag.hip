// Host-side check of the dual family's sparse outlier operand (dual_frag.h):
// for every combination of positions in a group, the stored values and index
// bits decode to the dense codes, and the two positions of every four ascend.
// Built and run by tests/test_dual_frag.py on the CPU; no GPU call is made.
#include <cstdio>

#include "dual_frag.h"

static long checked = 0;

// dense codes of the lane's four groups, from the stored form
static bool decode(const sdq::dual::SparseOut& s, uint8_t (&d)[4][8]) {
  for (int g = 0; g < 4; ++g) {
    for (int p = 0; p < 8; ++p) d[g][p] = 0;
    for (int four = 0; four < 2; ++four) {
      const int i0 = (s.idx >> (8 * g + 4 * four)) & 3, i1 = (s.idx >> (8 * g + 4 * four + 2)) & 3;
      if (i0 >= i1) return false;
      d[g][4 * four + i0] = uint8_t(s.v[g] >> (16 * four));
      d[g][4 * four + i1] = uint8_t(s.v[g] >> (16 * four + 8));
    }
  }
  return true;
}

template <int NP>
static bool check(const int (&pos)[4][2], const int (&code)[4][2]) {
  uint32_t a[NP], b[NP];
  uint8_t want[4][8] = {};
  for (int p = 0; p < NP; ++p) {
    auto hw = [&](int g) { return uint32_t(pos[g][p] | (code[g][p] << 8)); };
    a[p] = hw(0) | (hw(1) << 16);
    b[p] = hw(2) | (hw(3) << 16);
    for (int g = 0; g < 4; ++g)
      if (code[g][p]) want[g][pos[g][p]] = uint8_t(code[g][p]);
  }
  uint8_t got[4][8];
  if (!decode(sdq::dual::sparse_outliers<NP>(a, b), got)) return false;
  for (int g = 0; g < 4; ++g)
    for (int p = 0; p < 8; ++p)
      if (got[g][p] != want[g][p]) return false;
  ++checked;
  return true;
}

int main() {
  // every position (pair) in each of the four groups, the others at a second one
  const int codes[4][2] = {{0x81, 0x7F}, {0x01, 0xFF}, {0x80, 0x55}, {0xAA, 0x03}};
  for (int g = 0; g < 4; ++g)
    for (int p0 = 0; p0 < 8; ++p0)
      for (int p1 = 0; p1 < 8; ++p1)
        for (int q0 = 0; q0 < 8; ++q0)
          for (int q1 = q0 + 1; q1 < 8; ++q1) {
            int pos[4][2], code[4][2];
            for (int i = 0; i < 4; ++i)
              for (int j = 0; j < 2; ++j) { pos[i][j] = j ? q1 : q0; code[i][j] = codes[i][j]; }
            pos[g][0] = p0;
            if (!check<1>(pos, code)) return std::printf("one plane: group %d position %d\n", g, p0), 1;
            pos[g][1] = p1;
            // ascending positions, or (no second outlier) both at 0 without codes
            if (p0 == p1) {
              if (p0) continue;
              code[g][0] = code[g][1] = 0;
            } else if (p0 > p1) {
              continue;
            }
            if (!check<2>(pos, code)) return std::printf("two planes: group %d positions %d %d\n", g, p0, p1), 1;
          }
  std::printf("dual fragments ok: %ld\n", checked);
  return 0;
}
