// Host check of the upper-triangle order of two-high tiles (index_math.hpp): every tile that holds an
// element on or above the block diagonal once, and every element of a square written exactly once
// by the rule of the symmetric schedule (sym_writes).
#include <cstdio>
#include <set>
#include <utility>
#include <vector>

#include "index_math.hpp"

int main() {
  using namespace ntk;
  for (int nb = 1; nb <= 41; ++nb) {   // nb x nb blocks, tiles of 2 x 1 blocks
    const int tm_n = (nb + 1) / 2, tn_n = nb;
    const int T = tri2_tiles(tm_n, tn_n);
    std::set<std::pair<int, int>> seen;
    constexpr int B = 3;   // elements of a block's edge
    const int R = nb * B - (nb > 1 ? 1 : 0);   // a ragged last block
    std::vector<int> writes(R * R, 0);
    for (int t = 0; t < T; ++t) {
      int tm, tn;
      tri2_index(t, tn_n, tm, tn);
      if (tm < 0 || tm >= tm_n || tn < 2 * tm || tn >= tn_n || !seen.insert({tm, tn}).second) {
        std::printf("bad tile %d of %d (nb %d): %d %d\n", t, T, nb, tm, tn);
        return 1;
      }
      for (int r = 2 * tm * B; r < (2 * tm + 2) * B && r < R; ++r)
        for (int s = tn * B; s < (tn + 1) * B && s < R; ++s) {
          bool direct, mirror;
          sym_writes(1, r, s, direct, mirror);
          writes[r * R + s] += direct;
          writes[s * R + r] += mirror;
        }
    }
    for (int i = 0; i < R * R; ++i)
      if (writes[i] != 1) {
        std::printf("element %d of nb %d written %d times\n", i, nb, writes[i]);
        return 1;
      }
  }
  std::puts("ok");
  return 0;
}
