// Host check of the upper-triangle order of two-high tiles (index_math.hpp): every tile that holds an
// element on or above the block diagonal once, and every element of a square written exactly once
// by the rule of the symmetric schedule (itself from the diagonal of blocks up, its mirror from
// above it).
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
    std::vector<int> writes(nb * nb, 0);
    for (int t = 0; t < T; ++t) {
      int tm, tn;
      tri2_index(t, tn_n, tm, tn);
      if (tm < 0 || tm >= tm_n || tn < 2 * tm || tn >= tn_n || !seen.insert({tm, tn}).second) {
        std::printf("bad tile %d of %d (nb %d): %d %d\n", t, T, nb, tm, tn);
        return 1;
      }
      for (int br = 2 * tm; br < 2 * tm + 2 && br < nb; ++br) {
        if (br <= tn) ++writes[br * nb + tn];
        if (br < tn) ++writes[tn * nb + br];
      }
    }
    for (int i = 0; i < nb * nb; ++i)
      if (writes[i] != 1) {
        std::printf("block %d of nb %d written %d times\n", i, nb, writes[i]);
        return 1;
      }
  }
  std::puts("ok");
  return 0;
}
