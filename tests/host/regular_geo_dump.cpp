// Host-only driver for the geometry of regular arrays: reads
//   nx ny nz sx sy sz, then b0 nact pairs until the end of input
// and prints, for every block of each of these tiles, the element offsets that
// a lane gathers its 64 values from and which of them lie inside the array:
// first by the block's own view, then (if the tile has one) by the run view.
#include <stdio.h>

#include "../../paper_2609_24294_amd/csrc/regular_geo.hpp"

using namespace zfpx;

static void print_block(char tag, int32_t b, const BlockView& v) {
  printf("%c %d", tag, b);
  unsigned long long inside = 0;
  for (int i = 0; i < 64; i++) {
    const int z = i / 16, y = i / 4 % 4, x = i % 4;
    const int32_t at = v.x0 + x < v.rlen[y] ? v.x0 + x : v.rlen[y] - 1;
    printf(" %lld", (long long)(v.rbase[y] + (z < v.nlev ? z : v.nlev - 1) * v.lstride + at * v.sx));
    if (z < v.nlev && y < v.nrow && v.x0 + x < v.rlen[y]) inside |= 1ull << i;
  }
  printf(" %llu\n", inside);
}

int main() {
  long long n[6];
  for (long long& x : n)
    if (scanf("%lld", &x) != 1) return 2;
  const RegularGeo geo{{n[0], n[1], n[2], n[3], n[4], n[5], (int32_t)((n[0] + 3) / 4),
                        (int32_t)((n[1] + 3) / 4)}};
  int b0, nact;
  while (scanf("%d %d", &b0, &nact) == 2) {
    RunView r;
    const bool run = n[3] == 1 && geo.one_run(b0, nact, r);
    for (int lane = 0; lane < nact; lane++) {
      BlockView v;
      geo.locate_tile(b0, lane, nact, v);
      print_block('b', b0 + lane, v);
      if (!run) continue;
      for (int i = 0; i < 4; i++) {
        v.rbase[i] = r.rbase[i];
        v.rlen[i] = r.rlen[i];
      }
      v.lstride = r.lstride;
      v.sx = 1;
      v.nlev = r.nlev;
      v.nrow = r.nrow;
      v.x0 = 4 * (b0 + lane - r.block0);
      print_block('r', b0 + lane, v);
    }
  }
  return 0;
}
