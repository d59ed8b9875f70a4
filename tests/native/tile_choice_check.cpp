// Host check of the LM head's kernel choice (lmhead_tiles.h): prints the choice
// for each "M d V aligned" line of stdin as "narrow positions nontemporal
// two_per_cu".
#include <stdio.h>

#include "lmhead_tiles.h"

int main() {
  int M, d, V, offset;
  while (scanf("%d %d %d %d", &M, &d, &V, &offset) == 4) {
    const void* W = reinterpret_cast<const void*>((uintptr_t)(4096 + offset));
    const fork::TileChoice t =
        fork::choose_tile(M, d, (V + 255) / 256, fork::whole_lines(W, d), 2LL * V * d);
    printf("%d %d %d %d\n", t.narrow, t.positions, t.nontemporal, t.two_per_cu);
  }
  return 0;
}
