// The rule that gives a problem of per-query supports to the masked tiles, for
// the problems on stdin (one "S q_offset Hq Hkv d k" a line): prints for each
// whether the masked kernel takes it and whether it splits the keys.
#include <stdio.h>

#include "attn_rules.hpp"

int main() {
  sp::Prob p{};
  while (scanf("%d %d %d %d %d %d", &p.S, &p.qo, &p.Hq, &p.Hkv, &p.d, &p.k) == 6) {
    p.G = p.Hq / p.Hkv;
    p.nq = p.S - p.qo;
    printf("%d %d\n", (int)sp::sparse_mask_pays(p), (int)sp::mask_shape(p).split);
  }
  return 0;
}
