// Threads per row of the register top-k for the problems on stdin (one "S
// q_offset b k W" a line).
#include <stdio.h>

#include "topk_rules.hpp"

int main() {
  sp::Prob p{};
  while (scanf("%d %d %d %d %d", &p.S, &p.qo, &p.b, &p.k, &p.W) == 5) {
    p.nq = p.S - p.qo;
    p.R = (p.nq + p.b - 1) / p.b;
    printf("%d\n", sp::topk_threads(p, p.S - (p.W < p.k ? p.W : p.k)));
  }
  return 0;
}
