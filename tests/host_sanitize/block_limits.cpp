// Which undetected blocks the reverse mode takes.  One line per plan on stdin:
// dtype (0 c128, 1 c64), the number of undetected modes, that of detected
// ones, then the cutoffs; prints 1 for a plan that is taken, else 0.
#include <cstdio>

#include "fd_internal.h"

int main() {
  int dt, nu, nd;
  while (std::scanf("%d %d %d", &dt, &nu, &nd) == 3) {
    std::vector<int> cut(nu + nd);
    for (int& c : cut)
      if (std::scanf("%d", &c) != 1) return 2;
    fd::Plan P;
    std::string err;
    const uint32_t mask = ((1u << nd) - 1) << nu;
    if (fd::build_plan(nu + nd, cut.data(), mask, dt ? FD_C64 : FD_C128, 0, &P, &err, -1) != FD_OK) return 3;
    std::printf("%d\n", (int)fd::vjp_takes_block(P));
  }
  return 0;
}
