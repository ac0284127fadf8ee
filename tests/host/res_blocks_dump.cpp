// Test harness (host only): blocks of a resident launch.  Argument: compute units.
// Prints res_blocks(g, n_cu) for g = 1 .. n_cu.
#include <cstdio>
#include <cstdlib>

#include "resident_plan.h"

int main(int argc, char** argv) {
  if (argc != 2) return 2;
  const int n_cu = std::atoi(argv[1]);
  for (int g = 1; g <= n_cu; ++g) std::printf("%d ", amrfld::res_blocks(g, n_cu));
  return 0;
}
