// Test harness (host only): the LDS layout of a resident share.  Arguments: cap, units,
// coarse units, held.  Prints the offsets (doubles) and the bytes.
#include <cstdio>
#include <cstdlib>

#include "resident_plan.h"

int main(int argc, char** argv) {
  if (argc != 5) return 2;
  const amrfld::ResLds l(std::atol(argv[1]), std::atol(argv[2]), std::atol(argv[3]), std::atoi(argv[4]) != 0);
  std::printf("%zu %zu %zu %zu %zu %zu %zu\n", l.p, l.rh, l.ex, l.diag, l.coarse, l.partner, l.bytes);
  return 0;
}
