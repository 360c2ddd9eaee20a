// Reads lines "last first batch" and prints msplat::round_limit for each
// (csrc/common.hpp, compiled for the host).
#include <cstdio>

#include "common.hpp"

int main() {
  unsigned last, first, batch;
  while (std::scanf("%u %u %u", &last, &first, &batch) == 3)
    std::printf("%u\n", msplat::round_limit(last, first, batch));
}
