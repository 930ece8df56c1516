// The rule by which the similarity pass takes 128 rows against one column tile a workgroup (csrc/gram_index.h).
// Usage: few_rule_check heads n beta beside other.  Prints 1 or 0.
#include <cstdio>
#include <cstdlib>

#include "gram_index.h"

int main(int argc, char** argv) {
  if (argc != 6) return 2;
  const auto i = [&](int k) { return std::atoi(argv[k]); };
  std::printf("%d", rkv::gram_few(i(1), i(2), i(3), i(4) != 0, i(5) != 0) ? 1 : 0);
  return 0;
}
