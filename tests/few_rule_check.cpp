// Rules of csrc/gram_index.h: when the similarity pass takes 128 rows against one column tile a workgroup.
// Usage: few_rule_check heads n beta beside other, or few_rule_check chunks resident aligned for the rule of the pre-pass.  Prints 1 or 0.
#include <cstdio>
#include <cstdlib>

#include "gram_index.h"

int main(int argc, char** argv) {
  const auto i = [&](int k) { return std::atoi(argv[k]); };
  if (argc == 4) return std::printf("%d", rkv::prepass_by_dma(i(1), i(2), i(3) != 0) ? 1 : 0), 0;
  if (argc != 6) return 2;
  std::printf("%d", rkv::gram_few(i(1), i(2), i(3), i(4) != 0, i(5) != 0) ? 1 : 0);
  return 0;
}
