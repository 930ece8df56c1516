// csrc/gather_index.h: every block of every head is taken by exactly one workgroup, those past the end take none, and the XCDs (workgroups
// are dealt to them in turn) get whole heads, and of up to seven heads that are left one run each.
// Long lists of large caches go to the XCDs block by block.
// Usage: gather_order_check heads blocks_per_head launch (workgroups a launch takes) cache_bytes.  Prints "ok" or what is wrong.
// gather_order_check streams heads n_tokens budget paged: whether the rows are read past the caches, 1 or 0.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "gather_index.h"

int main(int argc, char** argv) {
  if (argc == 6) return std::printf("%d", rkv::gather_streams(std::atoi(argv[2]), std::atoi(argv[3]), std::atoi(argv[4]), std::atoi(argv[5]) != 0) ? 1 : 0), 0;
  if (argc != 5) return 2;
  const int64_t heads = std::atoll(argv[1]), per = std::atoll(argv[2]), launch = std::atoll(argv[3]);
  const int64_t bytes = std::atoll(argv[4]);
  const rkv::GatherOrder order = rkv::gather_order(heads, per, bytes);
  if (order.blocks % 8 || order.blocks < heads * per || order.blocks >= heads * per + 8) return std::printf("grid %lld", (long long)order.blocks), 1;
  std::vector<int> taken(heads * per, 0), xcd_of(heads * per, -1);
  std::vector<int64_t> share(8, 0);
  for (int64_t first = 0; first < order.blocks; first += launch)
    for (int64_t i = 0; i < launch && first + i < order.blocks; ++i) {
      int head, blk;
      rkv::gather_piece((uint32_t)(first + i), (uint32_t)per, order.eights, order.run, order.step, head, blk);
      if (head < 0 || blk < 0 || blk >= per) return std::printf("block %lld: head %d blk %d", (long long)(first + i), head, blk), 1;
      if (head >= heads) continue;
      ++taken[head * per + blk];
      xcd_of[head * per + blk] = (int)(i & 7);       // dealt anew at each launch
      ++share[i & 7];
    }
  int64_t changes = 0;
  for (int64_t i = 0; i < heads * per; ++i) {
    if (taken[i] != 1) return std::printf("piece %lld taken %d times", (long long)i, taken[i]), 1;
    if (i % per && xcd_of[i] != xcd_of[i - 1]) ++changes;
  }
  if (!(bytes >= rkv::kGatherLargeBytes && per > rkv::kGatherLongBlocks) && changes > (heads % 8 ? 7 : 0)) return std::printf("heads cut %lld times", (long long)changes), 1;
  for (int x = 0; x < 8; ++x)
    if (share[x] > (heads * per + 7) / 8) return std::printf("XCD %d has %lld blocks", x, (long long)share[x]), 1;
  return std::printf("ok"), 0;
}
