// Which piece of the gather of kept rows a workgroup takes: head and block of rows.  Compiled for the host, too.
#pragma once

#include <cstdint>

#include "gram_index.h"

namespace rkv {

// Workgroups are dealt round-robin to the 8 XCDs, and the rows that neighbouring blocks read and write lie next to one another: a head's
// blocks go to one XCD.  Of each eight heads XCD x takes the x-th, so that the heads in hand at a time are neighbours; of the up to seven heads
// that are left each XCD takes an eighth of the blocks, in a run (by whole heads one head of budget 32376 takes 24 us instead of 3.9).
// Long lists of caches that the 256 MB behind the L2s don't hold are the exception: there eight heads in hand are eight places of memory
// MiB apart, and blocks in the order of the heads, one place, are faster.
// us of the gather, blocks in the order of the heads / as above, sums over 8 budgets and placements of the buffers; in brackets the worst of these
// against the better order of that placement: 300 heads of N = 300 78.0 (1.14) / 75.0 (1.02), 256 of 1152 226 (1.04) / 220 (1.00), 600 of 1152
// 704 (1.37) / 657 (1.00), 64 of 4224 and fewer by 4 to 6 % for the latter, 512 of 4224 2400 / 2375, 64 of 8320 576 (1.40) / 515 (1.01),
// 256 of 8320 2564 (1.06) / 2513 (1.01), 20 of 24000 506 / 488; 100 of 10000 1413 (1.26) / 1408 (1.04), 100 of 12000 1816 / 1845, 48 of 12288
// 927 (1.14) / 951 (1.06), 80 of 14000 1714 / 1778, 16 of 32768 555 (1.00) / 646 (1.20).  Paged caches beyond 256 MB lose 1 to 2 % of the gather by itself
// (256 of 2176 659 / 671) and nothing of a step.
constexpr int64_t kGatherLongBlocks = 640;          // of 16 rows
constexpr int64_t kGatherLargeBytes = 256ll << 20;  // K and V

RKV_HD int64_t gather_cache_bytes(int64_t heads, int64_t rows) { return heads * rows * 512; }

// Rows that the 256 MB behind the L2s cannot hold are read past them: the pre-pass's keys are gone from there and nothing reads these
// rows again.  Of contiguous caches the rows that are read count: with all of the cache's counted, a tenth kept of 256 heads of n = 4216 took
// 20.3 us instead of 17.4, half of 512 of 1144 49.9 instead of 44.0, three quarters of 256 of 2168 70.6 instead of 60.3.
// Paged ones count whole, since a dense copy of the keys is in the way, too: a step of 256 of n = 2168 240 / 230.
// K and V, us, ordinary / non-temporal loads, behind the other kernels of an attention-only step: 180 MiB 83 / 88, 252 114 / 116,
// 288 127 / 129, 325 170 / 170, 360 168 / 164, paged 180 106 / 104, 252 148 / 140, 288 168 / 159, 360 225 / 210; a whole step of 256 heads of
// n = 4216 (1.1 GB) 431 / 406, of 6144 heads of n = 2168 (6.8 GB) 4749 / 4657, of 1024 of n = 8312 3131 / 3081.
RKV_HD bool gather_streams(int64_t heads, int64_t n_tokens, int64_t budget, bool paged) {
  return gather_cache_bytes(heads, paged || budget > n_tokens ? n_tokens : budget) > (256ll << 20);
}

struct GatherOrder {
  int64_t blocks;              // of the whole call: a multiple of 8
  uint32_t eights;             // blocks that each XCD takes of the heads by the eight
  uint32_t run, step;          // block i of XCD x after those is block x * run + i * step of the heads that are left
};

RKV_HD GatherOrder gather_order(int64_t heads, int64_t blocks_per_head, int64_t cache_bytes) {
  if (cache_bytes >= kGatherLargeBytes && blocks_per_head > kGatherLongBlocks) return {(heads * blocks_per_head + 7) / 8 * 8, 0, 1, 8};
  const int64_t eights = heads / 8 * blocks_per_head, run = (heads % 8 * blocks_per_head + 7) / 8;
  return {(eights + run) * 8, (uint32_t)eights, (uint32_t)run, 1};
}

// Workgroup `block` of the whole call.  head may be past the last one: nothing to do then.
RKV_HD void gather_piece(uint32_t block, uint32_t blocks_per_head, uint32_t eights, uint32_t run, uint32_t step, int& head, int& blk) {
  const uint32_t xcd = block & 7, i = block >> 3;
  const bool left = i >= eights;
  const uint32_t at = left ? eights * 8 + xcd * run + (i - eights) * step : i;
  const uint32_t q = at / blocks_per_head;
  head = (int)(left ? q : q * 8 + xcd);
  blk = (int)(at - q * blocks_per_head);
}

}  // namespace rkv
