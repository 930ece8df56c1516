// Which key rows the similarity pass fetches, as plain integer functions shared by the kernel and by a
// host-side bounds check (tests/gram_bounds_check.cpp replays every copy of a launch on the CPU and
// asserts that no row index reaches n).  No floating point, no HIP types.
#pragma once

#if defined(__HIPCC__)
#define RKV_HD __host__ __device__ inline __attribute__((always_inline))
#else
#define RKV_HD inline
#endif

namespace rkv {

// Column tiles [lo, hi) that column part `part` of `parts` scans (descending), of nct_all tiles in all.
RKV_HD void gram_part_range(int part, int parts, int nct_all, int* lo, int* hi) {
  *lo = (int)((long long)part * nct_all / parts);
  *hi = (int)((long long)(part + 1) * nct_all / parts);
}

// The tile whose copy is issued while tile `ct` is used.  In the last iteration of a part this is `ct`
// itself: a redundant copy that keeps the copy code free of branches and is never read.
RKV_HD int gram_next_tile(int ct, int ct_lo) { return ct - 1 > ct_lo ? ct - 1 : ct_lo; }

// One wave-wide copy moves four consecutive rows (lane / 16 picks the row).  Clamped form, used for a
// part's first tile (the only one that can reach past n through a real copy): row per lane.
RKV_HD int gram_copy_row_clamped(int ct, int tc, int row0, int lane, int n) {
  const int r = ct * tc + row0 + (lane >> 4);
  return r < n - 1 ? r : n - 1;
}

// Unclamped form, used for every copy issued inside the scan: row = tile row + group row + lane row, the first
// two wave-uniform.  Every copy made this way that is later read lies in a tile that ends at or before n
// (so n >= tc), where all three functions are the identity.  The copy of a part's last iteration is never
// read and can name the head's last, partly filled tile: the tile's first row is pulled back so that the
// tile stays inside [0, n), and a head with fewer than tc candidates reads rows 0 .. min(3, n - 1) only.
RKV_HD int gram_copy_tile_row0(int ct, int tc, int n) {
  int r = ct * tc;
  if (r > n - tc) r = n - tc;
  return r > 0 ? r : 0;
}
RKV_HD int gram_copy_group_row(int row_in_tile, int tc, int n) { return n >= tc ? row_in_tile : 0; }
RKV_HD int gram_copy_lane_row(int lane, int n) {
  const int r = lane >> 4;
  return r < n - 1 ? r : n - 1;
}

// The scan with beta = 1 keeps a subtile's keys in another order: place q of the 32 holds key halves_key(q), which gives half h
// of a wave the keys 16 h .. 16 h + 15 of the subtile as its accumulator elements 0 .. 15.  Copy jj of a wave (four rows, at place
// (wave + 4 jj) * 4 of the tile) then moves rows halves_wave_row(wave) + halves_copy_row(jj) .. + 3 of the tile.
RKV_HD int halves_key(int q) { return 16 * ((q >> 2) & 1) + 4 * (q >> 3) + (q & 3); }
RKV_HD int halves_wave_row(int wave) { return 16 * (wave & 1) + 4 * (wave >> 1); }
RKV_HD int halves_copy_row(int jj) { return 32 * (jj >> 1) + 8 * (jj & 1); }
RKV_HD int halves_copy_clamped(int tile_row0, int wave, int jj, int lane, int n) {
  const int r = tile_row0 + halves_wave_row(wave) + halves_copy_row(jj) + (lane >> 4);
  return r < n - 1 ? r : n - 1;
}

// A row tile or subtile of 32 rows is moved by eight wave-wide copies; the row inside it that copy jj of a lane moves.
RKV_HD int gram_tile_copy_row(int jj, int lane) { return jj * 4 + (lane >> 4); }
// The row a workgroup reads for the row at place `at` of a row tile that begins at row0 (past n: row n - 1).
RKV_HD int gram_own_row(int row0, int at, int n) { return row0 + at < n - 1 ? row0 + at : n - 1; }

// When a row block may count its open rows (iteration `it` of nct): after tiles 1, 2, 4, 8 and every eighth, as long as
// what is left of the scan is at least a quarter of what is done.
RKV_HD bool gram_look(int it, int nct) { return ((it & (it + 1)) == 0 || (it & 7) == 7) && (nct - 1 - it) * 4 >= it + 1; }
// The iteration of the next such count after `it` (-1: of the first), -1 if there is none; with `rare` none before tile 8.
RKV_HD int gram_next_look(int it, int nct, bool rare) {
  const int next = it >= 7 ? it + 8 : (rare ? 7 : it * 2 + 1 + (it < 0));
  return gram_look(next, nct) ? next : -1;
}

// Whether a row block leaves the scan with its last open rows: the default direction of the recency rule with beta = 1,
// one workgroup per row block, T <= 0.9, and no other schedule asked for (`other`: RKV_FLAG_TRIANGULAR_SCAN, the transposed
// rule, or RKV_FLAG_SKIP_SATURATED, whose gathering of open rows inside a block is the better one where a third or more of
// the rows stay open: redundancy of 256 heads of n = 4216, 35 % of the rows without a partner, 580 us against 900, of 512
// heads of n = 2168 370 against 530; where nearly all rows meet one it is the worse, repeated text of n = 1144 80 against 56).
// Above T = 0.9 only near-copies are partners and too few rows meet one early.  Redundancy, us, full scan / hand-over
// at T = 0.95: 256 heads of n = 1144 repeated text 91.9 / 92.2, noisy copies 104 / 105, clusters 102 / 103; of
// n = 4216 936 / 945, 985 / 992, 979 / 1020; 48 heads of noisy copies 250 / 258; 8 heads of n = 32760 repeated text
// 1713 / 1862.  At T = 0.5 repeated text of n = 1144 takes 57 instead of 92.
// A scan of one tile has nothing to leave.
// Who takes the rows: the block itself (kOwnTail) reads the older keys once more for the few rows it has left, from L2 where
// the head's other blocks read them too; the tail kernel (kListTail) reads them once per 128 rows of a head, but is
// a launch of its own, empty where partners are rare (2 to 3 us).  The line is drawn at what all blocks would read, 500 MB.
// Redundancy, us, own / list, repeated text: 256 heads of n = 1144 (225 MB) 53.2 / 54.0, of n = 1692 (554 MB) 94 / 104, of
// n = 2168 (853 MB) 103.2 / 102.4, of n = 4216 (3 GB) 257 / 208; 64 heads of n = 2168 (213 MB) 35.6 / 41.9, 128 (426 MB)
// 62.7 / 60.9; 48 heads of n = 4216 (584 MB) 76 / 66; 8 heads of n = 32760 (6 GB) 362 / 246.  No partners: 128 heads of
// n = 2168 137.5 / 139.2, full scan 138.2.
enum GramHandover : int { kNoTail = 0, kOwnTail = 1, kListTail = 2 };
RKV_HD GramHandover gram_handover(int heads, int row_blocks, int n, float T, int beta, int parts, bool other) {
  if (beta != 1 || parts != 1 || other || !(T <= 0.9f) || n <= 128) return kNoTail;
  return (long long)heads * row_blocks * n * 256 <= 500000000ll ? kOwnTail : kListTail;
}

// Whether the pre-pass copies its chunks to LDS ahead (prepass_dma_kernel): two row tiles of queries, a contiguous cache of 16-byte aligned
// rows (what its copies move) and chunks for eight a workgroup, with `resident` workgroups at a time (768 on the 256 compute units of an
// MI355X).  Chunks a workgroup, us of the stand-alone importance without / with it, 40 query rows and n = 2168: 1.1 17.2 / 18.5, 3 31.2 / 31.4,
// 4.1 38.5 / 37.0, 6 52.4 / 48.1, 8 63.9 / 54.7, 10 84.7 / 70.9, 16 140 / 123, 32 273 / 241; 64 query rows, 1.1 18.7 / 20.1, 4.1 42.6 / 38.7,
// 8 72.5 / 57.0; n = 512, 40 query rows, 8 69.1 / 61.7.  Reading a chunk back from LDS costs its latency, which the copies in flight pay for
// from about four a workgroup on; from eight on it is ahead by a tenth and more at every size.
// With one row tile of queries both run at the same 4.9 TB/s, writes included (1024 heads of n = 8312 548 / 522 us in a trace, the whole step
// within 1 %).  Windows of 16 with two row tiles, and paged caches, have not been built this way.
RKV_HD bool prepass_by_dma(int chunks, int resident, bool aligned) { return aligned && (long long)chunks >= 8ll * resident; }

// Few heads: 128 rows against one column tile a workgroup (gram_few.hip), where a head has at most 16 tiles (so many reports a row
// the finalize kernel merges at once) and the workgroups, four to a compute unit, make about a round and a half at most.
// It gains where rows have partners, which the other launch's workgroups of 384 rows spend their time on.  It costs a little where there are
// none and its workgroups need another round of the one XCD that a head's lie on (which is also why one head costs what eight do).  Time of
// the other launch over this one's; keys of repeated text / noisy copies / 256 clusters at T = 0.5, repeated text / clusters at T = 0.95 /
// independent keys:
//   a step    1 head,  n = 384 1.23 1.31 1.35 / 1.18 1.25 / 1.10, 1152 1.11 1.12 1.14 / 1.01 1.09 / 0.98, 2048 1.12 1.11 1.17 / 0.99 1.09 / 0.94
//             8 heads, n = 640 1.24 1.25 1.28 / 1.16 1.21 / 1.08, 1152 1.10 1.11 1.13 / 1.01 1.10 / 0.99, 1792 1.07 1.12 1.21 / 1.00 1.10 / 0.95
//             16, n = 1152 1.05 1.07 1.09 / 0.96 1.04 / 0.96; 64, n = 640 1.11 1.20 1.26 / 1.04 1.16 / 1.00; 256, n = 192 1.00 1.02 1.02 / 1.00 1.01 / 0.97
//   the pass  8 heads, n = 1024 1.20 1.22 1.26 / 1.06 1.19 / 0.99, 1792 1.12 1.18 1.31 / 0.99 1.15 / 0.92; 96, n = 384 1.19 1.25 1.28 / 1.09 1.17 / 1.02
//   alone     132, n = 384 1.07 1.12 1.12 / 0.98 1.07 / 0.91; 160, n = 384 1.01 1.05 1.05 / 0.92 1.00 / 0.86; 256, n = 192 0.94 0.99 0.99 / 0.94 0.96 / 0.85
// (T = 0.95 draws no line: repeated text, whose noise is just above it, is even there or 4 % slower, noisy copies and clusters 4 to 16 %
// faster.)  With more than 128 heads, of two or three tiles then, the pass alone is the slower one; a step (`beside`: it forms the
// importance in the same launch) is not.
RKV_HD bool gram_few(int heads, int n, int beta, bool beside, bool other) {
  const int tiles = (n + 127) / 128;
  return beta == 1 && !other && tiles > 1 && tiles <= 16 && (long long)heads * tiles * tiles <= 1700 && (beside || heads <= 128);
}

// An open row, as it is listed: the row and the subtile of 32 keys below which it is still to be compared.
RKV_HD unsigned gram_open_word(int row, int below) { return (unsigned)row | ((unsigned)below << 16); }   // row < 2^15, below < 2^10
RKV_HD int gram_open_row(unsigned word) { return (int)(word & 0xffffu); }
RKV_HD int gram_open_below(unsigned word) { return (int)(word >> 16); }
// Place inside a group of `rows` rows that a lane reads for place `at` (past the end: the last one, not used).
RKV_HD int gram_open_slot(int at, int rows) { return at < rows - 1 ? at : rows - 1; }

}  // namespace rkv
