// Host-side replay of the key order of the scan with beta = 1 (csrc/gram_index.h): the copies put key halves_key(q) of a subtile
// at place q, every copy of every tile names rows inside [0, n) and, where it is read, exactly the rows it stands for, and a half's
// accumulator elements are 16 consecutive keys.  Prints "ok <copies>" or the first violation.  Usage: halves_order_check n
#include <cstdio>
#include <cstdlib>

#include "gram_index.h"

using namespace rkv;

int main(int argc, char** argv) {
  if (argc != 2) return 2;
  const int n = std::atoi(argv[1]), TC = 128, nct = (n + TC - 1) / TC;
  long long copies = 0;
  for (int i = 0; i < 16; ++i)
    for (int half = 0; half < 2; ++half)
      if (halves_key(8 * (i / 4) + 4 * half + i % 4) != 16 * half + i) return std::printf("element %d of half %d\n", i, half), 1;
  for (int ct = nct - 1; ct >= 0; --ct)
    for (int wave = 0; wave < 4; ++wave)
      for (int jj = 0; jj < 8; ++jj) {
        if (halves_copy_row(jj) % halves_copy_row(1) != 0) return std::printf("step %d\n", jj), 1;
        for (int lane = 0; lane < 64; lane += 16) {
          const int place = (wave + 4 * jj) * 4 + (lane >> 4), want = ct * TC + place / 32 * 32 + halves_key(place % 32);
          const int first = halves_copy_clamped(ct * TC, wave, jj, lane, n);
          const int steps = halves_copy_row(jj) / halves_copy_row(1);
          const int next = gram_next_tile(ct, 0);          // the copy issued while tile ct is used
          const int row = gram_copy_tile_row0(next, TC, n) + gram_copy_group_row(halves_wave_row(wave), TC, n) +
                          steps * gram_copy_group_row(halves_copy_row(1), TC, n) + gram_copy_lane_row(lane, n);
          ++copies;
          if (first < 0 || first >= n || (want < n && first != want)) return std::printf("first: n=%d ct=%d row %d for %d\n", n, ct, first, want), 1;
          if (row < 0 || row >= n || (next < ct && row != next * TC + place / 32 * 32 + halves_key(place % 32)))
            return std::printf("next: n=%d ct=%d row %d\n", n, next, row), 1;
        }
      }
  std::printf("ok %lld\n", copies);
  return 0;
}
