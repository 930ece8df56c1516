// Host-side replay of every key-row copy the similarity kernel issues for one head, and of the list its row blocks hand
// their open rows over in, using the kernel's own arithmetic (paper_2505_24133_amd/csrc/gram_index.h).  Prints
// "ok <copies>" when every row index lies in [0, n), every copy that is later read fetches exactly the rows it
// stands for, and every listed row is taken once, after it was stored, by a group inside the list; otherwise prints
// the first violation and exits 1.  Usage: gram_bounds_check n parts
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "gram_index.h"

using namespace rkv;

namespace {

const int TC = 128;                                 // keys per streamed tile (kGramTile)
const int BM = 384;                                 // rows per workgroup (kGramRows)
long long copies = 0;

// The rows of a workgroup, 32 at a time in eight copies, and as one row a lane.
bool own_rows(int n) {
  for (int row0 = 0; row0 < n; row0 += 32)
    for (int lane = 0; lane < 64; ++lane) {
      for (int jj = 0; jj < 8; ++jj) {
        const int at = gram_tile_copy_row(jj, lane), r = gram_own_row(row0, at, n);
        ++copies;
        if (at < 0 || at >= 32 || r < 0 || r >= n || (row0 + at < n && r != row0 + at))
          return std::printf("own row: n=%d row0=%d jj=%d lane=%d -> %d\n", n, row0, jj, lane, r), false;
      }
      if (gram_own_row(1 << 20, lane & 31, n) != n - 1) return std::printf("row tile past n: n=%d\n", n), false;
    }
  return true;
}

// The hand-over of one head: row blocks list a quarter of their rows or fewer at one of their looks, or none at all.  A
// list is taken in groups, by the block itself (its own rows) or by the tail kernel (all blocks' rows, in the order of
// arrival): every listed row once, with all the keys it has not been compared with, and no copy outside [0, n).
bool hand_over(int n, unsigned seed, bool own) {
  std::mt19937 rng(seed);
  const int nct = (n + TC - 1) / TC, n_pad = nct * TC, blocks = (n + BM - 1) / BM, waves = own ? 4 : (seed % 2 ? 8 : 4);
  int look = gram_next_look(-1, nct, false);
  for (int it = 0; it < nct; ++it) {
    if (gram_look(it, nct) != (it == look)) return std::printf("look: nct=%d it=%d next=%d\n", nct, it, look), false;
    if (it == look) look = gram_next_look(it, nct, false);
  }
  if (look != -1 || gram_next_look(0, nct, true) != (gram_look(7, nct) ? 7 : -1)) return std::printf("looks: nct=%d\n", nct), false;
  // the list of a head and the count behind it lie inside the head's 4 n_pad bytes
  const int places = own ? BM / 4 : n_pad / 4;
  if (!own && n_pad + 4 > 4 * n_pad) return std::printf("list region: n=%d\n", n), false;
  std::vector<unsigned> list;
  std::vector<int> taken(n, 0), expected(n, 0), below_of(n, 0);
  auto take_all = [&]() -> bool {
    if ((int)list.size() > places) return std::printf("list: n=%d seed=%u %zu rows\n", n, seed, list.size()), false;
    for (int first = 0; first < (int)list.size(); first += own ? 96 : 128) {
      const int most = own ? 96 : 128, rows = (int)list.size() - first < most ? (int)list.size() - first : most;
      int below = 0;
      for (int at = 0; at < most; ++at) {
        const int place = first + gram_open_slot(at, rows);
        if (place < first || place >= (int)list.size()) return std::printf("place: n=%d rows=%d at=%d\n", n, rows, at), false;
        if (gram_open_below(list[place]) > below) below = gram_open_below(list[place]);
        if (at < rows) ++taken[gram_open_row(list[place])];
      }
      for (int at = 0; at < rows; ++at)
        if (below < below_of[gram_open_row(list[first + at])]) return std::printf("keys left out: n=%d\n", n), false;
      std::vector<int> met(below, 0);
      for (int wave = 0; wave < waves; ++wave)
        for (int s = below - 1 - wave; s >= 0; s -= waves) {
          ++met[s];
          for (int next : {s, s - waves > 0 ? s - waves : 0})
            for (int lane = 0; lane < 64; ++lane) {
              const int r = next * 32 + gram_tile_copy_row(7, lane);
              ++copies;
              if (r < 0 || r >= n || next * 32 + 63 >= n_pad) return std::printf("subtile: n=%d s=%d row=%d\n", n, next, r), false;
            }
        }
      for (int m : met)
        if (m != 1) return std::printf("subtiles: n=%d below=%d\n", n, below), false;
    }
    list.clear();
    return true;
  };
  for (int rb = 0; rb < blocks; ++rb) {
    const int rows = n - rb * BM < BM ? n - rb * BM : BM;
    int it = 0;                                    // the look at which the block leaves
    do it = rng() % nct; while (!gram_look(it, nct));
    const int count = seed == 0 ? rows / 4 : (rng() % 4 ? (int)(rng() % (rows / 4 + 1)) : 0);
    for (int i = 0; i < count; ++i) {
      const int row = rb * BM + i * (rows / count);
      const unsigned word = gram_open_word(row, (nct - 1 - it) * 4);
      if (gram_open_row(word) != row || gram_open_below(word) != (nct - 1 - it) * 4) return std::printf("word: row=%d\n", row), false;
      expected[row] = 1;
      below_of[row] = (nct - 1 - it) * 4;
      list.push_back(word);
    }
    if (own && !take_all()) return false;
  }
  if (!take_all()) return false;
  for (int i = 0; i < n; ++i)
    if (taken[i] != expected[i]) return std::printf("row %d taken %d times: n=%d seed=%u\n", i, taken[i], n, seed), false;
  return true;
}

// A schedule that the caller asks for is the one that runs; the hand-over belongs to the default one, to scans of more than
// one tile, and is listed only where the blocks would read much for themselves.
bool schedule() {
  auto who = [](int heads, int n, float T, int beta = 1, int parts = 1, bool other = false) {
    return gram_handover(heads, (n + BM - 1) / BM, n, T, beta, parts, other);
  };
  if (who(256, 1144, 0.5f) != kOwnTail || who(300, 129, 0.9f) != kOwnTail || who(256, 4216, 0.9f) != kListTail ||
      who(1 << 22, 32767, 0.f) != kListTail)
    return std::printf("hand-over left out\n"), false;
  if (who(256, 1144, 0.5f, 1, 1, true) != kNoTail || who(256, 1144, 0.5f, 2) != kNoTail || who(256, 1144, 0.5f, 1, 2) != kNoTail ||
      who(256, 1144, 0.95f) != kNoTail || who(6144, 128, 0.5f) != kNoTail)
    return std::printf("hand-over where there is none\n"), false;
  return true;
}

}  // namespace

int main(int argc, char** argv) {
  if (argc != 3) return 2;
  if (!schedule()) return 1;
  const int n = std::atoi(argv[1]), parts = std::atoi(argv[2]);
  const int nct_all = (n + TC - 1) / TC;
  for (int part = 0; part < parts; ++part) {
    int lo, hi;
    gram_part_range(part, parts, nct_all, &lo, &hi);
    if (hi <= lo) continue;
    // the part's first tile, clamped form
    for (int row0 = 0; row0 < TC; row0 += 4)
      for (int lane = 0; lane < 64; ++lane) {
        const int r = gram_copy_row_clamped(hi - 1, TC, row0, lane, n);
        const int want = (hi - 1) * TC + row0 + (lane >> 4);
        ++copies;
        if (r < 0 || r >= n || (want < n && r != want)) {
          std::printf("clamped copy: n=%d parts=%d part=%d tile=%d row0=%d lane=%d -> row %d\n", n, parts, part, hi - 1, row0, lane, r);
          return 1;
        }
      }
    for (int ct = hi - 1; ct >= lo; --ct) {
      const int ctn = gram_next_tile(ct, lo);
      const bool read_later = ctn < ct;             // the last iteration's copy is never read
      for (int row0 = 0; row0 < TC; row0 += 4)                 // row0 = wave * 4 + jj * 16 over the four waves
        for (int lane = 0; lane < 64; ++lane) {
          const int r = gram_copy_tile_row0(ctn, TC, n) + gram_copy_group_row(row0 & 15, TC, n) +
                        gram_copy_group_row(row0 & ~15, TC, n) + gram_copy_lane_row(lane, n);
          ++copies;
          if (r < 0 || r >= n || (read_later && r != ctn * TC + row0 + (lane >> 4))) {
            std::printf("unclamped copy: n=%d parts=%d part=%d tile=%d next=%d row0=%d lane=%d -> row %d\n", n, parts, part, ct, ctn,
                        row0, lane, r);
            return 1;
          }
        }
    }
  }
  if (parts == 1) {
    if (!own_rows(n)) return 1;
    if (n > TC)                                     // a scan of one tile hands nothing over
      for (unsigned seed = 0; seed < 4; ++seed)
        if (!hand_over(n, seed, true) || !hand_over(n, seed, false)) return 1;
  }
  std::printf("ok %lld\n", copies);
  return 0;
}
