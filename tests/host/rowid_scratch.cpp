// The row-id path's workspace for tables of every size class: no larger than
// the ABI states (N/8 + 16 bytes per 2048 rows + 16 KB, and the rounding of
// its three arrays), and room for all that each way through it writes, none
// of which overlaps what the same way reads later.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "runtime.h"

using namespace sel;
using selrt::RowidScratch;

struct Span {
  size_t at, bytes;
};

static bool apart(std::vector<Span> s, size_t total) {
  std::sort(s.begin(), s.end(), [](const Span& a, const Span& b) { return a.at < b.at; });
  for (size_t k = 0; k + 1 < s.size(); ++k)
    if (s[k].at + s[k].bytes > s[k + 1].at) return false;
  return s.back().at + s.back().bytes <= total;
}

int main() {
  long n = 0;
  for (uint64_t tiles = 0; tiles < (1u << 21); tiles += tiles < 2100 ? 1 : tiles / 9) {
    for (uint64_t tail : {0u, 1u, 2047u}) {
      const uint64_t nrows = tiles * kTileRows + tail;
      const size_t nt = (size_t)((nrows + kTileRows - 1) / kTileRows);
      const RowidScratch L(nrows);
      if (L.total() > nt * 256 + nt * 16 + (16u << 10) + 3 * 255) {
        std::printf("%llu rows: %zu bytes\n", (unsigned long long)nrows, L.total());
        return 1;
      }
      // whole tiles: words, counts, offsets and chunk sums, maps
      const size_t chunks = (nt + 1023) / 1024;
      if (!apart({{0, nt * 256}, {L.o_meta(), nt * 4}, {L.o_offsets(), nt * 4}, {L.o_chunks(), chunks * 4}, {L.o_maps(), nt * 8}},
                 L.total())) {
        std::printf("%llu rows: whole tiles overlap\n", (unsigned long long)nrows);
        return 1;
      }
      // quarter tiles: words, counts and maps (their launch has a wave a quarter, and no counts' scan)
      if (nrows <= selrt::kSmallScanRows) {
        const size_t q = (size_t)((nrows + 256 * kSmallSteps - 1) / (256 * kSmallSteps));
        if (!apart({{0, nt * 256}, {L.o_meta(), q * 4}, {L.o_maps(), q * 8}}, L.total()) || q > selrt::kSumTiles) {
          std::printf("%llu rows: quarter tiles overlap\n", (unsigned long long)nrows);
          return 1;
        }
      }
      ++n;
    }
  }
  std::printf("ok %ld\n", n);
  return 0;
}
