// The mask scan's order of tiles (sel_device.h) against the scan's own loop:
// every tile's place is its wave's first place plus its turn, and the places
// are 0 .. ntiles - 1, each taken once.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "sel_device.h"

using namespace sel;

static int check(uint64_t nrows, uint32_t waves, uint32_t tps, bool small = false) {
  const MaskOrder o = mask_order(nrows, waves, tps, small);
  const uint32_t rows = small ? 256 * kSmallSteps : kTileRows;
  const uint32_t ntiles = (uint32_t)((nrows + rows - 1) / rows), nfull = small ? ntiles : (uint32_t)(nrows / rows);
  std::vector<char> seen(ntiles, 0);
  for (uint32_t w = 0; w < waves; ++w) {
    uint32_t turn = 0, place = wave_place(o, w);
    auto take = [&](uint32_t tile) {
      uint32_t t = 0;
      const uint32_t p = tile_place(o, tile, t);
      if (p >= ntiles || p != place + turn || t != turn || seen[p]) {
        std::printf("rows %llu waves %u tps %u: tile %u at place %u turn %u, taken %u of place %u\n",
                    (unsigned long long)nrows, waves, tps, tile, p, t, turn, place);
        return false;
      }
      seen[p] = 1;
      ++turn;
      return true;
    };
    if (w == waves - 1 && nfull < ntiles && !take(nfull)) return 1;
    for (uint32_t run = w; run * tps < nfull; run += waves)
      for (uint32_t k = 0; k < tps && run * tps + k < nfull; ++k)
        if (!take(run * tps + k)) return 1;
  }
  for (char s : seen)
    if (!s) return 1;
  // few tiles, one a wave: places are tile numbers
  if (ntiles <= waves && tps == 1)
    for (uint32_t t = 0; t < ntiles; ++t) {
      uint32_t turn = 0;
      if (tile_place(o, t, turn) != t) return 1;
    }
  return 0;
}

int main() {
  long n = 0;
  for (uint32_t tps : {1u, 2u, 4u})
    for (uint32_t waves : {1u, 2u, 3u, 4u, 7u, 64u, 250u})
      for (uint32_t tiles = 0; tiles <= 1100; tiles += tiles < 70 ? 1 : 37)
        for (uint32_t tail : {0u, 1u, 2047u}) {
          if (check((uint64_t)tiles * kTileRows + tail, waves, tps)) return 1;
          if (tps == 1 && check((uint64_t)tiles * kTileRows + tail, waves, tps, true)) return 1;
          ++n;
        }
  if (check((1ull << 32) - 1, 3072, 1) || check((1ull << 32) - 1, 1, 4)) return 1;
  std::printf("ok %ld\n", n);
  return 0;
}
