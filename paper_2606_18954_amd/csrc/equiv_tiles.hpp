// Work list of the large-prompt similarity kernel (equiv.hip): which tile runs on which XCD.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

#include <hip/hip_runtime.h>

namespace ga {

constexpr int kXcds = 8;

struct EquivTiles {
  int32_t tile = 0;                   // states along a tile's side: 128 or 64
  std::vector<int4> items;            // (first row state, first column state, prompt end, 0)
};

// Tiles are 64 x 64 as long as all of them run at once (four per CU), else 128 x 128.  us a call at
// width 4096, 128 x 128 | 64 x 64: one prompt of 300 states (15 small tiles) 64 | 26, 12 of 700 (792) 74 |
// 53, 32 of 400 (896) 72 | 54, 2 of 2000 (1056) 78.6 | 79.1, one of 4000 (2016) 123 | 149.
constexpr int64_t kFewTiles = 4 * 256;

// The upper-triangle tiles of the prompts [first, end).  Workgroups go to the 8 XCDs in turn, so
// entry 8 k + x runs on XCD x.  A prompt goes whole to the XCD with the least work so far, whose L2
// then holds what its tiles share, as long as that XCD stays within a sixteenth of the mean;
// otherwise its tiles, row strip after row strip, fill the XCDs up to the mean, the least loaded first.
// So no XCD gets more than a sixteenth, or a tile, beyond its eighth, whatever the prompts' sizes.
// Width 4096, 128 x 128 tiles, us a call, whole prompts always | this: 4000 + 7 x 300 states 594 |
// 132, 1500 + 7 x 500 117 | 67, 9 x 2000 317 | 217; 64 x 517, where no prompt is cut, 171 | 171; 100 x
// 300 104.5 | 104.7 (107.5 with eight runs of equal weight, which cut seven of the prompts).
// Narrow tiles go last in a list and fill the gaps; lists are padded with empty tiles.
inline EquivTiles equiv_tiles(const std::vector<int2>& prompts) {
  EquivTiles out;
  int64_t small = 0;                                               // tiles of 64 x 64
  for (const int2& p : prompts) {
    const int64_t t = (p.y - p.x + 63) / 64;
    small += t * (t + 1) / 2;
  }
  const int32_t tile = out.tile = small <= kFewTiles ? 64 : 128;
  // Relative time of a tile whose columns start `left` states before its prompt's end: narrow ones
  // (at most half a tile of columns) take about a third.
  auto tile_weight = [&](int32_t left) -> int64_t { return left > tile / 2 ? 3 : 1; };
  auto weight = [&](int2 p) {
    const int64_t t = (p.y - p.x + tile - 1) / tile;               // tiles along a side
    return 3 * (t * (t - 1) / 2) + t * tile_weight(p.y - p.x - (int32_t)(t - 1) * tile);
  };
  int64_t total = 0;
  for (const int2& p : prompts) total += weight(p);
  std::vector<int4> full[kXcds], narrow[kXcds];
  int64_t load[kXcds] = {0};
  for (const int2& p : prompts) {
    int x = (int)(std::min_element(load, load + kXcds) - load);
    const bool whole = 16 * kXcds * (load[x] + weight(p)) <= 17 * total;
    for (int32_t i0 = p.x; i0 < p.y; i0 += tile)
      for (int32_t j0 = i0; j0 < p.y; j0 += tile) {
        if (!whole && kXcds * load[x] >= total) x = (int)(std::min_element(load, load + kXcds) - load);
        const int64_t w = tile_weight(p.y - j0);
        (w > 1 ? full : narrow)[x].push_back(make_int4(i0, j0, p.y, 0));
        load[x] += w;
      }
  }
  size_t longest = 0;
  for (int x = 0; x < kXcds; ++x) {
    full[x].insert(full[x].end(), narrow[x].begin(), narrow[x].end());
    longest = std::max(longest, full[x].size());
  }
  out.items.reserve(longest * kXcds);
  for (size_t k = 0; k < longest; ++k)
    for (int x = 0; x < kXcds; ++x)
      out.items.push_back(k < full[x].size() ? full[x][k] : make_int4(0, 0, 0, 0));
  return out;
}

}  // namespace ga
