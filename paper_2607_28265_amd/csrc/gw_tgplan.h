// Work split of the time marginal's frequency grid (host only): samples in order
// of their grid cell are dealt to chunks, each chunk's sums go to its own points,
// and the grid kernel adds the chunks that reach a grid point.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

namespace gw {

constexpr int kTgW = 14;  // grid points that a sample is spread over

// Chunk c adds to grid points a0[c] .. a0[c] + len[c] - 1, stored from off[c]
// on (off the running sum of len); a0 and a0 + len nondecreasing.  Per grid
// point g < n_g (pts [n_g][4]): where the first and the second chunk that
// reach it hold it (-1: none), then the third and the last of them; per chunk
// off - a0 (shift).  n_many: leading points, some with more than four chunks,
// which k_tgrid sums with four lanes each (at most 256 of them, else none).
struct TgCoverPlan {
  std::vector<int32_t> pts, shift;
  int n_pts = 0, n_many = 0;
};
inline TgCoverPlan tgrid_cover(const std::vector<int32_t>& a0, const std::vector<int32_t>& len, int n_g) {
  TgCoverPlan p;
  const int nc = (int)a0.size();
  for (int c = 0; c < nc; ++c) {
    p.shift.push_back(p.n_pts - a0[c]);
    p.n_pts += len[c];
  }
  p.pts.resize(4 * (size_t)n_g);
  int lo = 0, hi = -1;
  for (int g = 0; g < n_g; ++g) {
    while (hi + 1 < nc && a0[hi + 1] <= g) ++hi;
    while (lo <= hi && a0[lo] + len[lo] <= g) ++lo;
    p.pts[4 * g] = lo <= hi ? p.shift[lo] + g : -1;
    p.pts[4 * g + 1] = lo < hi ? p.shift[lo + 1] + g : -1;
    p.pts[4 * g + 2] = lo + 2;
    p.pts[4 * g + 3] = hi;
    if (hi - lo >= 4) p.n_many = g + 1;
  }
  if (p.n_many > 256) p.n_many = 0;
  return p;
}

// Chunks of samples in order of frequency: cell[q] (nondecreasing) is sample q's
// grid cell, ``most`` the samples a wave takes, max_cells the cells it may span.
// Chunk c holds samples first[c] .. first[c + 1] - 1 and the grid points a0[c] ..
// a0[c] + len[c] - 1.  The first n_dense chunks are one cell each (or a part of
// one), of at most 4 most samples that a workgroup's four waves share: the leading
// cells of more than 2 most samples.  The others are whole cells, a wave each.
struct TgChunkPlan {
  std::vector<int32_t> first, a0, len;
  int n_dense = 0;
  int n() const { return (int)a0.size(); }
};
inline TgChunkPlan tgrid_chunks(const std::vector<int32_t>& cell, int n_cell, int most, int max_cells) {
  TgChunkPlan p;
  const int n = (int)cell.size();
  std::vector<int32_t> count(n_cell, 0);
  for (const int32_t a : cell) ++count[a];
  auto put = [&](int q, int a, int len) {
    p.first.push_back(q);
    p.a0.push_back(a);
    p.len.push_back(len);
  };
  for (int q = 0; q < n;) {
    const int a = cell[q];
    int e = q + count[a], top = a;
    if (count[a] > 2 * most && p.n_dense == p.n()) {
      // parts of equal size, the last one with what is left
      const int parts = (count[a] + 4 * most - 1) / (4 * most), each = (count[a] + parts - 1) / parts;
      for (; q < e; q += each) {
        put(q, a, kTgW);
        ++p.n_dense;
      }
      q = e;
      continue;
    }
    while (e < n && e - q + count[cell[e]] <= most && cell[e] - a < max_cells) {
      top = cell[e];
      e += count[top];
    }
    put(q, a, top - a + kTgW);
    q = e;
  }
  p.first.push_back(n);
  return p;
}

}  // namespace gw
