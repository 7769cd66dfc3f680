"""Host logic of the time marginal's work split (csrc/gw_tgplan.h, gw_hetplan.h).

Samples in order of frequency are dealt to chunks (interpolation nodes of the full
band, edges of the heterodyned bins), each chunk's sums over the grid points that
its samples reach lie in points of its own, and the grid kernel adds the chunks of
each grid point by the cover's lists.  The driver simulates that on whole numbers,
where any order of the sums gives the same, and compares with spreading every
sample directly: every sample once, every chunk within its points.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2607_28265_amd", "csrc")

DRIVER = r"""
#include "gw_hetplan.h"
#include "gw_tgplan.h"
#include <cstdio>
#include <cstdlib>
#include <random>
using namespace gw;

using Grid = std::vector<long long>;

static void spread(Grid& g, int at, int q) {
  for (int m = 0; m < kTgW; ++m) g[at + m] += (long long)(q + 1) * (m + 3);
}

// What the kernels do with chunks of samples [first, end) at grid points [a0, a0 + len).
static bool simulate(const std::vector<int32_t>& cell, const std::vector<int32_t>& first,
                     const std::vector<int32_t>& a0, const std::vector<int32_t>& len, int n_g, const char* what) {
  const TgCoverPlan cov = tgrid_cover(a0, len, n_g);
  Grid pts(cov.n_pts, 0), want(n_g, 0), got(n_g, 0);
  std::vector<int> seen(cell.size(), 0);
  for (size_t c = 0; c < a0.size(); ++c) {
    for (int q = first[c]; q < first[c + 1]; ++q) {
      ++seen[q];
      if (cell[q] < a0[c] || cell[q] + kTgW > a0[c] + len[c]) return std::printf("%s: chunk %d leaves its points\n", what, (int)c), false;
      spread(pts, cov.shift[c] + cell[q], q);
    }
  }
  for (size_t q = 0; q < cell.size(); ++q) {
    if (seen[q] != 1) return std::printf("%s: sample %d taken %d times\n", what, (int)q, seen[q]), false;
    spread(want, cell[q], q);
  }
  for (int g = 0; g < n_g; ++g) {
    const int32_t* p = &cov.pts[4 * g];
    for (int j = 0; j < 2; ++j)
      if (p[j] >= 0) got[g] += pts.at(p[j]);
    for (int c = p[2]; c <= p[3]; ++c) got[g] += pts.at(cov.shift[c] + g);
    if (got[g] != want[g]) return std::printf("%s: grid point %d\n", what, g), false;
    if (g >= cov.n_many && cov.n_many > 0 && p[3] - p[2] + 3 > 4) return std::printf("%s: leading points\n", what), false;
  }
  return true;
}

static bool nodes(std::mt19937& rng, int n_cell, int n, int most, int skew) {
  std::vector<int32_t> cell(n);
  for (auto& c : cell) {
    double u = (rng() >> 8) / 16777216.0;
    for (int k = 0; k < skew; ++k) u *= (rng() >> 8) / 16777216.0;
    c = std::min((int)(n_cell * u), n_cell - 1);
  }
  std::sort(cell.begin(), cell.end());
  const TgChunkPlan p = tgrid_chunks(cell, n_cell, most, 64);
  char what[96];
  std::snprintf(what, sizeof what, "nodes n_cell %d n %d most %d skew %d", n_cell, n, most, skew);
  for (int c = 0; c < p.n(); ++c) {
    if (p.first[c] >= p.first[c + 1]) return std::printf("%s: chunk %d empty\n", what, c), false;
    if (c < p.n_dense && (p.len[c] != kTgW || p.first[c + 1] - p.first[c] > 4 * most))
      return std::printf("%s: dense chunk %d\n", what, c), false;
  }
  return simulate(cell, p.first, p.a0, p.len, n_cell + kTgW - 1, what);
}

static bool edges(std::mt19937& rng, int n_cell, int ne, int want, int skew) {
  std::vector<int32_t> cell(ne), bs(n_cell + 1, 0);
  for (auto& c : cell) {
    double u = (rng() >> 8) / 16777216.0;
    for (int k = 0; k < skew; ++k) u *= (rng() >> 8) / 16777216.0;
    c = std::min((int)(n_cell * u), n_cell - 1);
    ++bs[c + 1];
  }
  std::sort(cell.begin(), cell.end());
  for (int b = 0; b < n_cell; ++b) bs[b + 1] += bs[b];
  const HetTmPlan p = het_tm_plan(bs, n_cell, ne, want);
  std::vector<int32_t> len(p.nch());
  for (int c = 0; c < p.nch(); ++c) len[c] = p.bhi[c] - p.blo[c] + kTgW - 1;
  char what[96];
  std::snprintf(what, sizeof what, "edges n_cell %d ne %d want %d skew %d", n_cell, ne, want, skew);
  return simulate(cell, p.e0, p.blo, len, n_cell + kTgW - 1, what);
}

int main() {
  std::mt19937 rng(11);
  int failures = 0;
  // a long segment at a short window: all nodes in a few cells
  for (int n_cell : {1, 2, 4})
    for (int n : {1, 12, 97, 4801, 9409, 36900, 40000, 65003, 70001, 130000, 262144})
      for (int most : {12, 47, 48}) failures += !nodes(rng, n_cell, n, most, 0);
  for (int trial = 0; trial < 3000; ++trial) {
    const int n_cell = 1 + (int)(rng() % 700), skew = (int)(rng() % 4);
    failures += !nodes(rng, n_cell, 1 + (int)(rng() % 9000), 12 + (int)(rng() % 37), skew);
    failures += !edges(rng, n_cell, 1 + (int)(rng() % 600), 1 + (int)(rng() % 300), skew);
  }
  std::printf("%d failures\n", failures);
  return failures != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_time_grid_work_split(tmp_path):
    src = tmp_path / "plan_check.cpp"
    src.write_text(DRIVER)
    exe = tmp_path / "plan_check"
    subprocess.run(["g++", "-O2", "-std=c++17", "-D_GLIBCXX_ASSERTIONS", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    assert "0 failures" in r.stdout
