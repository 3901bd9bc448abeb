"""The order in which workgroups take a product's tiles (gws_launch.h), compiled for the host (no GPU needed)."""
import os
import subprocess

from paper_2505_11170_amd import build

SOURCE = r"""
#include "gws_launch.h"
#include <cstdio>
#include <cstdlib>
#include <vector>
using namespace gws;
static void check(uint32_t mt, uint32_t nt, uint32_t band, bool groups, bool pairs) {
  GemmArgs g{};
  set_tile_grid(g, mt, nt, band);
  const TileGrid t{mt, nt, g.inv_band, g.inv_last};
  std::vector<char> seen((size_t)mt * nt, 0);
  for (uint32_t L = 0; L < mt * nt; ++L) {
    uint32_t m, n;
    if (groups) tile_of_groups(t, pairs, L, m, n);
    else tile_of(t, L, m, n);
    if (m >= mt || n >= nt || seen[(size_t)m * nt + n]++) {
      printf("%u x %u tiles, bands of %u, groups %d, pairs %d: number %u -> %u, %u\n", mt, nt, band, groups, pairs, L, m, n);
      exit(1);
    }
  }
}
int main() {
  for (uint32_t mt = 1; mt <= 60; ++mt)
    for (uint32_t nt = 1; nt <= 60; ++nt)
      for (int k = 0; k < 4; ++k) check(mt, nt, k == 1 ? 4 : 8, k > 1, k > 2);
  srand(1);
  for (int i = 0; i < 40; ++i) check(1 + rand() % 20000, 1 + rand() % 200, i % 4 == 1 ? 4 : 8, i % 4 > 1, i % 4 > 2);
  for (int i = 0; i < 2000000; ++i) {   // below 2^31 the reciprocal's lowest bit is not needed
    const uint32_t d = 1 + rand() % (i & 1 ? 300 : 1 << 20), n = i & 2 ? (uint32_t)rand() : 0x7FFFFFFFu - rand() % 1000;
    if (divide(n, d, reciprocal(d)) != n / d || divide(n, d, reciprocal(d) & ~1u) != n / d) {
      printf("%u / %u\n", n, d);
      return 1;
    }
  }
  return 0;
}
"""


def test_every_tile_is_taken_once(tmp_path):
    src, exe = tmp_path / "tiles.hip", tmp_path / "tiles"
    src.write_text(SOURCE)
    root = os.path.dirname(build.CSRC)
    subprocess.run([build.hipcc(), *build.FLAGS, "-I", build.CSRC, "-I", os.path.join(os.path.dirname(root), "include"), str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


JOINED = r"""
#include "gws_launch.h"
#include <cstdio>
#include <cstdlib>
#include <set>
#include <vector>
using namespace gws;
int main() {
  for (uint32_t mt = 1; mt <= 70; ++mt)
    for (uint32_t nt = 1; nt <= 60; ++nt)
      for (int way = 0; way < 2; ++way) {
        GemmArgs g{};
        const uint32_t band = way == 1 && !leaves_few(mt) ? 4 : 8;
        set_tile_grid(g, mt, nt, band, way == 0);
        const TileGrid t{mt, nt, g.inv_band, g.inv_last};
        std::vector<char> seen((size_t)mt * nt, 0);
        std::set<uint32_t> columns[8];
        for (uint32_t L = 0; L < mt * nt; ++L) {
          uint32_t m, n;
          if (way == 0) tile_of_joined(t, L, m, n);
          else tile_of(t, L, m, n);
          if (m >= mt || n >= nt || seen[(size_t)m * nt + n]++) {
            printf("%u x %u tiles, way %d: number %u -> %u, %u\n", mt, nt, way, L, m, n);
            return 1;
          }
          columns[L % 8].insert(n);
        }
        // one or two tile rows over whole bands: no XCD reads the weight's columns for all the others
        const uint32_t over = mt % (way == 0 ? 8 : 4);
        for (uint32_t x = 0; x < 8; ++x)
          if ((over == 1 || over == 2) && mt > 4 && mt < (way == 0 ? 27 : 8) && columns[x].size() > nt / 2 + 2) {
            printf("%u x %u tiles, way %d: XCD %u has tiles of %zu columns\n", mt, nt, way, x, columns[x].size());
            return 1;
          }
      }
  return 0;
}
"""


def run(tmp_path, source):
    src, exe = tmp_path / "tiles.hip", tmp_path / "tiles"
    src.write_text(source)
    root = os.path.dirname(build.CSRC)
    subprocess.run([build.hipcc(), *build.FLAGS, "-I", build.CSRC, "-I", os.path.join(os.path.dirname(root), "include"), str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_a_row_or_two_over_whole_bands_is_no_part_of_its_own(tmp_path):
    run(tmp_path, JOINED)


ONE = r"""
#include "gws_launch.h"
#include <cstdio>
#include <cstring>
using namespace gws;
int main() {
  static LaunchArgs a;
  memset(&a, 0, sizeof a);
  a.n = a.tiles_per_wg = 1;
  // workgroups, column tiles of each -> how many are dealt out: above 2048 tiles, whole rounds of 128
  const uint32_t cases[][3] = {{1, 1, 0}, {2048, 1, 0}, {2049, 1, 2048}, {2176, 1, 2176}, {683, 3, 640}, {682, 3, 0}, {0x7FFFFFEF, 4, 0x7FFFFF80}};
  for (const auto& c : cases) {
    a.tiles_per_wg_x = c[1];
    if (one_of(a, c[0]).dealt != c[2]) {
      printf("%u workgroups of %u tiles: %u\n", c[0], c[1], one_of(a, c[0]).dealt);
      return 1;
    }
  }
  return 0;
}
"""


def test_one_large_weight_is_dealt_out(tmp_path):
    run(tmp_path, ONE)
