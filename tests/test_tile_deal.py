"""How the workgroups of a launch share the tiles of its products: csrc/tile_deal.h compiled for the
host (no GPU needed)."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# reads "W nseg tiles cost ..." per line; prints whether every tile is taken exactly once, and the longest share
PROGRAM = r"""
#include <cstdio>
#include <vector>
#define __host__
#define __device__
#define __forceinline__ inline
#include "tile_deal.h"
int main() {
  int W, nseg;
  while (std::scanf("%d %d", &W, &nseg) == 2) {
    std::vector<int> n(nseg), cost(nseg);
    for (int j = 0; j < nseg; ++j) if (std::scanf("%d %d", &n[j], &cost[j]) != 2) return 1;
    std::vector<std::vector<int>> taken(nseg);
    for (int j = 0; j < nseg; ++j) taken[j].assign(n[j], 0);
    const int lo = 1000;                     // any first tile
    bool ok = true;
    long longest = 0;
    for (int slot = 0; slot < W; ++slot) {
      mlc::Dealer d{W, slot, 0, 0};
      long share = 0;
      auto take = [&](int j, int t) {
        if (t < lo || t >= lo + n[j]) { ok = false; return; }
        ++taken[j][t - lo];
        share += cost[j];
      };
      for (int j = 0; j < nseg; ++j) {
        const mlc::Deal x = mlc::deal_tiles(d, lo, n[j], cost[j], j + 1 < nseg);
        if (x.step < 1 || x.step2 < 1) { ok = false; break; }
        for (int t = x.at; t < x.end; t += x.step) take(j, t);
        for (int t = x.at2; t < x.end2; t += x.step2) take(j, t);
      }
      if (share > longest) longest = share;
    }
    for (const auto& seg : taken) for (int c : seg) ok = ok && c == 1;
    std::printf("%d %ld\n", ok ? 1 : 0, longest);
  }
}
"""


@pytest.fixture(scope="module")
def deal(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no C++ compiler")
    tmp = tmp_path_factory.mktemp("deal")
    (tmp / "deal.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2505_23725_amd", "csrc"), str(tmp / "deal.cpp"), "-o", str(tmp / "deal")], check=True)

    def run(sets):
        text = "".join(f"{W} {len(s)} " + " ".join(f"{n} {c}" for n, c in s) + "\n" for W, s in sets)
        out = subprocess.run([str(tmp / "deal")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


def test_every_tile_once_and_no_share_a_tile_over_the_average(deal):
    """Sets of one to three products, deepest first, with few, ragged and many rounds, of equal and
    different depth."""
    rnd = random.Random(5)
    sets = []
    for _ in range(20000):
        W = rnd.choice([32, 32, 32, rnd.randint(1, 40)])
        depths = [rnd.randint(4, rnd.choice([8, 80, 300])) for _ in range(rnd.randint(1, 3))]
        if rnd.random() < 0.4:
            depths[-1] = depths[0]
        sets.append((W, [(rnd.choice([rnd.randint(0, 40), rnd.randint(1, 300)]), k + 3) for k in sorted(depths, reverse=True)]))
    for (W, s), (once, longest) in zip(sets, deal(sets)):
        assert once, (W, s)
        average = sum(n * c for n, c in s) / W
        assert longest <= average + max(c for _, c in s), (W, s, longest, average)


# sets where a product is taken whole by the workgroups that were a tile short, or is rounded over their
# gap: (tiles, cost) per product, and the longest share that dealing each tile to whoever has least gives
@pytest.mark.parametrize("products,best", [([(40, 47), (10, 19), (32, 19)], 94), ([(29, 67), (32, 43)], 110), ([(29, 83), (7, 55)], 138),
                                           ([(97, 203), (6, 195), (67, 195)], 1194),
                                           ([(50, 43), (20, 11), (29, 7)], 86), ([(17, 15), (332, 11), (5, 11)], 132)])
def test_longest_share_of_uneven_sets(deal, products, best):
    (once, longest), = deal([(32, products)])
    assert once and longest <= 1.02 * best, longest
