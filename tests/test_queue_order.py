"""The work queues of the large-tile kernels on the CPU: every item is handed out once, and the odd
queues run backwards for sorted tiles only."""
import os
import subprocess

import pytest

from paper_2607_23099_amd import build

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "queue.h"
using namespace damoe;
int main(int argc, char** argv) {
  const int n_tiles = atoi(argv[1]), n_fb = atoi(argv[2]), grid = atoi(argv[3]);
  const bool sorted = sort_tiles(n_tiles, n_fb, grid);
  const ItemMap map(n_tiles, n_fb, sorted, grid);
  printf("%d\n", sorted);
  for (int q = 0; q < map.nq; ++q)
    for (int t = 0; t < map.queue_len(q); ++t) {
      int tile = -1, fb = -1;
      if (map.item(q, t, n_tiles, tile, fb)) printf("%d %d %d\n", q, tile, fb);
    }
}
"""


@pytest.fixture(scope="module")
def items(tmp_path_factory):
    d = tmp_path_factory.mktemp("queue")
    (d / "order.hip").write_text(SRC)
    subprocess.run([build._hipcc(), "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17",
                    "-I" + build.INCLUDE, "-I" + os.path.join(build.PKG, "csrc"), str(d / "order.hip"), "-o",
                    str(d / "order")], check=True, capture_output=True)

    def run(*args):
        out = subprocess.run([str(d / "order"), *map(str, args)], check=True, capture_output=True, text=True).stdout
        head, *rows = out.splitlines()
        return head == "1", [tuple(map(int, r.split())) for r in rows]
    return run


@pytest.mark.parametrize("n_tiles,n_fb,grid,sorted_", [
    (16, 16, 256, False),     # one item a workgroup
    (17, 16, 256, True),
    (1000, 15, 256, True),    # odd feature blocks, a partial last chunk
    (300, 56, 304, True),
    (33, 7, 100, True),       # a grid that is no multiple of the XCDs: one queue
    (8192, 2, 256, True),
    (8193, 2, 256, False),    # a list past the limit runs in list order
    (8200, 1, 256, False),
])
def test_order(items, n_tiles, n_fb, grid, sorted_):
    got_sorted, rows = items(n_tiles, n_fb, grid)
    assert got_sorted == sorted_
    assert sorted((t, f) for _, t, f in rows) == [(t, f) for t in range(n_tiles) for f in range(n_fb)]
    for q in {q for q, _, _ in rows}:
        tiles = [t for qq, t, _ in rows if qq == q]
        backwards = tiles[0] > tiles[-1]
        assert backwards <= (sorted_ and q % 2 == 1), q
