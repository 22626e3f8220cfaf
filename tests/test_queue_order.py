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
  const int n_tiles = atoi(argv[1]), n_fb = atoi(argv[2]), grid = atoi(argv[3]), fp8 = atoi(argv[4]);
  const bool ends = both_ends(n_tiles, n_fb, grid, fp8);
  const ItemMap map(n_tiles, n_fb, ends, grid);
  printf("%d %d\n", sort_tiles(n_tiles, n_fb, grid), ends);
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
        return head, [tuple(map(int, r.split())) for r in rows]
    return run


@pytest.mark.parametrize("fp8", [0, 1], ids=["bf16", "fp8"])
@pytest.mark.parametrize("n_tiles,n_fb,grid,sorted_,ends", [
    (16, 16, 256, 0, 0),     # one item a workgroup
    (17, 16, 256, 1, 0),     # few items a workgroup: long tiles first
    (111, 16, 256, 1, 0),
    (112, 16, 256, 1, 1),
    (1000, 15, 256, 1, 1),   # odd feature blocks, a partial last chunk
    (300, 56, 304, 1, 1),
    (133, 7, 100, 1, 1),     # a grid that is no multiple of the XCDs: one queue
    (8192, 2, 256, 1, 1),
    (8193, 2, 256, 0, 0),    # a list past the limit runs in list order
    (8200, 1, 256, 0, 0),
])
def test_order(items, n_tiles, n_fb, grid, sorted_, ends, fp8):
    head, rows = items(n_tiles, n_fb, grid, fp8)
    ends = ends and not fp8
    assert head == f"{sorted_} {int(ends)}"
    assert sorted((t, f) for _, t, f in rows) == [(t, f) for t in range(n_tiles) for f in range(n_fb)]
    for q in {q for q, _, _ in rows}:
        tiles = [t for qq, t, _ in rows if qq == q]
        assert (tiles[0] > tiles[-1]) <= (ends and q % 2 == 1), q
