"""The two-step pass's launch plan (host arithmetic, compiled here with g++):
the z chunks against a search through every number of chunks, the tiles against
a search through the same candidates, and the work of planning bounded whatever
the box (long ducts had their launches held up by it)."""
import os
import shutil
import subprocess
import time

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1112_0850_amd", "csrc")
ROWS = {0: [13, 10, 8], 1: [13, 10, 8], 2: [13, 10, 8], 3: [5, 4], 4: [8]}
COST = {0: [1, 0.74, 0.67], 1: [1, 0.74, 0.67], 2: [1, 0.74, 0.67], 3: [1, 0.85], 4: [1]}
MAIN = r"""
#include <cstdio>
#include "pair_plan.h"
int main() {
  int st, nx, ny, nz;
  while (std::scanf("%d %d %d %d", &st, &nx, &ny, &nz) == 4) {
    const lbm::PairPlan p = lbm::plan_pairs(st, nx, ny, nz);
    std::printf("%d %d %d %d %d %d %d %d %d %d\n", p.choice, p.zc[0], p.zc[1], p.zc[2], p.tiles, p.tile.tx,
                p.tile.ty, p.tile.tz, p.tile.nblocks, p.pays);
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ is not installed")
    d = tmp_path_factory.mktemp("pair_plan")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I" + CSRC, "main.cpp", "-o", "plan"],
                   cwd=d, check=True)

    def run(boxes):
        text = "\n".join(" ".join(str(int(v)) for v in b) for b in boxes)
        out = subprocess.run([str(d / "plan")], input=text, capture_output=True, text=True, check=True)
        return np.array([[int(v) for v in line.split()] for line in out.stdout.splitlines()])

    return run


def ceil(a, b):
    return -(-a // b)


def chunk(nx, ny, nz, rows):
    """(time in planes, z chunk): every number of chunks of at most 128 planes."""
    tiles = ceil(nx, 64) * ceil(ny, rows)
    best = None
    for n in range(ceil(nz, 128), nz + 1):
        zc = ceil(nz, n)
        if zc < 2 and n > 1:
            break
        cost = ceil(tiles * ceil(nz, zc), 256) * (zc + 4)
        if best is None or cost < best[0]:
            best = (cost, zc)
    return best


def boxes(n, seed):
    rng = np.random.default_rng(seed)
    fixed = [(st, *b) for st in range(5) for b in [(1, 1, 1), (64, 64, 64), (1, 1, 1000), (300, 300, 300),
                                                   (2, 2, 2), (512, 512, 512), (7, 5, 129), (64, 13, 256)]]
    return fixed + [(int(rng.integers(5)), *(int(v) for v in np.exp(rng.uniform(0, [6, 6, 7]))))
                    for _ in range(n)]


def test_plan_equals_an_exhaustive_search(plan):
    todo = boxes(400, 3)
    for (st, nx, ny, nz), got in zip(todo, plan(todo)):
        best = [chunk(nx, ny, nz, r) for r in ROWS[st]]
        assert list(got[1:1 + len(best)]) == [zc for _, zc in best], (st, nx, ny, nz)
        cost = [c * k for (c, _), k in zip(best, COST[st])]
        cost[0] *= 0.88 if nx * ny * nz > 1 << 23 else 0.94
        assert got[0] == int(np.argmin(cost)), (st, nx, ny, nz)
        tile = min(((ceil(nx, x) * ceil(ny, y) * ceil(nz, z), (x, y, z))
                    for x, y, z in [(8, 4, 2), (16, 2, 4), (8, 4, 4), (8, 8, 4), (12, 6, 6)]),
                   key=lambda t: ceil(t[0], 256) * (
                       ceil((t[1][0] + 2) * (t[1][1] + 2) * (t[1][2] + 2), 64) +
                       ceil(t[1][0] * t[1][1] * t[1][2], 64) + 0.1 * (t[1][1] + 2) * (t[1][2] + 2)))
        assert (got[8], tuple(got[5:8])) == tile, (st, nx, ny, nz)


def test_planning_long_ducts_is_bounded(plan):
    """At most 128 chunk lengths are looked at per tile height: 20000 plans of
    ducts up to 16 million planes long within seconds (a walk through all numbers
    of chunks would take minutes)."""
    t = time.time()
    plan([(k % 5, 2, 2, 1 << 24 >> k % 8) for k in range(20000)])
    assert time.time() - t < 10


def test_flat_and_ragged_boxes(plan):
    """Where the rules lie: flat boxes march over z though they are small, thin ones
    take tiles and pairs, small ragged and large flat FP32 boxes single steps."""
    tiles, pays = 4, 9
    todo = [(0, 24, 24, 24), (0, 64, 64, 64), (0, 128, 128, 128), (0, 1, 179, 310), (0, 1, 341, 299),
            (3, 1, 256, 256), (4, 2, 256, 256), (0, 33, 29, 32), (0, 35, 33, 26), (0, 1, 128, 128),
            (0, 1, 1, 30000), (0, 1, 512, 512), (0, 2020, 16, 16), (0, 57, 55, 86), (1, 4396, 24, 1)]
    got = dict(zip(todo, plan([(st, nx, ny, nz) for st, nz, ny, nx in todo])))
    assert got[0, 24, 24, 24][[tiles, pays]].all()
    for b in [(0, 64, 64, 64), (0, 128, 128, 128)]:
        assert not got[b][tiles] and got[b][pays], b
    for b in [(0, 1, 179, 310), (0, 1, 341, 299), (3, 1, 256, 256), (4, 2, 256, 256)]:
        assert not got[b][tiles], b
    for b in [(0, 33, 29, 32), (0, 35, 33, 26), (0, 1, 128, 128), (0, 1, 1, 30000), (0, 1, 512, 512),
              (0, 2020, 16, 16), (0, 57, 55, 86)]:
        assert not got[b][pays], b
    assert got[1, 4396, 24, 1][[tiles, pays]].all()


def test_flat_boxes_by_cells_per_plane_of_the_pass(plan):
    """FP64 and 16-bit pairs pay by the cells per plane of the pass's time, so not in
    single planes of any size, and in flat boxes below the size that a cube needs."""
    pays = 9
    yes = [(3, 2, 1000, 650), (3, 4, 175, 328), (3, 4, 121, 477), (3, 1, 1226, 3328),
           (1, 3, 204, 603), (2, 3, 326, 389),
           (1, 6, 527, 411), (1, 128, 128, 128), (2, 512, 512, 512), (3, 64, 64, 64), (3, 512, 512, 512)]
    no = [(3, 1, 804, 336), (3, 1, 664, 723), (1, 1, 445, 1536), (2, 1, 1226, 3328), (1, 2, 397, 529),
          (2, 3, 381, 1728), (1, 1, 1351, 592)]
    got = plan([(st, nx, ny, nz) for st, nz, ny, nx in yes + no])[:, pays]
    assert got[:len(yes)].all() and not got[len(yes):].any(), list(zip(yes + no, got))
