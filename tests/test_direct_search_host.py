"""The host's search for the box of a direct pass (csrc/direct_split.hip), on the CPU: what it looks at, and that it takes the least."""
import os
import random
import subprocess

import pytest

from direct_layers import BESIDE
from paper_1510_06706_amd import build

SOURCE = r"""
#include <cstdio>
#include <cstring>
#include "direct.h"
int main()
{
    znn::Geom g;
    memset(&g, 0, sizeof g);
    int s, backward;
    while (scanf("%d %d %d %d %d %d %d %d %d %d", &g.f, &g.fo, &g.nz, &g.ny, &g.nx, &g.kz, &g.ky, &g.kx, &s, &backward) == 10) {
        g.spz = g.spy = g.spx = s;
        g.oz = g.nz - s * (g.kz - 1); g.oy = g.ny - s * (g.ky - 1); g.ox = g.nx - s * (g.kx - 1);
        const znn::SplitChoice c = znn::choose_split(g, backward != 0);
        printf("%d %d %d %d %.17g %.17g %d %d %d %d %d\n", c.ok, c.NJ, c.beside, c.boxes, c.cost, c.between, c.c[0] * c.c[1] * c.c[2] * c.phases, c.jgroups,
               c.splits, c.cps, c.H[0] * c.H[1] * c.H[2]);
    }
}
"""


@pytest.fixture(scope="module")
def search(tmp_path_factory):
    lib = build.LIB if os.path.exists(build.LIB) else build.build()
    folder = tmp_path_factory.mktemp("search")
    src, obj, exe = folder / "search.hip", folder / "search.o", folder / "search"
    src.write_text(SOURCE)
    flags = [f for f in build.FLAGS if f != "-O3"]
    subprocess.run([build.HIPCC] + flags + ["-O1", "-w", "--offload-host-only", "-c", "-o", str(obj), str(src)], check=True)
    subprocess.run([build.HIPCC, "-o", str(exe), str(obj), lib, "-Wl,-rpath," + os.path.dirname(lib)], check=True)

    def run(layers, **env):
        text = "".join("%d %d %d %d %d %d %d %d %d %d\n" % (f, fo, *n, *k, s, b) for f, fo, n, k, s, b in layers)
        r = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True, env={**os.environ, **env})
        rows = [line.split() for line in r.stdout.splitlines()]
        return [dict(ok=int(a), nj=int(b), beside=int(c), boxes=int(d), cost=float(e), between=float(h), launched=int(i), shape=(int(b), *map(int, rest)))
                for a, b, c, d, e, h, i, *rest in rows]

    return run


# 16-voxel tiles of a wave that an instance of so many map tiles has
TILES = {1: (1, 2, 3, 4, 6, 8), 2: (1, 2, 3, 4, 6, 8), 3: (1, 2, 3, 4, 6), 4: (1, 2, 3), 5: (1, 2)}


def boxes_of(extent, caps):
    return sum(min(extent[1], cap // x) for cap in caps for x in range(1, min(extent[2], cap) + 1))


@pytest.mark.parametrize("f,fo,n,k,s,nj,more", [
    # no box of theirs lets four more waves stage beside: those of the least groups of map tiles, once for each shape of tiles
    (80, 80, (1, 256, 256), (1, 11, 11), 1, 5, 0),
    (100, 100, (1, 250, 250), (1, 9, 9), 1, 4, 0),
    (40, 40, (1, 99, 99), (1, 11, 11), 1, 3, 0),
    (24, 36, (23, 75, 61), (3, 5, 5), 1, 3, 0),
    (60, 40, (70, 70, 70), (3, 3, 3), 2, 3, 0),
    # two and three groups of one shape of tiles besides
    (40, 40, (20, 20, 20), (3, 3, 3), 1, 3, 2),
])
def test_the_search_looks_at_each_box_once(search, f, fo, n, k, s, nj, more):
    (found,) = search([(f, fo, n, k, s, 0)])
    extent = [-(-(a - s * (b - 1)) // s) for a, b in zip(n, k)]
    caps = [16 * nv * nw for nw in (4, 8) for nv in TILES[nj]]
    assert found["ok"] and found["boxes"] == boxes_of(extent, caps) + more * boxes_of(extent, [64])
    assert bool(more) == bool(found["beside"])


@pytest.mark.parametrize("beside,layers", [
    # passes that took 1.05 to 1.25 of their time when waves staged beside: shares of few results, and many tiles of maps
    (0, [(32, 3, (13, 13, 13), (3, 3, 3), 4, 0), (30, 3, (5, 5, 5), (3, 3, 3), 1, 0), (31, 3, (21, 21, 21), (3, 3, 3), 4, 0), (10, 30, (14, 11, 17), (3, 3, 3), 1, 1),
         (40, 3, (20, 20, 20), (3, 3, 3), 4, 0), (48, 48, (11, 11, 11), (3, 3, 3), 1, 0), (48, 30, (19, 29, 19), (3, 3, 3), 4, 0),
         (36, 94, (1, 38, 63), (1, 5, 5), 1, 0), (85, 7, (1, 77, 114), (1, 5, 5), 1, 1),
         # two workgroups of two tiles of maps on a unit, one after another
         (10, 63, (1, 245, 67), (1, 5, 5), 1, 0), (14, 52, (1, 190, 49), (1, 5, 5), 1, 0), (33, 5, (21, 38, 17), (1, 5, 5), 1, 1)]),
    # and that took 0.73 to 0.97: no shares, shares of many results, five tiles of maps with a workgroup on a unit
    (1, [(16, 24, (15, 15, 15), (3, 3, 3), 2, 0), (8, 3, (13, 13, 13), (3, 3, 3), 4, 0), (40, 40, (20, 20, 20), (3, 3, 3), 1, 0), (40, 40, (21, 21, 21), (3, 3, 3), 1, 1),
         (14, 88, (13, 13, 9), (1, 5, 5), 1, 0), (90, 15, (11, 11, 16), (3, 3, 3), 1, 1)]),
])
def test_waves_stage_beside_where_that_is_faster(search, beside, layers):
    assert [found["beside"] for found in search(layers)] == [beside] * len(layers)


def test_no_xcd_takes_more_than_its_units(search):
    """81 boxes of three groups are fewer than there are units, but 33 workgroups for the 32 units of seven of the eight XCDs."""
    for found in search([(12, 88, (1, 135, 26), (1, 5, 5), 1, 0), (71, 7, (1, 30, 41), (1, 5, 5), 1, 1)]):
        assert found["beside"] and found["shape"][:2] == (2, 3)
        assert -(-found["launched"] // 8) * 3 <= 32


def test_the_tested_passes_stage_beside(search):
    """Each branch of the kernel has a pass in the tests on the GPU that takes it."""
    for layer, found in zip(BESIDE, search([layer[:6] for layer in BESIDE])):
        assert found["ok"] and found["beside"] and found["shape"] == layer[6], (layer, found)


@pytest.mark.parametrize("layer", [(40, 40, (24, 24, 24), (3, 3, 3), 1, 0), (20, 28, (23, 31, 35), (3, 5, 5), 1, 1), (130, 17, (1, 90, 77), (1, 7, 7), 1, 0)])
def test_no_pinned_box_is_expected_to_take_less(search, layer):
    (found,) = search([layer])
    rng = random.Random(5)
    priced = 0
    for _ in range(25):
        tiles = rng.choice([4, 8, 12, 16, 24, 32])
        x = rng.randint(2, 20)
        y = rng.randint(1, max(1, 16 * tiles // x))
        z = rng.randint(1, max(1, 16 * tiles // (x * y)))
        (pinned,) = search([layer], ZNN_CONV_TILE="%d,%d,%d,%d" % (tiles, z, y, x))
        if pinned["ok"]:
            priced += 1
            assert pinned["cost"] >= found["cost"] and pinned["between"] >= found["between"], (tiles, z, y, x)
    assert priced >= 5
