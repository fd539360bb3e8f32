"""Host geometry of the tilings, checked without a GPU: csrc/geometry.h is compiled with g++ into a
small program that prints, for ragged grids and both tile sizes, every tile's anchor token next to
the token of its slot 0; the oracle's own slot map says which tiles are real."""
import shutil
import subprocess
from pathlib import Path

import numpy as np
import pytest

from oracle import oracle as vo

ROOT = Path(__file__).resolve().parent.parent
CSRC = ROOT / "paper_2605_30325_amd" / "csrc"

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "geometry.h"
int main(int argc, char** argv) {
    const int T = atoi(argv[1]), H = atoi(argv[2]), W = atoi(argv[3]), grp = atoi(argv[7]);
    const int32_t shape[3] = {atoi(argv[4]), atoi(argv[5]), atoi(argv[6])};
    veda::HeadGeom g;
    veda::head_extents(g, shape, grp, T, H, W);
    printf("%d\n", g.n_tiles);
    for (int i = 0; i < g.n_tiles; ++i) printf("%d\n", veda::tile_anchor_token(g, i, T, H, W));
    return 0;
}
"""

CASES = [
    # grid, whole-tile shape, 64-slot tiles per whole tile
    ((21, 5, 6), (16, 2, 4), 2),     # second halves along t wholly outside the grid
    ((9, 18, 18), (8, 4, 4), 2),
    ((9, 18, 18), (1, 8, 16), 2),    # cut along h: halves outside in h
    ((3, 5, 70), (1, 1, 128), 2),    # cut along w
    ((9, 18, 18), (2, 8, 8), 2),
    ((5, 9, 10), (4, 4, 4), 1),
    ((7, 9, 11), (16, 2, 2), 1),
    ((61, 45, 80), (1, 8, 8), 1),
]


@pytest.fixture(scope="module")
def geometry_tool(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("geom")
    (d / "geom.cc").write_text(PROGRAM)
    exe = d / "geom"
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", f"-I{CSRC}", str(d / "geom.cc"), "-o", str(exe)])
    return exe


@pytest.mark.parametrize("grid,shape,grp", CASES)
def test_every_tile_anchor_is_a_real_token(geometry_tool, grid, shape, grp):
    out = subprocess.run([str(geometry_tool), *map(str, grid), *map(str, shape), str(grp)], capture_output=True,
                         text=True, check=True).stdout.split()
    n_tiles, anchors = int(out[0]), np.asarray(out[1:], np.int64)
    tokens = grid[0] * grid[1] * grid[2]
    whole = vo.num_tiles(grid, shape)
    assert n_tiles == grp * whole and len(anchors) == n_tiles
    assert anchors.min() >= 0 and anchors.max() < tokens, "an anchor outside the tensor"
    # the oracle's token -> (tile, slot) map of the whole tiles: slot 0 of 64-slot tile i is slot
    # 64*(i % grp) of whole tile i / grp
    tile_of = vo.token_tile_map(grid, shape)
    slot0 = {}
    B = shape[0] * shape[1] * shape[2]
    t, h, w = np.meshgrid(np.arange(grid[0]), np.arange(grid[1]), np.arange(grid[2]), indexing="ij")
    slot = ((t % shape[0]) * shape[1] + h % shape[1]) * shape[2] + w % shape[2]
    for n, (ti, sl) in enumerate(zip(tile_of.reshape(-1), slot.reshape(-1))):
        if sl % (B // grp) == 0:
            slot0[grp * int(ti) + int(sl) // (B // grp)] = n
    empty = 0
    for i in range(n_tiles):
        if i in slot0:
            assert anchors[i] == slot0[i], (i, anchors[i], slot0[i])
        else:      # a half with no real slot: anchored at its first half
            assert grp == 2 and i % 2 == 1 and anchors[i] == slot0[i - 1], i
            empty += 1
    if (grid, shape) in (((21, 5, 6), (16, 2, 4)), ((9, 18, 18), (1, 8, 16))):
        assert empty > 0


LIST_PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "geometry.h"
int main(int argc, char** argv) {
    printf("%d\n", veda::kListWindow);
    for (int i = 1; i + 1 < argc; i += 2) printf("%lld\n", (long long)veda::list_blocks(atoll(argv[i]), atoi(argv[i + 1])));
    return 0;
}
"""


def test_workgroups_over_a_list_of_query_tiles(tmp_path):
    """Every pair of listed tiles of one head finds a workgroup, and workgroups without one are few: not one per
    listed tile, of which half would exit (alternating with the others in ordinary lists, they left half the chip idle)."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no C++ compiler")
    (tmp_path / "list.cc").write_text(LIST_PROGRAM)
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", f"-I{CSRC}", str(tmp_path / "list.cc"), "-o", str(tmp_path / "list")])
    rng = np.random.default_rng(3)
    lists = []
    for heads in (1, 2, 40, 128):
        for n in (1, 2, 3, 16, 127, 3600, 4095, 4096, 4097, 9000, 57600):
            lists.append((heads, np.sort(np.arange(n) % heads)))                     # head after head
            lists.append((heads, np.arange(n) % heads))                              # interleaved
            lists.append((heads, rng.integers(0, heads, n)))
    args = [str(x) for heads, l in lists for x in (len(l), heads)]
    out = [int(x) for x in subprocess.run([str(tmp_path / "list"), *args], capture_output=True, text=True, check=True).stdout.split()]
    window = out[0]
    for blocks, (heads, l) in zip(out[1:], lists):
        parts = [l[i:i + window] for i in range(0, len(l), window)]
        pairs = [int(((np.bincount(p, minlength=heads) + 1) // 2).sum()) for p in parts]
        rooms = [(len(p) + min(heads, len(p))) // 2 for p in parts]                  # of each window, one after the other
        assert blocks == sum(rooms) and all(a <= b <= a + heads // 2 for a, b in zip(pairs, rooms)), (heads, len(l))


ITEMS_PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "geometry.h"
int main(int argc, char** argv) {
    const int T = atoi(argv[1]), H = atoi(argv[2]), W = atoi(argv[3]), grp = atoi(argv[4]), dies = atoi(argv[5]), full = atoi(argv[6]), thin = atoi(argv[7]);
    std::vector<veda::HeadGeom> heads;
    for (int i = 8; i + 3 < argc; i += 4) {
        const int32_t shape[3] = {atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2])};
        veda::HeadGeom g;
        veda::head_extents(g, shape, grp, T, H, W);
        g.pair_ax = atoi(argv[i + 3]);
        heads.push_back(g);
    }
    for (const veda::HeadGeom& g : heads) {
        printf("%d", g.n_tiles);
        for (int i = 0; i < g.n_tiles; ++i) printf(" %llx", (unsigned long long)veda::tile_real_slots(g, i, T, H, W));
        printf("\n");
    }
    for (const veda::HeatItem& it : veda::heat_items(heads, T, H, W, dies, 2 * thin)) printf("run %d %d %d\n", it.head, it.first, it.n);
    for (int f = 0; f < 40; ++f) for (int t = 0; t < 40; ++t) printf("list %d %d %d\n", f, t, veda::list_items(f, t));
    for (const veda::AttnItem& it : veda::attn_items(heads, T, H, W, dies, {full, thin})) printf("%d %d %d %d %d %d %u\n", it.head, it.n_tiles, it.tile[0], it.tile[1], it.tile[2], it.tile[3], it.waves);
    return 0;
}
"""


@pytest.mark.parametrize("grp,full,thin", [(1, 1, 1), (1, 2, 2), (1, 2, 4), (2, 2, 4)])
@pytest.mark.parametrize("grid", [(1, 1, 1), (1, 2, 3), (5, 9, 13), (17, 6, 7), (21, 30, 52), (4, 57, 32), (9, 18, 18)])
def test_every_wavefront_of_rows_is_in_one_work_item(tmp_path, grid, grp, full, thin):
    """The attention kernels' launch table: every 32-row part of a query tile that holds real rows belongs to exactly one
    wavefront, at most two workgroups of a head have wavefronts to spare, and no die has more than one item of either kind over its share."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no C++ compiler")
    (tmp_path / "items.cc").write_text(ITEMS_PROGRAM)
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", f"-I{CSRC}", str(tmp_path / "items.cc"), "-o", str(tmp_path / "items")])
    grow = grp
    shapes = [(4 * grow, 4, 4), (grow, 8, 8), (16 * grow, 2, 2), (grow, 1, 64)]
    axes = [3] if grp == 2 else [0, 1, 2]
    heads = [(s, ax) for s in shapes for ax in axes]
    args = [str(x) for s, ax in heads for x in (*s, ax)]
    lines = subprocess.run([str(tmp_path / "items"), *map(str, grid), str(grp), "8", str(full), str(thin), *args], capture_output=True, text=True, check=True).stdout.splitlines()
    real = []
    for (s, _), line in zip(heads, lines):
        masks = [int(x, 16) for x in line.split()[1:]]
        slots = np.asarray([[(m >> l) & 1 for l in range(64)] for m in masks], bool).reshape(-1, 64 * grp)
        tile_of = vo.token_tile_map(grid, s).reshape(-1)
        assert (slots.sum(1) == np.bincount(tile_of, minlength=len(slots))).all()
        real.append([bin(m).count("1") for m in masks])
    # the target scores': runs of tiles in order, no more rows than fit, all of them once
    runs = [[int(x) for x in l.split()[1:]] for l in lines if l.startswith("run")]
    for h, rows in enumerate(real):
        mine = [(a, n) for i in range(8) for head, a, n in runs[i::8] if head == h and n]
        assert [a + i for a, n in mine for i in range(n)] == list(range(len(rows)))
        assert all(n <= (2 if grp == 2 else 2 * thin) and sum(rows[a:a + n]) <= 128 for a, n in mine)
    for f, t, n in ([int(x) for x in l.split()[1:]] for l in lines if l.startswith("list")):
        left = max(0, t - 2) if f % 2 else t
        assert n == (f + 1) // 2 + (left + 3) // 4 <= (f + t + 1) // 2
    items = [[int(x) for x in l.split()] for l in lines[len(heads):] if l[0].isdigit() or l[0] == "-"]
    assert len(items) % 8 == 0
    for h, rows in enumerate(real):
        seen, spare = [], 0
        dies = np.zeros((2, 8), int)
        for i, (head, n, *tiles, waves) in enumerate(items):
            if head != h:
                continue
            assert 1 <= n <= max(full, thin) and len(set(tiles[:n])) == n and all(t == tiles[0] for t in tiles[n:])
            dies[int(n > 2), i % 8] += 1
            places = [(waves >> (8 * w)) & 255 for w in range(4)]
            live = [p for p in places if not p & 8]
            assert all((p & 3) < n for p in live)
            seen += [(tiles[p & 3], (p >> 2) & 1) for p in live]
            spare += len(live) < 4
        want = [(t, r) for t, m in enumerate(rows) for r in (0, 1) if grp == 2 or r == 0 or m > 32]
        assert sorted(seen) == want, (h, len(seen), len(want))
        assert thin < 4 or spare <= (0 if grp == 2 else 1 if sum(m > 32 for m in rows) % 2 == 0 else 2), (h, spare)
        assert (dies.max(1) - dies.min(1)).max() <= 1


PARTNERS_PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "geometry.h"
int main(int argc, char** argv) {
    const int T = atoi(argv[1]), H = atoi(argv[2]), W = atoi(argv[3]);
    std::vector<veda::HeadGeom> heads;
    for (int i = 5; i + 3 < argc; i += 4) {
        const int32_t shape[3] = {atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2])};
        veda::HeadGeom g;
        veda::head_extents(g, shape, 1, T, H, W);
        g.pair_ax = atoi(argv[i + 3]);
        heads.push_back(g);
    }
    for (const veda::HeadGeom& g : heads) printf("%d %d %d\n", g.nt, g.nh, g.nw);
    for (const veda::AttnItem& it : veda::attn_items(heads, T, H, W, 8, {2, atoi(argv[4]), true}))
        printf("%d %d %d %d %d %d %u %d\n", it.head, it.n_tiles, it.tile[0], it.tile[1], it.tile[2], it.tile[3], it.waves, it.partners);
    return 0;
}
"""


@pytest.mark.parametrize("thin", [2, 4])
@pytest.mark.parametrize("grid", [(1, 1, 1), (5, 9, 13), (17, 6, 7), (21, 30, 52), (9, 33, 33)])
def test_partners_share_a_workgroup(tmp_path, grid, thin):
    """Where tiles stay with their partners (neighbours along the head's axis): both are in one work item, marked as such, and nothing else
    is; every tile is in one item, with wavefronts for its real rows."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no C++ compiler")
    (tmp_path / "partners.cc").write_text(PARTNERS_PROGRAM)
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", f"-I{CSRC}", str(tmp_path / "partners.cc"), "-o", str(tmp_path / "partners")])
    heads = [(s, ax) for s in ((4, 4, 4), (1, 8, 8), (16, 2, 2)) for ax in (0, 1, 2)]
    args = [str(x) for s, ax in heads for x in (*s, ax)]
    lines = subprocess.run([str(tmp_path / "partners"), *map(str, grid), str(thin), *args], capture_output=True, text=True, check=True).stdout.splitlines()
    rows = [[int(x) for x in l.split()] for l in lines]
    items = rows[len(heads):]
    for h, (s, ax) in enumerate(heads):
        ids = np.moveaxis(np.arange(int(np.prod(rows[h]))).reshape(rows[h]), ax, 2)
        want = sorted(tuple(l[i:i + 2]) for l in ids.reshape(-1, ids.shape[2]).tolist() for i in range(0, len(l) - 1, 2))
        real = np.bincount(vo.token_tile_map(grid, s).reshape(-1), minlength=ids.size)
        mine = [it for it in items if it[0] == h]
        assert sorted(t for it in mine for t in it[2:2 + it[1]]) == list(range(ids.size))
        assert sorted(tuple(it[2 + 2 * p:4 + 2 * p]) for it in mine for p in (0, 1) if it[7] >> p & 1) == want
        for _, n, *tiles, waves, marks in mine:
            assert 1 <= n <= thin and marks < 1 << n // 2
            places = [(waves >> (8 * w)) & 255 for w in range(4)]
            live = [(p & 3, p >> 2 & 1) for p in places if not p & 8]
            assert len(set(live)) == len(live) and all(p < n for p, _ in live)
            assert all((p, r) in live for p in range(n) for r in (0, 1) if r == 0 or real[tiles[p]] > 32)


TABLES_PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "geometry.h"
int main(int argc, char** argv) {
    const int T = atoi(argv[1]), H = atoi(argv[2]), W = atoi(argv[3]), grp = atoi(argv[7]);
    const int32_t shape[3] = {atoi(argv[4]), atoi(argv[5]), atoi(argv[6])};
    std::vector<veda::HeadGeom> heads(2);
    for (veda::HeadGeom& g : heads) {
        veda::head_extents(g, shape, grp, T, H, W);
        g.pair_ax = grp == 2 ? 3 : 2;
    }
    size_t items = 0;
    for (const veda::AttnShare s : {veda::AttnShare{1, 1}, veda::AttnShare{2, 2}, veda::AttnShare{2, 4}, veda::AttnShare{2, 4, true}})
        items += veda::attn_items(heads, T, H, W, 8, s).size();
    printf("%zu %zu %zu", items, veda::heat_items(heads, T, H, W, 8, 8).size(), veda::tile_real_table(heads, T, H, W).size());
    return 0;
}
"""


@pytest.mark.parametrize("grid,shape", [((3, 9, 10), (2, 8, 8)), ((3, 9, 100), (1, 1, 128)), ((21, 45, 80), (8, 4, 4)), ((5, 9, 10), (32, 2, 2))])
def test_tables_of_ragged_128_token_tiles(tmp_path, grid, shape):
    """Built with the undefined-behaviour sanitizer: the tables are made for the 64-slot halves, and none for the whole tiles, which
    have more slots than a mask has bits."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no C++ compiler")
    flags = [gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all", f"-I{CSRC}", "-o", str(tmp_path / "tables"), "-x", "c++", "-"]
    if subprocess.run(flags, input="int main() {}", capture_output=True, text=True).returncode:
        pytest.skip("no sanitizer library")
    subprocess.run(flags, input=TABLES_PROGRAM, text=True, check=True)
    tiles = vo.num_tiles(grid, shape)
    for grp in (1, 2):
        r = subprocess.run([str(tmp_path / "tables"), *map(str, grid), *map(str, shape), str(grp)], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        items, heat, real = (int(x) for x in r.stdout.split())
        assert (items, heat, real) == (0, 0, 0) if grp == 1 else items >= 4 * 2 * tiles and heat >= 2 * tiles and real == 4 * tiles
