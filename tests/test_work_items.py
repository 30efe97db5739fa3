"""Size of the refinement's work items, compiled from the header on the CPU.  A launch is as long as its largest item, so
an item stays within a small multiple of an even share of the tiles however many layers there are; and there are
no more items than the partial histograms have room for."""
import os
import subprocess

import numpy as np
import pytest

from paper_2210_17357_amd import workloads as W

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2210_17357_amd", "csrc")
MOST = 64                                       # 2^19 elements in tiles of 8192

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "work_items.h"
int main() {
    int n, slots, most;
    while (std::scanf("%d %d %d", &n, &slots, &most) == 3) {
        std::vector<int> t(n);
        for (int& v : t)
            if (std::scanf("%d", &v) != 1) return 1;
        std::printf("%d\n", lgreco::tiles_per_item(n, [&](int l) { return t[l]; }, slots, most));
    }
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("work_items")
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "main")], check=True)

    def call(tiles, slots, most=MOST):
        line = " ".join(str(int(v)) for v in (len(tiles), slots, most, *tiles))
        return int(subprocess.run([str(d / "main")], input=line, capture_output=True, text=True, check=True).stdout)
    return call


def _tiles(shapes, tile=8192):
    n = np.array([int(np.prod(s)) for s in shapes])
    rest = n % tile
    return n // tile + (rest >= 512) + (rest % 512 > 0)


def _items(tiles, group):
    return int((-(-np.asarray(tiles) // group)).sum())


def _check(tiles, slots, group, most=MOST):
    tiles = np.asarray(tiles)
    share = max(1, min(most, -(-int(tiles.sum()) // slots)))         # an even share, rounded up
    assert share <= group <= min(most, 3 * share), (group, share)
    assert _items(tiles, group) <= slots + int((tiles > 0).sum()) or group == most


@pytest.mark.parametrize("slots", [256, 512])
@pytest.mark.parametrize("blocks, width, vocab", [(24, 96, 3000), (24, 176, 5000), (24, 256, 9000), (20, 256, 9000),
                                                  (20, 128, 3000), (40, 256, 9000)])
def test_models_of_about_as_many_layers_as_slots_and_more(rule, slots, blocks, width, vocab):
    tiles = _tiles(W.gpt2_medium_shapes(blocks, width, 4 * width, vocab, 1024))
    _check(tiles, slots, rule(tiles, slots))


@pytest.mark.parametrize("slots", [256, 512])
def test_edges(rule, slots):
    for tiles in ([1], [0, 0, 5], [1] * slots, [1] * (slots + 1), [2] * (slots - 1) + [50000], [70000], [1] * 2000,
                  [0] * 300 + [40] * 3, [10] * (slots // 2), [7] * (slots - 1)):
        _check(tiles, slots, rule(tiles, slots))
    rng = np.random.default_rng(5)
    for _ in range(60):
        tiles = rng.integers(0, 4, rng.integers(1, 700))
        tiles[rng.integers(0, tiles.size, 5)] = rng.integers(1, 3000, 5)
        _check(tiles, slots, rule(tiles, slots))


@pytest.mark.parametrize("shapes", [W.resnet50_shapes(1000), W.resnet18_shapes(1000)], ids=["resnet50", "resnet18"])
def test_few_layers_fill_the_slots_once(rule, shapes):
    """Where layers are few, small ones are an item each and all items start at once."""
    tiles = _tiles(shapes)
    for slots in (256, 512):
        items = _items(tiles, rule(tiles, slots))
        assert 0.75 * slots <= items <= slots, items
