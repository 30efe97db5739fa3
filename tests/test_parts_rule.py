"""Sizes of tiles and how many workgroups a tile is dealt to, compiled from the header on the CPU: as many as its size asks for where
most tiles are full, and no more than one for 4096 elements (and 4096) that find nothing to do unless every tile has one."""
import os
import subprocess

import numpy as np
import pytest

from paper_2210_17357_amd import workloads as W

from gpu_util import many_small, tile_count as _tiles, tile_size

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2210_17357_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "parts.h"
int main() {
    // part 0: the size of the tiles, `tile` 1 in calls with Top-K layers
    long long n, total, tile, part;
    while (std::scanf("%lld %lld %lld %lld", &n, &total, &tile, &part) == 4)
        std::printf("%d\n", part ? lgreco::part_shift(n, total, tile, part) : lgreco::tile_size(total, tile != 0));
}
"""
PARTS = (512, 2048, 4096, 8192)


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("parts")
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "main")], check=True)

    def call(*rows):
        text = "\n".join(" ".join(str(int(v)) for v in r) for r in rows)
        return [int(v) for v in subprocess.run([str(d / "main")], input=text, capture_output=True, text=True,
                                               check=True).stdout.split()]
    return call


@pytest.mark.parametrize("name", ["resnet18", "resnet50", "gpt2_medium", "transformer_lm", "tiny"])
@pytest.mark.parametrize("part", PARTS)
def test_models_keep_the_parts_asked_for(rule, name, part):
    shapes = {"resnet18": W.resnet18_shapes, "resnet50": W.resnet50_shapes, "gpt2_medium": W.gpt2_medium_shapes,
              "transformer_lm": W.transformer_lm_shapes, "tiny": W.tiny_shapes}[name]()
    numels = [int(np.prod(s)) for s in shapes]
    total = sum(numels)
    for tile in (8192, 32768) if total > 1 << 26 else (8192,):
        assert rule((_tiles(numels, tile), total, tile, part)) == [int(np.log2(tile // part))]


def test_bounds_over_tables_of_all_kinds(rule):
    rng = np.random.default_rng(3)
    rows = []
    for _ in range(400):
        tile = int(rng.choice((8192, 16384, 32768)))
        n = int(np.exp(rng.uniform(0, np.log(3e6))))
        total = max(1, int(n * tile * np.exp(rng.uniform(np.log(1e-4), 0))))
        rows += [(n, total, tile, p) for p in PARTS]
    for (n, total, tile, part), s in zip(rows, rule(*rows)):
        assert 0 <= s and tile >> s >= part
        groups, used = n << s, total // (tile >> s)
        assert s == 0 or groups - used <= total // 4096 + 4096
        assert groups * 256 < 2 ** 32
        if (tile >> s) > part:                           # the next shorter parts would be too many
            groups, used = n << (s + 1), total // (tile >> (s + 1))
            assert groups - used > total // 4096 + 4096 or groups > 1 << 23


def test_tens_of_thousands_of_small_layers(rule):
    numels = [1500] * 50000
    n = _tiles(numels, 32768)
    assert rule(*((n, sum(numels), 32768, p) for p in PARTS)) == [0] * len(PARTS)
    with_one_large = numels[:5000] + [1 << 26]
    n = _tiles(with_one_large, 32768)
    assert rule((n, sum(with_one_large), 32768, 512)) == [1]


def test_sizes_of_tiles(rule):
    """The GPU tests' copy of the rule, around every size at which a tile changes."""
    edges = [t * 2 ** k + d for t in (1024, 2048) for k in range(12, 17) for d in (-1, 0, 1)]
    totals = edges + [1, 511, 10 ** 6, 3 * 10 ** 8] + [e * 3 // 2 for e in edges]
    for topk in (0, 1):
        assert rule(*((0, t, topk, 0) for t in totals)) == [tile_size(t, bool(topk)) for t in totals]


def test_lengths_that_the_gpu_tests_rely_on(rule):
    for n_layers, shift in ((1200, 1), (3000, 0)):
        lengths = many_small(n_layers)
        total = int(lengths.sum())
        assert tile_size(total, False) == 8192
        assert rule(*((_tiles(lengths, 8192), total, 8192, p) for p in (512, 2048, 4096))) == [shift] * 3
