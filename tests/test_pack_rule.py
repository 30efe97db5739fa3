"""Where a low-rank profile packs its matrices, compiled from the header on the CPU: one behind the other, and a matrix whose rows are
whole lines (or whole 16-byte vectors) where it lies is so where it is packed."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2210_17357_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "pack.h"
int main() {
    int n;
    if (std::scanf("%d", &n) != 1) return 1;
    std::vector<long long> off(n), rows(n), at(n, -1);
    std::vector<int> cols(n), used(n);
    for (int l = 0; l < n; ++l)
        if (std::scanf("%lld %lld %d %d", &off[l], &rows[l], &cols[l], &used[l]) != 4) return 1;
    lgreco::pack_matrices(n, [&](int l) { return off[l]; }, [&](int l) { return cols[l]; },
                          [&](int l) { return used[l] ? rows[l] * cols[l] : 0; }, [&](int l, long long a) { at[l] = a; });
    for (long long a : at) std::printf("%lld\n", a);
}
"""


@pytest.fixture(scope="module")
def pack(tmp_path_factory):
    d = tmp_path_factory.mktemp("pack")
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "main")], check=True)

    def call(rows):
        text = "\n".join([str(len(rows))] + [" ".join(str(int(v)) for v in r) for r in rows])
        return [int(v) for v in subprocess.run([str(d / "main")], input=text, capture_output=True, text=True,
                                               check=True).stdout.split()]
    return call


@pytest.mark.parametrize("seed", range(20))
def test_packed_matrices_keep_their_alignment(pack, seed):
    rng = np.random.default_rng(seed)
    table, off = [], 0
    for _ in range(int(rng.integers(1, 60))):
        off += int(rng.integers(0, 3)) * int(rng.choice((1, 4, 28, 32)))
        off = off if rng.random() < 0.5 else (off + 31) // 32 * 32       # a gap that restores the offset
        cols, rows = int(rng.choice((1, 3, 4, 12, 32, 36, 64, 96, 211))), int(rng.integers(1, 9))
        table.append((off, rows, cols, int(rng.random() < 0.9)))
        off += rows * cols
    at = pack(table)
    spans = sorted((a, a + r * c) for a, (_, r, c, used) in zip(at, table) if used)
    assert [a for a, _ in spans] == [0] * bool(spans) + [e for _, e in spans[:-1]]
    for a, (o, _, c, used) in zip(at, table):
        assert (a >= 0) == bool(used)
        for unit in (4, 32):
            if used and o % unit == 0 and c % unit == 0:
                assert a % unit == 0, (o, c, a)
