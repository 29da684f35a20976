"""Which tensors share memory (csrc/overlap.h): the rule against every byte of both, rows of one leading dimension and of two.  Host only."""
import random
import subprocess

import pytest

from paper_2601_17261_amd import build as B

PROGRAM = r"""
#include <cstdio>
#include "overlap.h"
int main() {
    long long v[8];
    while (scanf("%lld %lld %lld %lld %lld %lld %lld %lld", v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6, v + 7) == 8) {
        const agzo::Rows a{(uintptr_t)v[0], v[1], v[2], v[3]}, b{(uintptr_t)v[4], v[5], v[6], v[7]};
        printf("%d%d\n", (int)agzo::rows_overlap(a, b), (int)agzo::rows_overlap(b, a));
    }
}
"""


def _bytes(at, ld, n, size):
    return {at + i * ld + k for i in range(n) for k in range(size)}


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("overlap")
    src, exe = d / "overlap.cpp", d / "overlap"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", B.CSRC, str(src), "-o", str(exe)], check=True)
    return lambda rows: subprocess.run([str(exe)], input="\n".join(" ".join(map(str, a + b)) for a, b in rows), capture_output=True, text=True, check=True).stdout.split()


def test_against_every_byte(ask):
    rng, rows = random.Random(1), []
    for _ in range(4000):
        ld = rng.randint(1, 12)
        other = ld if rng.random() < 0.7 else rng.randint(1, 12)
        rows.append(((rng.randint(100, 180), ld, rng.randint(0, 6), rng.randint(1, ld)), (rng.randint(100, 180), other, rng.randint(0, 6), rng.randint(1, other))))
    got = ask(rows)
    assert len(got) == len(rows)
    seen = set()
    for (a, b), g in zip(rows, got):
        share = bool(_bytes(*a) & _bytes(*b))
        assert g[0] == g[1]
        if a[1] == b[1]:
            assert (g[0] == "1") == share, (a, b)
        else:
            assert g[0] == "1" or not share, (a, b)
        seen.add((a[1] == b[1], share, g[0]))
    assert len(seen) >= 5
