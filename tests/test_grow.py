"""How a context's workspace grows (csrc/grow.h): a call fails only where what it needs cannot be had, whatever else is wished for.  Host only."""
import subprocess

import pytest

from paper_2601_17261_amd import build as B

PROGRAM = r"""
#include <cstdio>
#include "grow.h"
int main() {
    unsigned long long have, need, wish, left;
    while (scanf("%llu %llu %llu %llu", &have, &need, &wish, &left) == 4) {
        unsigned long long asked = 0;
        const size_t got = agzo::grow(have, need, wish, [&](size_t n) { ++asked; return n <= left; });
        printf("%llu %llu\n", (unsigned long long)got, asked);
    }
}
"""
MB = 1 << 20


@pytest.fixture(scope="module")
def grow(tmp_path_factory):
    d = tmp_path_factory.mktemp("grow")
    src, exe = d / "grow.cpp", d / "grow"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", B.CSRC, str(src), "-o", str(exe)], check=True)

    def run(*v):
        return tuple(map(int, subprocess.run([str(exe)], input=" ".join(map(str, v)), capture_output=True, text=True, check=True).stdout.split()))
    return run


@pytest.mark.parametrize("have", [0, MB, 100 * MB])
def test_the_need_is_enough(grow, have):
    need, wish = 120 * MB + 5, 500 * MB
    assert grow(have, need, wish, need) == (need, 2)                 # room for the need alone
    assert grow(have, need, wish, need - 1) == (0, 2)
    got, asked = grow(have, need, wish, 10 ** 12)
    assert asked == 1 and wish <= got < wish + 2 * MB
    got, asked = grow(have, need, 0, 10 ** 12)
    assert asked == 1 and got >= need


def test_a_first_allocation_is_what_is_asked_for(grow):
    assert grow(0, 12345, 0, 10 ** 12) == (12345, 1)
    assert grow(0, 12345, 0, 12344) == (0, 1)


def test_growth(grow):
    """half as much again, at first up to 16 times but no more than 32 MiB more, in whole pages of 2 MiB"""
    assert grow(MB, MB + 1, 0, 10 ** 12)[0] == 16 * MB
    assert grow(10 * MB, 11 * MB, 0, 10 ** 12)[0] == 42 * MB
    assert grow(100 * MB, 101 * MB, 0, 10 ** 12)[0] == 150 * MB
    assert grow(100 * MB, 200 * MB + 1, 0, 10 ** 12)[0] == 202 * MB
