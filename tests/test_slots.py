"""On how many workgroups per XCD a lone forward runs beside its extraction (csrc/slots.h).  Host only."""
import subprocess

import pytest

from paper_2601_17261_amd import build as B

PROGRAM = r"""
#include <cstdio>
#include "slots.h"
int main() {
    long long run, slots; double tile, latency, sweep, fork;
    while (scanf("%lld %lld %lf %lf %lf %lf", &run, &slots, &tile, &latency, &sweep, &fork) == 6)
        printf("%d\n", agzo::lone_slots(run, (int)slots, tile, latency, sweep, fork));
}
"""


@pytest.fixture(scope="module")
def slots(tmp_path_factory):
    d = tmp_path_factory.mktemp("slots")
    src, exe = d / "slots.cpp", d / "slots"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", B.CSRC, str(src), "-o", str(exe)], check=True)
    return lambda cases: [int(x) for x in subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True, text=True, check=True).stdout.split()]


def test_few_compute_units(slots):
    """devices of fewer than eight compute units have none per XCD: nothing is divided by that, and four are always left"""
    got = slots([(run, n, 60.0, 150.0, 20.0, 25.0) for n in range(0, 33) for run in (0, 1, 30, 200)])
    assert len(got) == 33 * 4
    for i, s in enumerate(got):
        assert 0 <= s <= max(0, i // 4 - 4)


def test_a_long_chain_beside_a_short_forward_and_a_forward_that_fills_its_rounds(slots):
    # one round of 28 tiles is hidden in a chain of 148 us; 32 tiles, which would take a second round of 100 us for a chain of 60, are not
    assert slots([(28, 32, 60.0, 148.0, 10.0, 25.0), (32, 32, 100.0, 60.0, 0.0, 25.0)]) == [14, 0]
