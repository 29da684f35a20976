"""The fork of a stream (csrc/fork.h) where calls of the runtime fail: a call never leaves work on the second stream that nothing waits
for.  The class takes the runtime's calls as a parameter, so its failures are played on the host."""
import subprocess

import pytest

from paper_2601_17261_amd import build as B

# Streams hold numbers of work; an event remembers what its stream held; a stream that waits for an event has seen that.  A call whose
# number is in `failing` fails
PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <set>
#include <stdexcept>
#include <string>
#include "fork.h"
struct Stream { int work = 0; int seen_of_side = 0; bool host_waited = false; };
struct Event { int at = 0; };
static std::set<int> failing;
static int calls = 0;
static Stream *the_side;
struct Fake {
    typedef Stream* stream_t; typedef Event* event_t; typedef int error_t;
    static int record(Event* e, Stream* s) { if (failing.count(calls++)) return 1; e->at = s->work; return 0; }
    static int wait(Stream* s, Event* e) { if (failing.count(calls++)) return 2; if (s != the_side) s->seen_of_side = e->at; return 0; }
    static int synchronize(Stream* s) { if (failing.count(calls++)) return 3; s->host_waited = true; return 0; }
};
// one call: some work on the side; then returned, left early, or by an exception.  Prints what came of it
int main(int argc, char** argv) {
    const std::string how = argv[1];
    for (int i = 2; i < argc; ++i) failing.insert(atoi(argv[i]));
    Stream main_, side; Event fork, join;
    the_side = &side;
    side.work = 5; join.at = 5; main_.seen_of_side = 5;          // an older fork, joined
    int rc = 0, closed = 0;
    bool enqueued = false;
    try {
        agzo::Fork<Fake> f(&main_, &side, &fork, &join);
        rc = f.run([&](Stream* s) {
            s->work += 1;
            enqueued = true;
            if (how == "throws") throw std::runtime_error("no memory");
            return how == "refuses" ? 9 : 0;
        });
        if (how == "closes") { closed = f.close(); if (f.open()) closed = -closed; }
    } catch (const std::runtime_error&) { rc = 99; }
    printf("%d %d %d %d\n", rc, closed, (int)enqueued, (int)(!enqueued || main_.seen_of_side == side.work || side.host_waited));
}
"""


@pytest.fixture(scope="module")
def play(tmp_path_factory):
    d = tmp_path_factory.mktemp("fork")
    src, exe = d / "fork.cpp", d / "fork"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", B.CSRC, str(src), "-o", str(exe)], check=True)

    def run(how, *failing):
        out = subprocess.run([str(exe), how] + [str(f) for f in failing], check=True, capture_output=True, text=True).stdout
        return tuple(int(v) for v in out.split())
    return run


# the runtime's calls in order: 0 record fork, 1 side waits, 2 record join, 3 main waits (4: or the host does)
@pytest.mark.parametrize("how", ["closes", "leaves", "throws", "refuses"])
def test_all_is_waited_for(play, how):
    rc, closed, enqueued, waited = play(how)
    assert rc == {"throws": 99, "refuses": 9}.get(how, 0) and closed == 0 and enqueued == 1 and waited == 1


@pytest.mark.parametrize("how", ["closes", "leaves", "throws", "refuses"])
@pytest.mark.parametrize("failing", [0, 1])
def test_nothing_is_launched_where_the_fork_fails(play, how, failing):
    rc, _, enqueued, waited = play(how, failing)
    assert rc == failing + 1 and enqueued == 0 and waited == 1


@pytest.mark.parametrize("how", ["closes", "leaves", "throws", "refuses"])
@pytest.mark.parametrize("failing", [2, 3])
def test_the_host_waits_where_joining_fails(play, how, failing):
    rc, closed, enqueued, waited = play(how, failing)
    assert enqueued == 1 and waited == 1
    assert how != "closes" or closed > 0          # and the caller hears of it (one that left early has an error of its own)


def test_a_close_that_fails_stays_open_and_is_tried_again(play):
    rc, closed, enqueued, waited = play("closes", 3, 4)          # neither the stream nor, at first, the host waits
    assert rc == 0 and closed == -2 and enqueued == 1 and waited == 1
