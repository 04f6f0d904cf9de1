"""The rules of a sweep's waits and of the end of an iteration (csrc/tt_wait.h),
compiled for the host: a wait is bounded by polls, not by time, the word itself has
the last say, and a source that lost a wave never ends as converged."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "tt_wait.h"
#include <cstdio>
using namespace tt;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
    unsigned polls = 0, pauses = 0;
    auto pause = [&] { ++pauses; };
    auto no = [] { return false; };
    // there at once; there after a while
    CHECK(poll_until([&] { return true; }, no, pause, 1) && pauses == 0);
    CHECK(poll_until([&] { return ++polls == 5000; }, no, pause, kWaitPolls) && pauses == 4999);
    // never there: `limit` polls and a last look, then given up
    polls = 0;
    CHECK(!poll_until([&] { ++polls; return false; }, no, pause, 7) && polls == 8);
    // the word arrives while the wave is off the chip, between its last poll and its giving up
    polls = 0;
    CHECK(poll_until([&] { return ++polls > 7; }, no, pause, 7));
    // a pause of any length costs one poll: the limit is not a time
    polls = 0;
    CHECK(poll_until([&] { return ++polls == 3; }, no, [&] { for (volatile int q = 0; q < 100000000; ++q) {} }, 4));
    // another wave gave up: noticed within kLostPolls polls, and the word still has the last say
    polls = 0;
    CHECK(!poll_until([&] { ++polls; return false; }, [] { return true; }, pause, kWaitPolls) && polls == kLostPolls + 1);
    polls = 0;
    CHECK(poll_until([&] { return ++polls > kLostPolls; }, [] { return true; }, pause, kWaitPolls));
    // ends of iterations
    Outcome o = iteration_outcome(1e-9, 1e-8, 12, 400, false);
    CHECK(o.status == 12 && o.done);
    o = iteration_outcome(1e-7, 1e-8, 12, 400, false);
    CHECK(o.status == -12 && !o.done);
    o = iteration_outcome(1e-7, 1e-8, 400, 400, false);
    CHECK(o.status == -400 && o.done);
    o = iteration_outcome(1e-9, 1e-8, 12, 400, true);
    CHECK(o.status == -12 && o.done);
    o = iteration_outcome(__builtin_nan(""), 1e-8, 3, 400, false);
    CHECK(o.status == -3 && !o.done);
    std::puts("ok");
    return 0;
}
"""


def test_wait_and_outcome_rules(tmp_path):
    src, exe = tmp_path / "wait.cpp", tmp_path / "wait"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2412_00031_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
