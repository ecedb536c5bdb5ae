"""The launch schedule of the row-resident sweeps (tilings with k = -K, K >= 2), checked on the host.

The schedule that the library's own code uses (csrc/rows_schedule.h) is compiled as it stands and
replayed over symbolic buffers for every chain length and every K: no launch writes a buffer
that another workgroup of the same launch reads (through the stencil, with halo rows, or from the
other half), every read sees the value the step needs, and every slot ends as the term of
its bead (bead 1's as G_1).  Also the forward sweep alone, which measures the per-step scales."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include "rows_schedule.h"
static void half(bool has, const hsf::RowsHalf &h)
{
    std::printf(" %d %d %d %d %d %d %d", (int)has, h.first, h.n, h.start, h.late, h.from_pp, h.out);
}
int main()
{
    for (int N = 2; N <= 64; ++N)
        for (int K = 2; K <= 4; ++K) {
            for (int j = 1; j <= hsf::rows_launches(N, K); ++j) {
                const hsf::RowsLaunch l = hsf::rows_schedule(N, K, j);
                std::printf("both %d %d", N, K);
                half(l.has_f, l.f);
                half(l.has_g, l.g);
                std::printf("\n");
            }
            for (int j = 1; j <= hsf::rows_blocks_of(N, K); ++j) {
                const hsf::RowsLaunch l = hsf::rows_forward(N, K, j);
                std::printf("forward %d %d", N, K);
                half(l.has_f, l.f);
                half(l.has_g, l.g);
                std::printf("\n");
            }
        }
}
"""


@pytest.fixture(scope="module")
def schedules(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("rows")
    src, exe = str(d / "driver.cpp"), str(d / "driver")
    with open(src, "w") as f:
        f.write(DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_1204_2088_amd", "csrc"),
                    src, "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout
    names = ("has", "first", "n", "start", "late", "from_pp", "out")
    sched = {}
    for line in out.splitlines():
        kind, *v = line.split()
        v = [int(x) for x in v]
        f, g = (dict(zip(names, v[k:k + 7])) for k in (2, 9))
        sched.setdefault((kind, v[0], v[1]), []).append((f, g))
    return sched


def accesses(N, j, f, g, gin, gout):
    """What launch j does: accesses (half, buffer, mode) with mode 's' (read with halo rows), 'r' (own
    sites) or 'w'; expected contents of the reads; contents of the writes in order."""
    acc, reads, writes = [], [], []

    def read(half, buf, mode, value):
        acc.append((half, buf, mode))
        reads.append((buf, value))

    def write(half, buf, value):
        acc.append((half, buf, "w"))
        writes.append((buf, value))

    if f["has"]:
        fin, fout = ("Gf", (j - 1) & 1), ("Gf", j & 1)
        if f["start"]:
            assert f["first"] == 2
            write("f", ("slot", 1), ("G", 1))
        else:
            read("f", fin if f["from_pp"] else ("slot", f["first"] - 1), "s", ("G", f["first"] - 1))
        for s in range(f["first"], f["first"] + f["n"]):
            if f["late"]:
                if s < N:   # bead N's sigma is a constant
                    read("f", ("slot", s), "r", ("sigma", s))
                write("f", ("slot", s), ("term", s))
            else:
                write("f", ("slot", s), ("G", s))
        if f["out"]:
            write("f", fout, ("G", f["first"] + f["n"] - 1))
    if g["has"]:
        if g["start"]:
            assert g["first"] == N - 1
            if g["late"]:
                read("b", ("slot", N), "r", ("G", N))
                write("b", ("slot", N), ("term", N))
        else:
            read("b", gin, "s", ("G+", g["first"] + 1))
        for s in range(g["first"], g["first"] - g["n"], -1):
            if g["late"]:
                read("b", ("slot", s), "r", ("G", s))
                write("b", ("slot", s), ("term", s))
            else:
                write("b", ("slot", s), ("sigma", s))
        if g["out"]:
            write("b", gout, ("G+", g["first"] - g["n"] + 1))
    return acc, reads, writes


def run(N, launches):
    """Replay; returns the buffers' final contents and the parity of the backward propagator."""
    state, par = {}, 0
    for j, (f, g) in enumerate(launches, 1):
        acc, reads, writes = accesses(N, j, f, g, ("Gp", par ^ 1), ("Gp", par))
        if g["has"]:
            par ^= 1
        for buf in {b for _, b, _ in acc}:
            use = [(h, m) for h, b, m in acc if b == buf]
            writers = {h for h, m in use if m == "w"}
            assert len(writers) <= 1, (N, j, buf, use)
            for h, m in use:
                if writers:
                    assert m != "s" and h in writers, (N, j, buf, use)
        for buf, value in reads:
            assert state.get(buf) == value, (N, j, buf, value, state.get(buf))
        for buf, value in writes:
            state[buf] = value
    return state, par


@pytest.mark.parametrize("K", [2, 3, 4])
def test_rows_schedule_is_race_free_and_complete(schedules, K):
    for N in range(2, 65):
        launches = schedules["both", N, K]
        assert all(f["n"] <= K and g["n"] <= K for f, g in launches)
        beads = [s for f, _ in launches if f["has"] for s in range(f["first"], f["first"] + f["n"])]
        back = [s for _, g in launches if g["has"] for s in range(g["first"], g["first"] - g["n"], -1)]
        assert beads == list(range(2, N + 1)) and back == list(range(N - 1, 1, -1))
        complete(N, launches)


@pytest.mark.parametrize("K", [2, 3, 4])
def test_forward_sweep_alone(schedules, K):
    for N in range(2, 65):
        launches = schedules["forward", N, K]
        assert not any(g["has"] for _, g in launches)
        state, _ = run(N, launches)
        assert state == {("slot", s): ("G", s) for s in range(1, N + 1)}


def complete(N, launches):
    """Replay with the density launch: G+_2 through the stencil, G_1 and the terms."""
    state, par = run(N, launches)
    assert state[("Gp", par ^ 1)] == ("G+", 2) and state[("slot", 1)] == ("G", 1)
    assert all(state[("slot", s)] == ("term", s) for s in range(2, N + 1))


def test_replay_finds_mistakes(schedules):
    """The replay itself: a wrong flag in any launch, and a block that both halves take at once, do
    not pass."""
    good = schedules["both", 12, 2]
    complete(12, good)
    for j in range(len(good)):
        for half in (0, 1):
            bad = [[dict(f), dict(g)] for f, g in good]
            bad[j][half]["late"] ^= 1
            if good[j][half]["n"]:
                with pytest.raises(AssertionError):
                    complete(12, bad)
    bad = [[dict(f), dict(g)] for f, g in good]
    bad[3][1].update(first=good[3][0]["first"] + 1, n=2)
    with pytest.raises(AssertionError):
        complete(12, bad)
