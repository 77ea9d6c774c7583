"""The host's rules for splitting stage launches (csrc/schedule.h), compiled
by themselves: every launch size at three chip sizes."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2107_10987_amd", "csrc")
FACE, COLUMN, PERSISTENT, TILED = 1, 2, 3, 4
SHIM = """
#include "schedule.h"
using namespace hydro;
extern "C" {
int bucket(int n) { return bucket_of(n); }
int parts(int n, int cu) { return leaf_parts(n, cu); }
int beside(int n, int nstage, int nlaunch, int streams) { return blocks_beside(n, nstage, nlaunch, streams); }
int automatic(int beside, int cu) { return auto_schedule(beside, cu); }
int table(const int32_t *t, int n, int beside, int cu) { return table_schedule(t, n, beside, cu); }
void split(int sched, int n, int beside, int alone, int cu, int *o) {
    const Split s = split_launch(sched, n, beside, alone, cu);
    o[0] = s.kernel, o[1] = s.tiles, o[2] = s.whole;
}
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("schedule")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "shim.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", so,
                           str(d / "shim.cpp")])
    return C.CDLL(so)


def split(rules, *args):
    o = (C.c_int * 3)()
    rules.split(*args, o)
    return tuple(o)


@pytest.mark.parametrize("cu", [32, 256, 304])
def test_every_size_splits_into_whole_and_parts(rules, cu):
    for n in range(1, 4 * cu):
        for sched in (FACE, COLUMN, PERSISTENT, TILED):
            for alone in (0, 1):
                kernel, tiles, whole = split(rules, sched, n, n, alone, cu)
                if kernel == 1:   # direct: a workgroup a whole block, parts for the rest, which run at once
                    assert 0 <= whole <= n and tiles in (1, 2, 3, 4, 8)
                    assert (whole == n) == (tiles == 1)
                    assert (n - whole) * tiles <= cu and whole % cu == 0 or tiles == 1
                else:
                    assert kernel == {FACE: 0, PERSISTENT: 2, TILED: 2}[sched]
                    assert tiles == (3 if sched == TILED else 1)


@pytest.mark.parametrize("cu", [32, 256, 304])
def test_table_takes_tiled_as_parts_only(rules, cu):
    """A bucket holds sizes that a winner at its smallest was not timed at:
    where parts no longer fit at once the launch is whole leaves, never the
    queue of axis items."""
    table = (C.c_int32 * 16)(*[TILED] * 16)
    for n in range(1, 4 * cu):
        s = rules.table(table, n, n, cu)
        assert s == (TILED if 2 * n <= cu else COLUMN), n
        assert split(rules, s, n, n, 1, cu)[0] == 1
    for other in (FACE, COLUMN, PERSISTENT):
        table = (C.c_int32 * 16)(*[other] * 16)
        assert {rules.table(table, n, n, cu) for n in range(1, 4 * cu)} == {other}


@pytest.mark.parametrize("cu", [32, 256, 304])
def test_launches_side_by_side_share_the_chip(rules, cu):
    """Equal launches on up to four streams: their parts fit at once as far as
    blocks_beside says how many run, and small launches go in parts however
    many of them a stage has."""
    for n in range(1, cu):
        for nlaunch in (1, 2, 3, 4, 5, 16, 60):
            streams = min(4, nlaunch)
            beside = rules.beside(n, n * nlaunch, nlaunch, streams)
            assert max(n, 4 * n * streams // 5) <= beside <= n * streams
            sched = rules.automatic(beside, cu)
            assert (sched == TILED) == (2 * beside <= cu)
            kernel, tiles, whole = split(rules, sched, n, beside, int(streams == 1), cu)
            assert kernel == 1 and (whole, tiles) == (n, 1) if sched == COLUMN else tiles * beside <= cu
            kernel, tiles, whole = split(rules, TILED, n, beside, int(streams == 1), cu)
            assert kernel == (1 if 2 * n <= cu else 2) and tiles >= 2
    assert rules.beside(10, 600, 60, 4) == 32 and rules.automatic(32, 256) == TILED   # was whole leaves
    assert split(rules, TILED, 32, rules.beside(32, 128, 4, 4), 0, 256)[1] == 2       # was eight parts
