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
int table(const int32_t *t, int n, int cu) { return table_schedule(t, n, cu); }
void split(int sched, int n, int alone, int cu, int *o) {
    const Split s = split_launch(sched, n, alone, cu);
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
                kernel, tiles, whole = split(rules, sched, n, alone, cu)
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
        s = rules.table(table, n, cu)
        assert s == (TILED if 2 * n <= cu else COLUMN), n
        assert split(rules, s, n, 1, cu)[0] == 1
    for other in (FACE, COLUMN, PERSISTENT):
        table = (C.c_int32 * 16)(*[other] * 16)
        assert {rules.table(table, n, cu) for n in range(1, 4 * cu)} == {other}
