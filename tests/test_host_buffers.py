"""The buffers that follow a mesh's size (csrc/host_buffers.h, built here with
g++ over a pretended card, tests/host/buffers_driver.cpp): growing takes an
eighth more, a smaller size keeps the buffer, and where the slack is what a
later buffer lacks, giving it back serves every size that exact buffers would
have: all buffers released and asked for again (a mesh change), or trimmed
with their contents kept (the stage buffers of a step)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
GXX = shutil.which("g++")
SLACK = (32 << 20) // 8


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if GXX is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("bufdrv") / "buffers_driver")
    subprocess.run([GXX, "-O2", "-std=c++17", os.path.join(HERE, "host", "buffers_driver.cpp"), "-o", exe],
                   check=True, capture_output=True)
    return exe


def run(exe, card, *cmds):
    out = subprocess.run([exe], input="%d\n%s\n" % (8 * card, "\n".join(cmds)), capture_output=True, text=True,
                         check=True).stdout
    rows = [tuple(map(int, l.split())) for l in out.splitlines()]
    assert len(rows) == len(cmds) and all(r[4] for r in rows)
    return [(bool(r[0]), r[1], r[2], r[3] // 8) for r in rows]


def test_grow_keep_and_replace(driver):
    r = run(driver, 10 ** 9, "mesh 0 1000", "mesh 0 1100", "mesh 0 900", "mesh 0 1238", "mesh 0 0",
            "mesh 1 40000000", "mesh 1 40000001", "mesh 1 39000000", "mesh 1 38000000")
    assert r == [(True, 1000, 1000, 1000), (True, 1100, 1237, 1237), (True, 900, 1237, 1237),
                 (True, 1238, 1238 + 154, 1392), (True, 0, 0, 0),
                 (True, 40000000, 40000000, 40000000), (True, 40000001, 40000001 + SLACK, 40000001 + SLACK),
                 (True, 39000000, 39000000, 39000000),
                 (True, 38000000, 39000000, 39000000)]


def test_slack_is_given_back(driver):
    first = ["mesh %d 8000" % i for i in range(4)]
    # 4 x 9,000 elements fit a card of 36,100 exactly, not with an eighth more each
    grown = ["mesh %d 9000" % i for i in range(4)]
    r = run(driver, 36100, *first, *grown, *["free %d" % i for i in range(4)], *grown)
    assert not all(x[0] for x in r[4:8])
    assert r[-4:] == [(True, 9000, 9000, 9000 * (k + 1)) for k in range(4)]


def test_trimmed_with_contents(driver):
    # three grown buffers hold 3 x 10,125; two of 10,000 need the slack
    cmds = ["mesh %d %d" % (i, n) for n in (8000, 9000) for i in range(3)]
    r = run(driver, 47100, *cmds, "exact 3 10000", "exact 4 10000", "free 3", "trim 0", "trim 1", "trim 2",
            "exact 3 10000", "exact 4 10000")
    assert not r[7][0]
    assert [x[1:3] for x in r[9:12]] == [(9000, 9000)] * 3
    assert r[-2:] == [(True, 10000, 10000, 37000), (True, 10000, 10000, 47000)]
    # no room for a copy: the buffer stays as it is
    r = run(driver, 10125, "mesh 0 8000", "mesh 0 9000", "trim 0")
    assert r[-1] == (True, 9000, 10125, 10125)
