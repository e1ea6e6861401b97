"""The one-launch sessions under chosen schedules, on the host: the device code of
session_dev.hpp and its two single-source policies, a fiber per lane, workgroups
that start late or are held up between any two steps (tests/emu).  Distances and
totals have to equal a plain search's.  The limits between a level's forms are
lowered so that small graphs meet all of them."""
import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2208_04514_amd", "csrc")
EMU = os.path.join(ROOT, "tests", "emu")
SMALL = {"kSB = 512;": "kSB = 128;", "kClusterEdges = 32768;": "kClusterEdges = 150;",
         "kEdgesPerWg = 256;": "kEdgesPerWg = 8;", "kClusterWords = 1024;": "kClusterWords = 6;"}
RECORDS = ("constexpr unsigned kRecordLevels = 4096;", "constexpr unsigned kRecordLevels = 8;")


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    d = str(tmp_path_factory.mktemp("emu"))
    for f in os.listdir(CSRC):
        shutil.copy(os.path.join(CSRC, f), d)
    path = os.path.join(d, "session_dev.hpp")
    with open(path) as f:
        text = f.read()
    for a, b in [("constexpr int " + x, "constexpr int " + y) for x, y in SMALL.items()] + [RECORDS]:
        assert text.count(a) == 1, a
        text = text.replace(a, b)
    with open(path, "w") as f:
        f.write(text)
    exe = os.path.join(d, "session_emu")
    subprocess.run(["g++", "-x", "c++", "-std=c++17", "-O2", "-w", f"-I{EMU}", f"-I{d}",
                    f"-I{os.path.join(ROOT, 'include')}", os.path.join(EMU, "session_emu.cpp"),
                    os.path.join(EMU, "emu.cpp"), "-o", exe], check=True)

    def run(kind, first, count, jobs=4, **opts):
        args = [f"{k}={v}" for k, v in opts.items()]
        per = -(-count // jobs)

        def one(j):
            return subprocess.run([exe, kind, str(first + j * per), str(per), *args],
                                  capture_output=True, text=True, timeout=250)
        with ThreadPoolExecutor(jobs) as ex:
            for r in ex.map(one, range(jobs)):
                assert r.returncode == 0, r.stdout + r.stderr
    return run


@pytest.mark.parametrize("kind", ["hop", "weighted"])
def test_plain(emu, kind):
    emu(kind, 1, 8)


def test_member_overtaken(emu):
    """Members held up after they reported a cluster level: the cluster may have
    begun another run of levels by then, which they join with counters at zero."""
    emu("hop", 500008, 1, jobs=1, grid=34, hold=0.001, held=20000, levels=50, wide=40)
    emu("hop", 200003, 1, jobs=1, grid=34, hold=0.001, held=20000, levels=50, wide=40)
    emu("hop", 1, 16, grid=34, hold=0.001, held=20000, levels=50, wide=40)
    emu("weighted", 1, 8, grid=34, hold=0.001, held=20000, levels=40, wide=40)


@pytest.mark.parametrize("kind,small", [("hop", 40), ("hop", 0), ("weighted", 6)])
def test_long_path_before_wide_levels(emu, kind, small):
    """Levels of one workgroup, or of one cluster, for several times the wait that
    workgroups without work are given, then levels that need them."""
    emu(kind, 1, 4, grid=40, ticks=6000, path=300, levels=320, small=small, wide=400, wmax=3)


@pytest.mark.parametrize("k", [40, 100])
def test_batch(emu, k):
    emu("batch", 1, 4, grid=20, levels=40, wide=30, k=k)
    emu("batch", 1, 4, grid=20, levels=40, wide=30, k=k, hold=0.0003, held=20000)


def test_batch_goes_on_and_times_out(emu):
    """A run that stopped for more level planes goes on and a wait of its times out: it
    must not look stopped for planes again."""
    emu("batch", 1, 4, grid=20, levels=14, wide=30, stall=1)


@pytest.mark.parametrize("kind", ["hop", "weighted", "batch"])
def test_late_workgroups(emu, kind):
    """Workgroups that start while the levels run."""
    emu(kind, 1, 8, grid=40 if kind != "batch" else 20, late=0.8, levels=40)
    emu(kind, 1, 8, grid=40 if kind != "batch" else 20, late=0.8, levels=40, hold=0.0003, held=20000)


@pytest.mark.parametrize("kind", ["hop", "weighted"])
def test_late_workgroups_take_part(emu, kind):
    emu(kind, 1, 4, late=0.9, after=100000, levels=60, small=0, join=1)


def test_callers_share_the_device(emu):
    emu("callers", 0, 1, jobs=1)


@pytest.mark.parametrize("kind", ["hop", "weighted"])
def test_one_queue(emu, kind):
    emu(kind, 1, 4, stripes=1)


def test_row_of_nearly_two_to_the_31(emu):
    emu("walk", 0, 1, jobs=1)
