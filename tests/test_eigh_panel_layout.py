"""Host-only check of the kernels whose workgroups wait for one another (no GPU):
tests/eigh_panel_check.cpp, built with g++ and AddressSanitizer from the geometry header
that the kernels use, steps the exchange of the single-launch panels word by word under
random schedules and replays the sweeps of the bulge chase.

Sizes: one panel, partial last workgroups, both row counts per wave, the largest panel
(2304 trailing rows) and panels inside larger blocks; the chase around one and two tasks
per sweep and over several.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("check") / "eigh_panel_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-g", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-I",
                    os.path.join(ROOT, "paper_2603_24860_amd", "csrc"),
                    os.path.join(ROOT, "tests", "eigh_panel_check.cpp"), "-o", exe],
                   check=True, timeout=300)

    def run(*args):
        return subprocess.run([exe] + " ".join(args).split(), capture_output=True, text=True,
                              timeout=600, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    return run


def _ok(r, n):
    assert r.returncode == 0 and f"{n} checks passed" in r.stdout, r.stdout + r.stderr


@pytest.mark.parametrize("n,j0", [(97, 0), (104, 0), (105, 0), (300, 0), (300, 192), (333, 32),
                                  (1570, 0)])
def test_panel_exchange(check, n, j0):
    seeds = range(0, 8 if n < 1000 else 3)
    _ok(check(*[f"panel {n} {j0} {s} 4" for s in seeds]), len(seeds))


def test_largest_panel_in_one_workgroup(check):
    _ok(check("panel 2305 0 0 4", "panel 4000 1696 0 4"), 2)


@pytest.mark.parametrize("ring", [1, 2, 3])
def test_fewer_slots_are_caught(check, ring):
    """The exchange needs its four slots: with fewer, some schedule reads an old word,
    publishes over one that is still needed, or never ends."""
    out = [check(f"panel 300 0 {s} {ring}") for s in range(1, 9)]
    assert any(r.returncode == 1 and "FAILED" in r.stdout for r in out)


def test_layout(check):
    ns = [1, 96, 97, 128, 129, 300, 720, 1536, 1537, 2160, 2304, 2305, 2306, 4500, 16384]
    _ok(check(*[f"layout {n} 0" for n in ns], "layout 300 20", "layout 2400 5"), len(ns) + 2)


def test_chase(check):
    ns = [2, 3, 32, 33, 34, 64, 65, 66, 97, 130, 200]
    _ok(check(*[f"chase {n}" for n in ns]), len(ns))
