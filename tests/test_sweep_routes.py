"""The library's host side without a GPU: tests/host/sweep_routes.cpp compiles
it over a runtime that launches nothing and notes what it is asked to launch."""
import os
import subprocess

import pytest

from paper_2306_01301_amd import build as hip_build
from paper_2306_01301_amd import planner as P

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "sweep_routes")
    src = [os.path.join(HERE, "host", "sweep_routes.cpp")] + [
        os.path.join(hip_build.CSRC, f) for f in ("nhp_api.cpp", "nhp_batch.cpp", "nhp_tables.cpp")]
    subprocess.check_call([CLANG, "-x", "c++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I" + hip_build.INCLUDE, "-I" + hip_build.CSRC] + src + ["-o", exe])

    def run(what):
        out = subprocess.run([exe, what], capture_output=True, text=True, timeout=60)
        assert out.returncode == 0, out.stdout + out.stderr
        return dict(line.split(": ", 1) for line in out.stdout.splitlines())

    return run


def test_a_failed_launch_leaves_no_tiles_in_the_next_list(ask):
    got = ask("failed_list_launch")
    assert got.pop("wrong") == "nothing"
    assert got == {"failure at launch %d" % k: "t %d 0 t" % P.EHIP for k in range(6)}


def test_back_tracking_waits_for_workgroups_that_start_late(ask):
    # six workgroups wait for one another; long kernels of other streams may
    # hold some of them up for seconds
    assert int(ask("extract_wait")["milliseconds at 2.4 GHz"]) >= 14000


def test_a_repeated_shared_call_is_found_by_words(ask):
    # 256 plans of 32^2 x 16: looking the launches up must not take longer than
    # going through the job table byte by byte
    got = ask("repeated_call")
    assert got["route"] == "f" and got["faster than its table's bytes"] == "yes"


def test_shared_launches_are_tracked_where_that_pays(ask):
    """t: only the tiles that changes have reached, f: all tiles.  2^24 poses each."""
    got = ask("shared_launches")
    assert got == {
        "four, 7 cycles": "ttttttt",
        "then one alone": "t",  # after 6 cycles
        "four, 5 cycles": "ttttt",
        "then one alone, then all": "f f",
        "two": "ff",
        "with a small one": "f",
        "sweep of four, 1 cycle": "t",
        "sweep of two, 7 and 8 cycles": "f t",
        "sweep of one, 15 and 16 cycles": "f t",
        "four, one handed out": "fff",
        "sweep of four, one handed out": "t",  # (a sweep starts from its own volume)
        "four more, one handed out": "ff",
        "wrong": "nothing",
    }


def test_whole_sweeps_are_tracked_where_that_pays(ask):
    """As above, at three numbers of cycles each."""
    got = ask("whole_sweeps")
    assert got == {"1024x64": "f f t", "1024x128": "f f t", "720x136": "t t t", "512x256": "t t t", "512x248": "f f f",
                   "wrong": "nothing"}


def test_row_workgroups_fit_side_by_side(ask):
    # by waves per workgroup, 1 to 16; two, not three, of 10 waves
    got = ask("row_workgroups")
    assert got["8 steps"] == "32 16 10 8 6 5 4 4 3 2 2 2 2 2 2 2"
    assert got["32 steps"] == "16 8 5 4 3 2 2 2 1 1 1 1 1 1 1 1"


def test_resumes_are_tracked_where_that_pays(ask):
    got = ask("resumes")
    assert got == {
        "after 2, 5 more": "t f",
        "after 2, 6 more, 1 more": "t t t",
        "after one maneuver, 7 more, 8 more": "f t",
        "after 0, 0, 3 more": "- - t",  # (still from the start)
        "after one maneuver and 0, 1 more": "f",
        "handed out, 9, 1 more, 8 more": "t f t",
        "few headings, after 12, 1 more": "t t",
        "after 11, 11 more, 12 more": "f f t",
        "64-step sections, after 12, 12 more": "t f",
        "wrong": "nothing",
    }
