"""Sweeps that skip tiles no change has reached (volumes of at least 2^26
poses) against the same passes run one by one, which visit every tile: value
volumes bit for bit.

The sizes leave short last tiles (sides that are no multiple of 64), short
last sections, every section size (8 to 64 steps), and one to sixteen tiles per
row; the schedules pair turns, repeat a maneuver, or leave a kind out."""
import numpy as np
import pytest
import torch

from paper_2306_01301_amd import planner as P
from paper_2306_01301_amd import scenes

pytestmark = pytest.mark.gpu

LF, SF, RB, RF, SB, LB = range(6)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P.lib()


def _scene(n, nt, seed, schedule):
    rng = np.random.default_rng(seed)
    img = scenes.mixed_clutter(rng, n, 0.08)
    img = np.where(img == 255, 255, rng.integers(0, 3, img.shape) * 40).astype(np.uint8)
    i, j = n // 3, n - n // 3
    img[j - 12:j + 13, i - 12:i + 13] = 0
    return scenes.Scene("t", n, nt, 9.0, img, (3, 1, 1), (i, j, nt // 5), (0, 0, 0), 0, ct=scenes.uniform_ct(18),
                        gear=scenes.reverse_gear(320), schedule=schedule)


def _passes(p, schedule, cycles):
    for a, b in P.schedule_passes(schedule, 0, cycles * len(schedule)):
        p.sweep_pass(a, b)


def _same(p, want, what):
    got = p.value
    assert torch.equal(got, want), (what, int((got != want).sum()))


SIZES = [(512, 256), (1000, 72), (264, 1000), (720, 136), (1024, 64), (760, 120)]
FULL = (LF, SF, RB, RF, SB, LB)


@pytest.mark.parametrize("n,nt,schedule,cycles", [(n, nt, FULL, 4) for n, nt in SIZES] + [
    (520, 256, (LF, SF, RF), 4), (512, 256, (RF, RB, SF), 3), (512, 256, (SB, SF), 3), (512, 256, (LB,), 3),
    (512, 256, (LF, LB, LF, SF, SF), 3)])
def test_tracked_sweeps_equal_every_pass_in_full(n, nt, schedule, cycles):
    sc = _scene(n, nt, n + nt, schedule)
    p = P.planner_for(sc)
    p.render(torch.from_numpy(sc.image).cuda(), sc.vehicle)
    p.sweep(sc.start, 0)
    _passes(p, schedule, cycles)
    want = p.value.clone()
    print("tracked %s" % ((n, nt, schedule, cycles),), flush=True)
    p.sweep(sc.start, cycles)
    _same(p, want, "sweep")
    # resumed after the caller has written the volume: nothing is known of it
    p.sweep(sc.start, 1)
    start = p.value.clone()
    start[3, 5:n // 2, 7:n // 3] = 1 << 20
    p.value.copy_(start)
    _passes(p, schedule, 3)
    want.copy_(p.value)
    p.value.copy_(start)
    p.resume(3)
    _same(p, want, "resume")
    p.close()


@pytest.mark.parametrize("n,nt", [(512, 256), (1000, 72)])
def test_tracked_start_set_equals_every_pass_in_full(n, nt):
    sc = _scene(n, nt, 5, FULL)
    p = P.planner_for(sc)
    p.render(torch.from_numpy(sc.image).cuda(), sc.vehicle)
    i, j, T = sc.start
    starts = [(i, j, T, 700, -1), (i + 2, j, T, 100, RB), (i, j + 3, (T + 7) % nt, 0, SF), (i, j, 0, 50, LB)]
    p.sweep_from_set(starts, 0)
    _passes(p, FULL, 3)
    want = p.value.clone()
    p.sweep_from_set(starts, 3)
    _same(p, want, "start set")
    p.close()
