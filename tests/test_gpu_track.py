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
    return scenes.Scene("t", n, nt, 9.0, img, (3, 1, 1) if n >= 32 else (0, 0, 0), (i, j, nt // 5), (0, 0, 0), 0, ct=scenes.uniform_ct(18),
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


def _mixed_plans(extra=()):
    """Plans of every section size and both grid kinds, over 2^24 poses together."""
    scs = [_scene(n, nt, 3 * n + nt, sched) for n, nt, sched in
           ((128, 128, FULL), (200, 72, FULL), (256, 256, FULL), (64, 512, (LF, SF, RF)), (384, 128, FULL),
            (72, 1000, (RB, RF, SF)), (96, 64, FULL)) + tuple(extra)]
    ps = [P.planner_for(sc) for sc in scs]
    for p, sc in zip(ps, scs):
        p.render(torch.from_numpy(sc.image).cuda(), sc.vehicle)
    return scs, ps


def _in_full(scs, cycles, edit=None):
    """The volumes after every pass run by itself (edit: (after cycles, change))."""
    out = []
    for sc, n in zip(scs, cycles):
        p = P.planner_for(sc)
        p.render(torch.from_numpy(sc.image).cuda(), sc.vehicle)
        p.sweep(sc.start, 0)
        if edit:
            _passes(p, sc.schedule, edit[0])
            edit[1](p)
            for a, b in P.schedule_passes(sc.schedule, edit[0] * len(sc.schedule), n * len(sc.schedule)):
                p.sweep_pass(a, b)
        else:
            _passes(p, sc.schedule, n)
        out.append(p.value.clone())
        p.close()
    return out


@pytest.mark.parametrize("extra", [(), ((16, 24, FULL),)])  # (a side under 32 leaves all of them untracked)
def test_tracked_batch_sweep_equals_every_pass_in_full(extra):
    scs, ps = _mixed_plans(extra)
    cycles = [3 + k % 4 for k in range(len(scs))]
    want = _in_full(scs, cycles)
    b = P.Batch(len(scs))
    for _ in range(2):
        b.sweep(ps, [sc.start for sc in scs], cycles)
    for p, w, sc in zip(ps, want, scs):
        _same(p, w, (sc.nx, sc.nt))
    b.close()
    for p in ps:
        p.close()


def test_tracked_batch_goes_on_over_calls():
    """Calls that go on from the last one's volumes, some plans sitting one
    out, then resumed by themselves and in the batch again."""
    scs, ps = _mixed_plans()
    b = P.Batch(len(scs))
    b.init(ps, [sc.start for sc in scs])
    done = [0] * len(scs)
    for call in range(5):
        counts = [0 if (k + call) % 5 == 0 else len(sc.schedule) * (1 + (k + call) % 2) for k, sc in enumerate(scs)]
        b.advance(ps, done, counts)
        done = [d + c for d, c in zip(done, counts)]
    torch.cuda.synchronize()
    for p in ps:
        p.resume(2)
    torch.cuda.synchronize()
    b.advance(ps, [0] * len(ps), [2 * len(sc.schedule) for sc in scs])
    cycles = [d // len(sc.schedule) + 4 for d, sc in zip(done, scs)]
    # (plain passes pair turns across cycles as one run does: the volumes are those of the sweeps one by one)
    want = _in_full(scs, cycles)
    for p, w, sc in zip(ps, want, scs):
        _same(p, w, (sc.nx, sc.nt))
    b.close()
    for p in ps:
        p.close()


def test_volumes_written_between_batch_calls():
    """A caller that has a volume's address may write it between two calls."""
    def change(p):
        p.value[2, 3:40, 5:50] = 1 << 18

    scs, ps = _mixed_plans()
    want = _in_full(scs, [3] * len(scs), (2, change))
    b = P.Batch(len(scs))
    b.init(ps, [sc.start for sc in scs])
    b.advance(ps, [0] * len(ps), [2 * len(sc.schedule) for sc in scs])
    for p in ps:
        change(p)
    b.advance(ps, [2 * len(sc.schedule) for sc in scs], [3 * len(sc.schedule) for sc in scs])
    for p, w, sc in zip(ps, want, scs):
        _same(p, w, (sc.nx, sc.nt))
    b.close()
    for p in ps:
        p.close()


def test_tracked_resume_of_a_volume_nobody_has_seen():
    sc = _scene(512, 256, 9, FULL)
    want = _in_full([sc], [5])[0]
    p = P.planner_for(sc)
    p.render(torch.from_numpy(sc.image).cuda(), sc.vehicle)
    p.sweep(sc.start, 2)
    p.resume(1)
    p.resume(2)
    _same(p, want, "resume")
    # a pass run by itself in between is not tracked
    q = P.planner_for(sc)
    q.render(torch.from_numpy(sc.image).cuda(), sc.vehicle)
    q.sweep(sc.start, 2)
    for mu in FULL:
        q.sweep_one(mu)
    q.resume(2)
    _same(q, want, "resume after single passes")
    p.close()
    q.close()


def test_captured_sweeps_between_eager_ones():
    """A sweep captured into a graph, not run, then run after other sweeps:
    every sweep goes on from what the volume holds when it runs."""
    sc = _scene(512, 256, 5, FULL)
    stream = torch.cuda.Stream()
    p = P.planner_for(sc, stream=stream)
    with torch.cuda.stream(stream):
        image = torch.from_numpy(sc.image).cuda()
    p.render(image, sc.vehicle)
    p.sweep(sc.start, 2)
    graph = torch.cuda.CUDAGraph()
    print("capture", flush=True)
    with torch.cuda.graph(graph, stream=stream):
        p.resume(1)
    p.resume(1)
    with torch.cuda.stream(stream):
        graph.replay()
    p.resume(1)
    stream.synchronize()
    got = p.value.clone()
    torch.cuda.synchronize()  # (the copy is on another stream than the plan's)
    p.sweep(sc.start, 0)
    _passes(p, FULL, 5)
    stream.synchronize()
    assert torch.equal(got, p.value)
    p.close()


# ---- what is known of a volume when a call goes on from it ----

@pytest.mark.parametrize("how", ["one plan", "batch"])
def test_zero_cycle_resume_knows_no_more_than_before(how):
    """resume(0) after passes that kept no record of their changes."""
    if how == "one plan":
        # a maze, in which every cycle still reaches new poses
        sc = _scene(512, 256, 11, FULL).with_(image=scenes.maze(np.random.default_rng(11), 16, 32, 4), start=(18, 18, 0))
        want = _in_full([sc], [9])[0]
        p = P.planner_for(sc)
        p.render(torch.from_numpy(sc.image).cuda(), sc.vehicle)
        p.sweep(sc.start, 7)
        for mu in FULL:
            p.sweep_one(mu)
        p.resume(0)
        p.resume(1)
        _same(p, want, "resume")
        p.close()
        return
    scs = [_scene(256, 256, 20 + k, FULL) for k in range(4)]
    want = _in_full(scs, [5] * 4)
    ps = [P.planner_for(sc) for sc in scs]
    for p, sc in zip(ps, scs):
        p.render(torch.from_numpy(sc.image).cuda(), sc.vehicle)
        p.sweep(sc.start, 3)
        p.resume(0)
    torch.cuda.synchronize()
    b = P.Batch(4)
    b.advance(ps, [18] * 4, [12] * 4)
    for p, w in zip(ps, want):
        _same(p, w, "batch")
    b.close()
    for p in ps:
        p.close()


@pytest.mark.parametrize("kind", ["set_cspace", "render", "batch render", "batch step"])
def test_captured_changes_between_eager_sweeps(kind):
    """A call that changes a plan's volumes, captured into a graph and run
    between two sweeps: the second goes on from what the volumes then hold."""
    sc = _scene(512, 256, 7, FULL)
    stream = torch.cuda.Stream()
    p, q = P.planner_for(sc, stream=stream), P.planner_for(sc, stream=stream)
    batches = {p: P.Batch(1, stream=stream), q: P.Batch(1, stream=stream)}
    with torch.cuda.stream(stream):
        image, clear = torch.from_numpy(sc.image).cuda(), torch.zeros(512, 512, dtype=torch.uint8, device="cuda")
        codes = torch.zeros(sc.nt, sc.nx, sc.nx, dtype=torch.uint8, device="cuda")
    change = {"set_cspace": lambda x: x.set_cspace(codes), "render": lambda x: x.render(clear, sc.vehicle),
              "batch render": lambda x: batches[x].render([x], [clear], [sc.vehicle]),
              "batch step": lambda x: [batches[x].step([x], [k]) for k in range(4)]}[kind]
    # what it comes to, every pass in full
    q.render(image, sc.vehicle)
    q.sweep(sc.start, 0)
    _passes(q, FULL, 7)
    change(q)
    _passes(q, FULL, 1)
    p.render(image, sc.vehicle)
    p.sweep(sc.start, 1)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    print("capture", kind, flush=True)
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="relaxed"):
        change(p)
    p.render(image, sc.vehicle)
    p.sweep(sc.start, 7)
    with torch.cuda.stream(stream):
        graph.replay()
    p.resume(1)
    stream.synchronize()
    assert torch.equal(p.value, q.value), int((p.value != q.value).sum())
    for x in (p, q):
        batches[x].close()
        x.close()


def test_views_of_a_closed_planner():
    """The volumes are in the planner's own workspace: its views outlive the plan."""
    sc = _scene(64, 64, 3, FULL)
    out = []
    for look_first in (True, False):
        p = P.planner_for(sc)
        p.render(torch.from_numpy(sc.image).cuda(), sc.vehicle)
        p.sweep(sc.start, 2)
        if look_first:
            p.value, p.cspace
        p.close()
        out.append((p.value_numpy().copy(), p.cspace_numpy().copy()))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    assert out[0][0].min() == 0 and out[0][1].max() == 255


def test_tracked_batches_of_mixed_plans_equal_every_pass_in_full():
    """At least 2^26 poses in every call, of every section size and both grid kinds."""
    scs, ps = _mixed_plans(((512, 128, FULL), (328, 256, FULL)))
    cycles = [3 + k % 4 for k in range(len(scs))]
    want = _in_full(scs, cycles)
    b = P.Batch(len(scs))
    print("sweep", flush=True)
    for _ in range(2):
        b.sweep(ps, [sc.start for sc in scs], cycles)
    for p, w, sc in zip(ps, want, scs):
        _same(p, w, (sc.nx, sc.nt))
        p.close()
    print("calls that go on from one another", flush=True)
    ps = [P.planner_for(sc) for sc in scs]
    for p, sc in zip(ps, scs):
        p.render(torch.from_numpy(sc.image).cuda(), sc.vehicle)
    b.init(ps, [sc.start for sc in scs])
    done = [0] * len(scs)
    for call in range(5):
        counts = [0 if k < 7 and (k + call) % 5 == 0 else len(sc.schedule) * (1 + (k + call) % 2) for k, sc in enumerate(scs)]
        b.advance(ps, done, counts)
        done = [d + c for d, c in zip(done, counts)]
    want = _in_full(scs, [d // len(sc.schedule) for d, sc in zip(done, scs)])
    for p, w, sc in zip(ps, want, scs):
        _same(p, w, (sc.nx, sc.nt))
        p.close()
    b.close()


@pytest.mark.parametrize("n,nt", [(1000, 72), (1024, 64), (760, 120), (736, 128)])
def test_tracked_sweeps_of_few_headings_equal_every_pass_in_full(n, nt):
    """Short sections: tracked from 12 cycles on."""
    sc = _scene(n, nt, n + nt, FULL)
    p = P.planner_for(sc)
    p.render(torch.from_numpy(sc.image).cuda(), sc.vehicle)
    p.sweep(sc.start, 0)
    _passes(p, FULL, 12)
    want = p.value.clone()
    print("tracked %s" % ((n, nt),), flush=True)
    p.sweep(sc.start, 12)
    _same(p, want, "sweep")
    i, j, T = sc.start
    starts = [(i, j, T, 700, -1), (i + 2, j, T, 100, RB), (i, j + 3, (T + 7) % nt, 0, SF), (i, j, 0, 50, LB)]
    p.sweep_from_set(starts, 0)
    _passes(p, FULL, 12)
    want.copy_(p.value)
    p.sweep_from_set(starts, 12)
    _same(p, want, "start set")
    p.close()


def test_tracked_resumes_equal_every_pass_in_full():
    """Late enough to be tracked, with stamps from before and without."""
    sc = _scene(512, 256, 15, FULL).with_(image=scenes.maze(np.random.default_rng(15), 16, 32, 4), start=(18, 18, 0))
    want = {n: _in_full([sc], [n])[0] for n in (11, 20)}
    p = P.planner_for(sc)
    p.render(torch.from_numpy(sc.image).cuda(), sc.vehicle)
    p.sweep(sc.start, 7)
    p.resume(1)
    p.resume(3)
    p.resume(0)
    for mu in FULL:
        p.sweep_one(mu)
    p.resume(8)
    _same(p, want[20], "sweep, resumes, single passes, resume")
    p.sweep(sc.start, 3)  # (its volumes have now been handed out)
    p.resume(8)
    _same(p, want[11], "resume of eight cycles")
    p.close()
    # a whole sweep, then resumes that go on from its stamps
    q = P.planner_for(sc)
    q.render(torch.from_numpy(sc.image).cuda(), sc.vehicle)
    q.sweep(sc.start, 7)
    q.resume(1)
    q.resume(3)
    _same(q, want[11], "sweep and resumes")
    q.close()
