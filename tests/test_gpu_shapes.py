"""Launch shapes of the kernels at their edges, against the oracle, bit for
bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_01301_amd import planner as P
from paper_2306_01301_amd import scenes
from tests.common import problem_of

pytestmark = pytest.mark.gpu

HARD = 255


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P.lib()


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# one word per row and many rows per workgroup; idle lanes in the last wave of
# sections; word counts that are no power of two; the sides on both sides of
# each thread count of the straight kernel; one to many waves of sections
@pytest.mark.parametrize("n,nt", [(32, 8), (32, 512), (64, 24), (96, 200), (160, 72), (192, 40), (320, 16), (352, 88),
                                  (480, 24), (512, 104)])
def test_reach_shapes_match_oracle(n, nt):
    print("reach %d x %d" % (n, nt), flush=True)
    cycles = 2
    sc = scenes.random_small(n + nt, n=n, nt=nt, R=4.0, n_rect=max(3, n // 10)).with_(vehicle=(2, 1, 1))
    prob = problem_of(sc)
    B = oracle.render(prob, sc.image, *sc.vehicle)
    free = np.argwhere(B != HARD)
    T, j, i = (int(v) for v in free[len(free) // 3])
    pl = P.planner_for(sc)
    rc = P.Reach(pl, cycles)
    rc.render(_dev(sc.image), sc.vehicle)
    rc.sweep((i, j, T), cycles)
    torch.cuda.synchronize()
    got = P.bits_to_levels([rc.level_words(m).cpu().numpy().view(np.uint32) for m in range(cycles + 1)], B.shape)
    assert np.array_equal(got, oracle.reach(prob, B, (i, j, T), cycles))
    rc.close()
    pl.close()


# tables on both sides of what travels in the kernel arguments, of a squared
# and of no squared radius; sides that leave a short bit word
@pytest.mark.parametrize("n", [16, 40, 264, 1024])
@pytest.mark.parametrize("length", [1, 2, 3, 17, 3072, 3073, 65536])
def test_soft_cost_tables_match_oracle(n, length):
    rng = np.random.default_rng(n + length)
    img = rng.integers(0, 255, (n, n)).astype(np.uint8)
    img[rng.random((n, n)) < 0.002] = HARD
    img[:, n // 2] = 3  # a column without hard pixels
    table = rng.integers(0, 255, length).astype(np.uint8)
    p = P.planner_for(scenes.free_space(n, 8, 2.0, 1))
    assert np.array_equal(p.soft_costs(_dev(img), table).cpu().numpy(), oracle.soft_costs(img, table))
    p.close()


# words per thread of the rendering kernels: sides on both sides of each rule
# and of each divisibility, boxes with sample counts around the unrolled four,
# codes that differ in every byte
@pytest.mark.parametrize("n,nt,box", [(16, 8, (0, 0, 0)), (120, 8, (3, 1, 1)), (128, 16, (2, 1, 2)), (136, 8, (4, 0, 1)),
                                      (248, 8, (9, 3, 4)), (256, 24, (40, 11, 9)), (264, 16, (5, 2, 1)),
                                      (272, 8, (255, 0, 255)), (512, 8, (7, 2, 2)), (1000, 8, (30, 7, 9))])
def test_render_shapes_match_oracle(n, nt, box):
    print("render %d x %d %s" % (n, nt, box), flush=True)
    rng = np.random.default_rng(n + nt)
    sc = scenes.free_space(n, nt, 2.0, 1, half_cell=1)
    img = rng.integers(0, 256, (n, n)).astype(np.uint8)
    img[rng.random((n, n)) < 0.9] = 0
    p = P.planner_for(sc)
    p.render(_dev(img), box)
    assert np.array_equal(p.cspace_numpy(), oracle.render(problem_of(sc), img, *box))
    p.close()


# straight launches of few tiles (64-column chunks): sides that leave chunks of
# 8 to 56 columns, one tile per row and several, and the first side above
@pytest.mark.parametrize("n,nt", [(64, 8), (72, 24), (120, 16), (136, 16), (248, 8), (264, 40), (512, 96), (448, 120), (448, 136)])
def test_straight_chunks_match_oracle(n, nt):
    rng = np.random.default_rng(n * 3 + nt)
    sc = scenes.random_small(n + nt, n=n, nt=nt, R=3.0, n_rect=max(2, n // 8)).with_(vehicle=(3, 1, 1))
    prob = problem_of(sc)
    B = oracle.render(prob, sc.image, *sc.vehicle)
    p = P.planner_for(sc)
    p.set_cspace(_dev(B))
    for mu in (oracle.SF, oracle.SB):
        print("straight %d x %d mu=%d" % (n, nt, mu), flush=True)
        V = rng.integers(0, 1 << 24, size=B.shape, dtype=np.uint64).astype(np.uint32)
        V[rng.random(B.shape) < 0.3] = 0xFFFFFFFF
        p.value.copy_(_dev(V.view(np.int32)))
        p.sweep_one(mu)
        oracle.sweep(prob, mu, B, V)
        assert np.array_equal(p.value_numpy(), V)
    p.close()


# straight passes over volumes in which few values change: chunks and sections
# with and without a change side by side, with one and two band buffers and with
# workgroups that walk several tiles
@pytest.mark.parametrize("knobs", [{}, {"xmajor_buffers": 2, "xmajor_wg_per_cu": 1}, {"xmajor_wg_per_cu": 1}])
@pytest.mark.parametrize("n,nt", [(40, 16), (136, 24), (200, 264), (512, 128)])
def test_sparse_changes_match_oracle(n, nt, knobs):
    print("sparse %d x %d %s" % (n, nt, knobs), flush=True)
    rng = np.random.default_rng(n + nt)
    sc = scenes.random_small(n + nt, n=n, nt=nt, R=3.0, n_rect=max(2, n // 8)).with_(vehicle=(3, 1, 1))
    prob = problem_of(sc)
    B = oracle.render(prob, sc.image, *sc.vehicle)
    p = P.planner_for(sc)
    p.set_cspace(_dev(B))
    V = rng.integers(0, 1 << 24, size=B.shape, dtype=np.uint64).astype(np.uint32)
    V[B == HARD] = 0xFFFFFFFF
    free = np.flatnonzero(B != HARD)
    try:
        for name, value in knobs.items():
            P.set_knob(P.KNOBS[name], value)
        for mu in (oracle.SF, oracle.SB):
            oracle.sweep(prob, mu, B, V)
            some = rng.choice(free, max(1, len(free) // 5000), replace=False)
            V.reshape(-1)[some] //= 4
            p.value.copy_(_dev(V.view(np.int32)))
            p.sweep_one(mu)
            oracle.sweep(prob, mu, B, V)
            assert np.array_equal(p.value_numpy(), V)
    finally:
        for name in knobs:
            P.set_knob(P.KNOBS[name], 0)
        P.apply_tuning()
        p.close()


# both sides of each thread count of the back-tracking workgroups, the longest
# curves, one maneuver and all six: a plan's cooperating workgroups against the
# batched kernel's one, over many goals in turn (reached, unreached, the start)
@pytest.mark.parametrize("n,nt,schedule", [
    (16, 8, scenes.DEFAULT_SCHEDULE), (200, 72, scenes.DEFAULT_SCHEDULE), (256, 256, scenes.DEFAULT_SCHEDULE),
    (264, 40, scenes.DEFAULT_SCHEDULE), (64, 512, scenes.DEFAULT_SCHEDULE), (64, 520, scenes.DEFAULT_SCHEDULE),
    (1024, 16, scenes.DEFAULT_SCHEDULE), (32, 1024, scenes.DEFAULT_SCHEDULE), (72, 64, scenes.FORWARD_SCHEDULE),
    (72, 64, (P.SF,)), (72, 64, (P.RB,))])
def test_extract_workgroups_agree(n, nt, schedule):
    print("extract %d x %d" % (n, nt), flush=True)
    rng = np.random.default_rng(n + nt)
    sc = scenes.random_small(n, n=n, nt=nt, R=max(2.0, n / 16), n_rect=6).with_(
        vehicle=(2, 1, 1), start=(n // 2, n // 3, nt // 5), schedule=tuple(schedule))
    img = sc.image.copy()
    img[n // 3 - 4:n // 3 + 5, n // 2 - 4:n // 2 + 5] = 0
    pl, batch = P.planner_for(sc), P.Batch(1)
    pl.render(_dev(img), sc.vehicle)
    pl.sweep(sc.start, 3)
    reached = np.argwhere(pl.value.cpu().numpy().view(np.uint32) != 0xFFFFFFFF)[:, ::-1]
    assert len(reached) > 1
    for r in range(24):
        goal = rng.integers(0, (n, n, nt)) if r % 2 else reached[rng.integers(len(reached))]
        goal = sc.start if r == 5 else tuple(int(v) for v in goal)
        radius = int(rng.integers(0, 4))
        want = batch.extract([pl], [goal], [radius], [1024], [700])[0]
        for call in (pl.extract, pl.extract_noalloc):
            try:
                got = call(goal, radius, 1024, 700)
            except P.NhpError as e:
                got = e.rc
            assert got == want
        assert r % 2 or not isinstance(want, int)
    batch.close()
    pl.close()


# the last sides of two x-major tiles per compute unit (64-column chunks) and the
# first of more: 456, 510, 516 and 540 tiles
@pytest.mark.parametrize("n,nt", [(256, 224), (320, 200), (128, 512), (328, 176)])
def test_straights_around_two_tiles_per_unit_match_oracle(n, nt):
    test_straight_chunks_match_oracle(n, nt)
