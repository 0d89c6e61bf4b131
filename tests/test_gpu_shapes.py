"""Launch shapes of the reachability and soft-cost kernels at their edges,
against the oracle, bit for bit."""
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
