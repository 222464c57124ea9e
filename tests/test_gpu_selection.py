"""Parent selection on both sides of the lines between its forms."""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_kernel_shapes import F32, F64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import paper_2001_04931_amd as E

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    E.lib()
    return E


# (population, parents): the short cut's last count and the first that runs the
# histogram passes alone, with two, three and four full wavefronts of 256
# threads and with 1024 threads; one line without the other's condition (more
# than 16 minima per wavefront past 16384 costs)
@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("pop,k", [(257, 32), (257, 33), (1000, 48), (1000, 49), (1024, 64),
                                   (1024, 65), (1024, 129), (4097, 96), (4097, 97), (16384, 96),
                                   (16384, 97), (16385, 256), (65537, 256)])
def test_selection_either_side_of_the_short_cut(oracle_lib, E, pop, k, dtype):
    """Spread costs, the lowest in one thread's range, ties at the threshold: the
    indices are exact."""
    from test_gpu_parity import gpu_generation

    prob = W.linear_chain(2, 10, 3, seed=0)
    ga = W.GA(pop=pop, n_elite=k, generations=1, sigma=0.1, seed=1)
    rng = np.random.default_rng(pop + k)
    spread = rng.normal(0, 1, pop).astype(np.float32).astype(np.float64)
    knots = W.draw_knots(prob, pop, 1)
    for cost in (spread, np.sort(spread), np.round(spread, 1)):
        _, eidx, best = gpu_generation(E, prob, ga, knots, cost, 0, 0, dtype)
        want_idx, want_best = oracle_lib.select(cost, k)
        np.testing.assert_array_equal(eidx, want_idx)
        assert best == want_best


@pytest.mark.parametrize("pop,k", [(256, 64), (256, 65), (1000, 48), (1000, 49), (2048, 64),
                                   (2048, 65)])
def test_batched_selection_either_side_of_the_short_cut(E, pop, k):
    """A batch's ticks equal the single solver's, parents and costs included: the
    same streams, the same costs, the same order of parents."""
    prob = W.linear_chain(2, 20, 5, seed=3).cast(np.float32)
    ga = W.GA(pop=pop, n_elite=k, generations=3, sigma=0.1, seed=11)
    x0 = torch.as_tensor(W.draw_x0(prob.n, 1), dtype=F32).cuda()
    dp = E.DeviceProblem(prob, F32)
    single = E.Solver(dp, ga)
    batch = E.BatchSolver([dp], ga, autotune=False)
    batch.set_x0(0, x0)
    for tick in range(2):
        u, J = single.solve(x0, tick)
        bu, bJ = batch.solve()
        assert torch.equal(bJ.cpu(), J.cpu()) and torch.equal(bu.cpu(), u.cpu())
