"""FP32 costs with full weights: how exact they are (shapes and options are
covered elsewhere)."""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_kernel_shapes import F32, dev, spd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import paper_2001_04931_amd as E

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    E.lib()
    return E


def cost_error(oracle_lib, E, prob, x0, knots, ncand):
    """Relative errors of the FP32 costs against the FP64 oracle's."""
    cost = dev(np.full(ncand, np.nan), F32)
    E.empc_rollout_cost(E.DeviceProblem(prob, F32), dev(x0, F32), dev(knots, F32), ncand, ncand,
                        cost)
    want = oracle_lib.rollout_cost(prob, x0, knots, ncand)
    return cost.cpu().numpy().astype(np.float64) / want - 1.0


@pytest.mark.parametrize("n,m", [(14, 7), (16, 8)])
def test_stage_costs_are_summed_per_state_row(oracle_lib, E, n, m):
    """400 steps, a knot every other one, |A| = 0.5: the states stay equally large
    and their own rounding does not build up (below 0.5e-7 of the cost).  A
    running sum of N equal positive terms has a relative error of u sqrt(N / 3)
    rms (u = 2^-24 / sqrt(3), the rms rounding of an addition): summed per row
    (N = T), n rows averaging, 1.1e-7; over the four rows of a lane (N = 4 T),
    four lanes averaging, up to 3.9e-7.  The bound is sqrt(1.1^2 + 0.5^2) with a
    quarter to spare."""
    T, p, ncand = 400, 200, 512
    rng = np.random.default_rng(n)
    A = rng.normal(0, 1, (n, n))
    A *= 0.5 / np.linalg.norm(A, 2)
    off = rng.uniform(-0.02, 0.02, (n, n))
    prob = W.Problem(model=W.LINEAR, n=n, m=m, T=T, p=p, Ad=A, Bd=rng.normal(0, 0.3, (n, m)),
                     q=np.ones(n), r=np.full(m, 0.01), qf=np.zeros(n), x_goal=np.zeros(n),
                     u_goal=np.zeros(m), u_min=-np.ones(m), u_max=np.ones(m),
                     Q=np.eye(n) + off + off.T).cast(np.float32)
    x0 = W.draw_x0(n, 4, scale=1.0).astype(np.float32).astype(np.float64)
    knots = W.draw_knots(prob, ncand, 3).astype(np.float32).astype(np.float64)
    err = cost_error(oracle_lib, E, prob, x0, knots, ncand)
    assert np.sqrt(np.mean(err**2)) < 1.5e-7


@pytest.mark.parametrize("n", [3, 7, 16, 20, 40, 64])
def test_terminal_cost_near_a_distant_goal(oracle_lib, E, n):
    """One step that leaves the state where it is, one to three units from a goal
    4096 away from the origin, both held exactly by FP32.  The cost of x_T - g
    is a sum of n^2 terms, each rounded a few times: n + 4 units in the last
    place of the sum of their sizes at most.  Q x_T - Q g would be off by about
    4096 units in the last place of Q."""
    rng = np.random.default_rng(n)
    Q = spd(n, rng)
    g = rng.choice([-4096.0, 4096.0], n)
    prob = W.Problem(model=W.LINEAR, n=n, m=1, T=1, p=1, Ad=np.eye(n), Bd=np.zeros((n, 1)),
                     q=np.ones(n), r=np.ones(1), qf=np.zeros(n), x_goal=g, u_goal=np.zeros(1),
                     u_min=-np.ones(1), u_max=np.ones(1), Q=Q, Qf=0.3 * Q).cast(np.float32)
    x0 = g + rng.integers(1, 4, n)
    e = x0 - g
    size = np.abs(e) @ np.abs(prob.Q + prob.Qf) @ np.abs(e) / (e @ (prob.Q + prob.Qf) @ e)
    err = cost_error(oracle_lib, E, prob, x0, np.zeros((1, 20)), 20)
    assert np.abs(err).max() <= (n + 4) * 2.0**-24 * size


@pytest.mark.parametrize("n,m", [(14, 7), (42, 21), (64, 32)])
def test_states_of_slow_dynamics(oracle_lib, E, n, m):
    """200 steps of A = I + N with |N| <= 0.02 and Q close to I: the increments are
    small, so a step that adds the state's own row last rounds once by the
    state's size.  The error of a state is then a random walk of u = 2^-24 /
    sqrt(3) a step, its mean over the steps u sqrt(T / 3), and the cost's, with n
    rows averaging, 2 u sqrt(T / (3 n)); the sums of the stage costs add half of
    that.  The bound is sqrt(1 + 1/4) of it with half to spare (state sizes are not
    all alike).  With the own row's term first, the n / 2 terms after it each
    round by the state's size as well."""
    T, p, ncand = 200, 20, 512
    rng = np.random.default_rng(n)
    N = rng.normal(0, 1, (n, n))
    N = 0.01 * (N - N.T) / np.linalg.norm(N, 2)
    off = rng.uniform(-0.02, 0.02, (n, n)) / n
    prob = W.Problem(model=W.LINEAR, n=n, m=m, T=T, p=p, Ad=np.eye(n) + N,
                     Bd=rng.normal(0, 1e-3, (n, m)), q=np.ones(n), r=np.full(m, 1e-3),
                     qf=np.zeros(n), x_goal=np.zeros(n), u_goal=np.zeros(m), u_min=-np.ones(m),
                     u_max=np.ones(m), Q=np.eye(n) + off + off.T).cast(np.float32)
    knots = W.draw_knots(prob, ncand, 3).astype(np.float32).astype(np.float64)
    err = []
    for seed in range(4):
        x0 = (1.5 * W.draw_x0(n, seed, scale=1.0)).astype(np.float32).astype(np.float64)
        err.append(cost_error(oracle_lib, E, prob, x0, knots, ncand))
    u = 2.0**-24 / np.sqrt(3)
    assert np.sqrt(np.mean(np.square(err))) < 1.5 * np.sqrt(1.25) * 2 * u * np.sqrt(T / (3 * n))


def test_stage_cost_near_a_distant_goal(oracle_lib, E):
    """The same for the stage costs of a single tile: 20 steps that leave the state
    where it is."""
    n, T = 14, 20
    rng = np.random.default_rng(n)
    Q = spd(n, rng)
    g = rng.choice([-4096.0, 4096.0], n)
    prob = W.Problem(model=W.LINEAR, n=n, m=1, T=T, p=1, Ad=np.eye(n), Bd=np.zeros((n, 1)),
                     q=np.ones(n), r=np.ones(1), qf=np.zeros(n), x_goal=g, u_goal=np.zeros(1),
                     u_min=-np.ones(1), u_max=np.ones(1), Q=Q).cast(np.float32)
    x0 = g + rng.integers(1, 4, n)
    e = x0 - g
    size = np.abs(e) @ np.abs(prob.Q) @ np.abs(e) / (e @ prob.Q @ e)
    err = cost_error(oracle_lib, E, prob, x0, np.zeros((1, 20)), 20)
    assert np.abs(err).max() <= (n + T + 4) * 2.0**-24 * size
