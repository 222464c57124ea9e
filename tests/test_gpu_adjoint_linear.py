"""Linear gradients and refinement on the matrix cores against the FP64 oracle.

Which kernel a call takes depends on the state count, the dtype and the number
of candidates; the counts here are chosen for the matrix-core kernel unless a
test says otherwise."""
import numpy as np
import pytest
import torch

import workloads as W
from test_gpu_kernel_shapes import F32, F64, dev, random_linear

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import paper_2001_04931_amd as E

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    E.lib()
    return E


def case(n, m, T, p, ncand, dtype, box=False, seed=0, x0_scale=0.5):
    """(problem, x0, knots [p m][ncand + 3]) rounded to the dtype."""
    npd = np.float64 if dtype == F64 else np.float32
    prob = random_linear(n, m, T, p, 10 * n + m + seed)
    if box:
        prob.x_min, prob.x_max = prob.x_goal - 0.3, prob.x_goal + 0.3
        prob.qb, prob.sb = np.linspace(0.5, 2.0, n), np.linspace(0.1, 0.7, n)
    prob = prob.cast(npd)
    x0 = W.draw_x0(n, 3, scale=x0_scale).astype(npd).astype(np.float64)
    knots = W.draw_knots(prob, ncand, 5, ld=ncand + 3).astype(npd).astype(np.float64)
    return prob, x0, knots


def check_grad(oracle_lib, E, prob, x0, knots, ncand, dtype):
    """FP64: 1e-9 of a column's largest entry (gradient), 1e-10 (cost); FP32:
    2e-3 and 1e-4, the rounding of T dependent steps."""
    dp, K = E.DeviceProblem(prob, dtype), dev(knots, dtype)
    dJ, cost = torch.full_like(K, float("nan")), dev(np.full(ncand + 2, np.nan), dtype)
    E.empc_grad(dp, dev(x0, dtype), K, ncand, knots.shape[1], dJ, cost)
    want, wcost = oracle_lib.grad(prob, x0, knots, ncand)
    got, gcost = dJ.cpu().numpy().astype(np.float64), cost.cpu().numpy().astype(np.float64)
    assert np.isnan(got[:, ncand:]).all() and np.isnan(gcost[ncand:]).all()
    err = np.abs(got[:, :ncand] - want[:, :ncand]).max(axis=0)
    scale = np.abs(want[:, :ncand]).max(axis=0)
    tg, tc = (1e-9, 1e-10) if dtype == F64 else (2e-3, 1e-4)
    assert (err <= tg * scale + 1e-30).all()
    np.testing.assert_allclose(gcost[:ncand], wcost, rtol=tc)
    return gcost[:ncand]


def check_refine(oracle_lib, E, prob, x0, knots, ncand, dtype, steps=3):
    """Adam steps of 0.01.  FP64: the oracle's knots and costs to 1e-9.  FP32:
    the sign of a gradient component near zero moves a knot by a whole step, so
    the knots are held against their own cost: the reported cost is the
    oracle's cost of the refined knots (1e-4) and lies below the entry cost."""
    K = dev(knots, dtype)
    entry = oracle_lib.rollout_cost(prob, x0, knots, ncand)
    C = dev(entry, dtype)
    E.empc_refine(E.DeviceProblem(prob, dtype), dev(x0, dtype), K, ncand, knots.shape[1], C, 0.01,
                  steps)
    got, gc = K.cpu().numpy().astype(np.float64), C.cpu().numpy().astype(np.float64)
    np.testing.assert_array_equal(got[:, ncand:], knots[:, ncand:])
    if dtype == F64:
        wk, wc = oracle_lib.refine(prob, x0, knots[:, :ncand].copy(), entry, lr=0.01, steps=steps)
        np.testing.assert_allclose(gc, wc, rtol=1e-9)
        np.testing.assert_allclose(got[:, :ncand], wk, rtol=0, atol=1e-9)
    else:
        np.testing.assert_allclose(gc, oracle_lib.rollout_cost(prob, x0, got, ncand), rtol=1e-4)
        moved = np.any(got[:, :ncand] != knots[:, :ncand], axis=0)
        assert moved.mean() > 0.5 and (gc[moved] <= entry[moved] * (1 + 1e-4)).all()


@pytest.mark.parametrize("n,m,ncand,dtype", [(17, 4, 20, F32), (33, 9, 40, F32), (48, 33, 16, F32),
                                             (49, 17, 530, F32), (17, 17, 530, F64),
                                             (33, 5, 515, F64)])
def test_one_step_horizon(oracle_lib, E, n, m, ncand, dtype):
    """T = 1 with several wavefronts per tile: the only step reads the other
    wavefronts' rows of x_0, which nothing may overwrite in the meantime."""
    prob, x0, knots = case(n, m, 1, 1, ncand, dtype)
    check_grad(oracle_lib, E, prob, x0, knots, ncand, dtype)
    check_refine(oracle_lib, E, prob, x0, knots, ncand, dtype)


@pytest.mark.parametrize("dtype,n,ncand", [(F32, 5, 20), (F32, 28, 20), (F64, 12, 1030),
                                           (F64, 20, 520)])
def test_cost_without_a_trace_of_the_start_state(oracle_lib, E, dtype, n, ncand):
    """A model that contracts to 1e-4 in one step: the cost sums x_1 .. x_T only,
    so x_0, whose square is 1e8 times the others', may leave no rounding in it.
    Bounds: (n + T + 20) roundings of positive terms; half a unit in the last
    place of x_0's square would be 1e8 of them."""
    m, T, p, u = 3, 6, 2, 2.0**-24 if dtype == F32 else 2.0**-53
    npd = np.float32 if dtype == F32 else np.float64
    rng = np.random.default_rng(n)
    A = rng.normal(0, 1, (n, n))
    A *= 1e-4 / np.linalg.norm(A, 2)
    prob = W.Problem(model=W.LINEAR, n=n, m=m, T=T, p=p, Ad=A, Bd=1e-4 * rng.normal(0, 1, (n, m)),
                     q=rng.uniform(0.5, 2, n), r=np.full(m, 1e-12), qf=rng.uniform(0.5, 2, n),
                     x_goal=np.zeros(n), u_goal=np.zeros(m), u_min=-np.ones(m),
                     u_max=np.ones(m)).cast(npd)
    x0 = W.draw_x0(n, 3, scale=1.0).astype(npd).astype(np.float64)
    knots = W.draw_knots(prob, ncand, 5).astype(npd).astype(np.float64)
    K = dev(knots, dtype)
    dJ, cost = torch.empty_like(K), dev(np.full(ncand, np.nan), dtype)
    E.empc_grad(E.DeviceProblem(prob, dtype), dev(x0, dtype), K, ncand, ncand, dJ, cost)
    want = oracle_lib.rollout_cost(prob, x0, knots, ncand)
    err = np.abs(cost.cpu().numpy().astype(np.float64) / want - 1.0)
    # the states' own rounding: n + m products summed, doubled by the square
    assert err.max() < 2 * (n + T + 20 + n + m) * u * 4


@pytest.mark.parametrize("dtype,n,ncand", [(F32, 8, 32), (F32, 28, 32), (F32, 44, 32),
                                           (F32, 60, 530), (F64, 8, 1030), (F64, 28, 530)])
def test_rounding_of_the_drive_averages_out(oracle_lib, E, dtype, n, ncand):
    """200 steps around a state 100 away from the origin and one away from the
    goal, two knots, |A| = 0.5.  A step rounds its state about three times, by
    2.2e-6 rms each in FP32 (0.29 units in the last place of 100), and the steps'
    errors are independent: twice 3.8e-6 / sqrt(200 / 2) of the distance to the goal
    or about 1e-6 in the gradient; the bound is twice that.  A drive B_d u + w_d
    rounded once per knot instead would push every step the same way: twice
    2.2e-6 at least."""
    m, T, p, unit = 4, 200, 2, 1.0 if dtype == F32 else 2.0**-29
    npd = np.float32 if dtype == F32 else np.float64
    rng = np.random.default_rng(n)
    A = rng.normal(0, 1, (n, n))
    A *= 0.5 / np.linalg.norm(A, 2)
    xs = rng.uniform(80, 120, n) * rng.choice([-1.0, 1.0], n)
    prob = W.Problem(model=W.LINEAR, n=n, m=m, T=T, p=p, Ad=A, Bd=rng.normal(0, 0.3, (n, m)),
                     wd=(np.eye(n) - A) @ xs, q=np.ones(n), r=np.full(m, 0.01), qf=np.zeros(n),
                     x_goal=xs + rng.normal(0, 1, n), u_goal=np.zeros(m), u_min=-np.ones(m),
                     u_max=np.ones(m)).cast(npd)
    x0 = xs.astype(npd).astype(np.float64)
    knots = W.draw_knots(prob, ncand, 3).astype(npd).astype(np.float64)
    K = dev(knots, dtype)
    dJ, cost = torch.empty_like(K), dev(np.zeros(ncand), dtype)
    E.empc_grad(E.DeviceProblem(prob, dtype), dev(x0, dtype), K, ncand, ncand, dJ, cost)
    want, wcost = grad_long(prob, x0, knots)
    err = np.abs(dJ.cpu().numpy() - want).max(axis=0) / np.abs(want).max(axis=0)
    assert np.sqrt(np.mean(err.astype(float) ** 2)) < 2e-6 * unit
    cerr = (cost.cpu().numpy() / wcost - 1).astype(float)
    assert np.sqrt(np.mean(cerr**2)) < 2e-6 * unit


def grad_long(prob, x0, knots):
    """Costs and knot gradients in extended precision (plain numpy, no box)."""
    L = np.longdouble
    T, p, m, N = prob.T, prob.p, prob.m, knots.shape[1]
    A, B = prob.Ad.astype(L), prob.Bd.astype(L)
    w, q, r, qf, xg, ug = (np.asarray(v, dtype=L)[:, None] for v in
                           (prob.wd, prob.q, prob.r, prob.qf, prob.x_goal, prob.u_goal))
    U, X, us, at = knots.astype(L).reshape(p, m, N), [np.repeat(x0.astype(L)[:, None], N, 1)], [], []
    for k in range(T):
        a = k * (p - 1) // (T - 1) if T > 1 else 0
        c = L(k * (p - 1) - a * (T - 1)) / L(max(T - 1, 1))
        b = min(a + 1, p - 1)
        at.append((a, b, c))
        us.append((1 - c) * U[a] + c * U[b])
        X.append(A @ X[-1] + B @ us[-1] + w)
    J, lam = (qf * (X[T] - xg) ** 2).sum(0), 2 * (q + qf) * (X[T] - xg)
    D = np.zeros((p, m, N), L)
    for k in range(T - 1, -1, -1):
        J = J + (q * (X[k + 1] - xg) ** 2).sum(0) + (r * (us[k] - ug) ** 2).sum(0)
        a, b, c = at[k]
        g = 2 * r * (us[k] - ug) + B.T @ lam
        D[a] += (1 - c) * g
        D[b] += c * g
        lam = 2 * q * (X[k] - xg) + A.T @ lam
    return D.reshape(p * m, N), J


# (states, inputs, horizon, knots, candidates, dtype): every instance of the
# matrix-core kernel, with every state kept in LDS and in recomputed blocks,
# ragged tiles of candidates, one knot, two steps per knot, a knot per step.  Few
# candidates are enough where the kernel is chosen for its shorter steps; the
# other cases have more than the per-candidate kernel holds at once.
KEPT = [
    (14, 5, 40, 4, 33, F32), (28, 14, 40, 6, 47, F32), (28, 28, 32, 5, 20, F32),
    (42, 10, 30, 3, 31, F32), (48, 20, 28, 2, 16, F32), (40, 40, 28, 4, 20, F32),
    (64, 16, 12, 12, 513, F32), (50, 20, 12, 1, 514, F32), (15, 7, 25, 25, 1031, F32),
    (16, 16, 20, 4, 1040, F64), (17, 5, 12, 6, 515, F64), (32, 32, 8, 3, 520, F64),
    (33, 9, 10, 5, 9, F64), (48, 20, 8, 2, 16, F64),
]
BLOCKS = [
    (12, 4, 150, 7, 1030, F32), (30, 9, 80, 5, 1041, F32), (20, 20, 80, 9, 1030, F32),
    (33, 16, 60, 6, 530, F32), (44, 31, 60, 4, 520, F32), (36, 36, 60, 3, 517, F32),
    (64, 16, 60, 5, 530, F32), (64, 32, 60, 3, 529, F32),
    (11, 3, 90, 9, 1025, F64), (28, 14, 60, 5, 530, F64), (32, 17, 40, 3, 514, F64),
    (48, 16, 30, 3, 40, F64), (40, 32, 30, 3, 33, F64),
]
# the per-candidate kernel: more input than state tiles, FP64 above 48 states or
# 32 inputs, few candidates where its step is the shorter one
PER_CANDIDATE = [
    (5, 20, 10, 3, 7, F64), (64, 40, 11, 11, 600, F32), (60, 12, 9, 2, 700, F64),
    (40, 36, 9, 3, 20, F64), (14, 7, 30, 30, 20, F32), (28, 14, 90, 4, 24, F32),
    (20, 4, 25, 2, 40, F64),
]


@pytest.mark.parametrize("box", [False, True])
@pytest.mark.parametrize("n,m,T,p,ncand,dtype", KEPT + BLOCKS + PER_CANDIDATE)
def test_every_instance(oracle_lib, E, n, m, T, p, ncand, dtype, box):
    prob, x0, knots = case(n, m, T, p, ncand, dtype, box=box)
    check_grad(oracle_lib, E, prob, x0, knots, ncand, dtype)
    check_refine(oracle_lib, E, prob, x0, knots, ncand, dtype)


@pytest.mark.parametrize("dtype,d,T", [(F32, 21, 100), (F32, 30, 60), (F64, 14, 60)])
def test_no_less_exact_than_the_per_candidate_kernel(E, dtype, d, T):
    """Spring chains, whose model is close to the identity: 64 candidates alone run
    the per-candidate kernel (their horizon does not fit in LDS), the same 64 among
    528 the matrix cores.  Against extended precision the second may be off by a
    tenth more than the first, the spread of an rms over 64 candidates' worst
    entries."""
    npd = np.float32 if dtype == F32 else np.float64
    prob = W.linear_chain(d, T, 5, seed=2).cast(npd)
    x0 = W.draw_x0(prob.n, 1, scale=1.0).astype(npd).astype(np.float64)
    knots = W.draw_knots(prob, 528, 4).astype(npd).astype(np.float64)
    want, wcost = grad_long(prob, x0, knots[:, :64])
    dp, rms = E.DeviceProblem(prob, dtype), []
    for nc in (64, 528):
        K = dev(knots[:, :nc], dtype)
        dJ, cost = torch.empty_like(K), dev(np.zeros(nc), dtype)
        E.empc_grad(dp, dev(x0, dtype), K, nc, nc, dJ, cost)
        err = np.abs(dJ.cpu().numpy()[:, :64] - want).max(axis=0) / np.abs(want).max(axis=0)
        cerr = cost.cpu().numpy()[:64] / wcost - 1
        rms.append([np.sqrt(np.mean(e.astype(float) ** 2)) for e in (err, cerr)])
    assert rms[1][0] <= 1.1 * rms[0][0] and rms[1][1] <= 1.1 * rms[0][1]
