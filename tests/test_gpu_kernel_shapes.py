"""Kernels with compile-time sizes and shape rules, at the edges of their ranges:
tiles, remainders, the smallest and the largest instance, against the FP64
oracle (or the library's own general form where the rule keeps the bits)."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

F32, F64 = torch.float32, torch.float64


@pytest.fixture(scope="module")
def E():
    import paper_2001_04931_amd as E

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    E.lib()
    return E


def dev(a, dtype=F64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype).cuda()


@pytest.mark.parametrize("N", range(1, 17))
def test_robot_every_row_length(oracle_lib, E, N):
    """The robot kernels are instantiated for even row lengths up to 16 (an odd
    link count runs with one padded link) and, from 9 links, on 2 x 2 tiles of
    the hold.  Both formulations are exact, so only FP64 rounding amplified by
    the mass matrix (condition below 1e4 here) separates them: 1e-11."""
    rng = np.random.default_rng(40 + N)
    mass, length, b = rng.uniform(0.5, 2.0, N), rng.uniform(0.1, 0.4, N), 0.05
    x = np.concatenate([rng.uniform(-2, 2, N), rng.uniform(-1.5, 1.5, N)])
    u = rng.uniform(-2, 2, N)
    R = E.NLinkRobot(mass, length, b, F64)
    n = 2 * N
    Ad, Bd, wd, xn = dev(np.full((n, n), np.nan)), dev(np.full((n, N), np.nan)), \
        dev(np.full(n, np.nan)), dev(np.full(n, np.nan))
    E.empc_nlink_linearize(R, 0.01, dev(x), dev(u), Ad, Bd, wd)
    E.empc_nlink_step(R, 0.01, 3, dev(x), dev(u), xn)
    wA, wB, ww = oracle_lib.nlink_linearize(mass, length, b, x, u, 0.01)
    # the offset is a difference of terms of size |A_d x| + |B_d u|
    sw = max(1.0, np.abs(wA).max() * np.abs(x).max() + np.abs(wB).max() * np.abs(u).max())
    for got, want, scale in ((Ad, wA, max(1.0, np.abs(wA).max())),
                             (Bd, wB, max(1.0, np.abs(wB).max())), (wd, ww, sw)):
        np.testing.assert_allclose(got.cpu().numpy(), want, rtol=1e-11, atol=1e-12 * scale)
    np.testing.assert_allclose(xn.cpu().numpy(),
                               oracle_lib.nlink_rk4(mass, length, b, x, u, 0.01, 3),
                               rtol=1e-11, atol=1e-12)


def random_linear(n, m, T, p, seed):
    rng = np.random.default_rng(seed)
    A = rng.normal(0, 1, (n, n))
    A *= 0.97 / max(abs(np.linalg.eigvals(A)))
    return W.Problem(model=W.LINEAR, n=n, m=m, T=T, p=p, Ad=A, Bd=rng.normal(0, 1, (n, m)),
                     wd=rng.normal(0, 0.1, n), q=rng.uniform(0.5, 2, n),
                     r=rng.uniform(0.01, 0.1, m), qf=rng.uniform(0, 1, n),
                     x_goal=rng.normal(0, 1, n), u_goal=rng.normal(0, 0.2, m),
                     u_min=-np.ones(m), u_max=np.ones(m))


# (states, inputs, horizon, knots): knot parameters 1, 15, 16, 17, 64, 65, 144,
# 160 (the last of the LDS factor), 161 (the first of the global one), and
# states at the ends of the response kernel's row lengths
@pytest.mark.parametrize("n,m,T,p", [(2, 1, 1, 1), (3, 3, 9, 5), (16, 4, 12, 4), (17, 17, 7, 1),
                                     (32, 8, 20, 8), (33, 13, 11, 5), (64, 9, 66, 16),
                                     (65, 16, 30, 10), (80, 23, 8, 7)])
def test_convex_sizes(oracle_lib, E, n, m, T, p):
    """P, q, c to FP64 rounding of the oracle's (1e-11 of the largest entry) and
    the minimizer by its optimality conditions (1e-9 of the gradient's scale:
    the solver stops at rounding level)."""
    from oracle import convex as C

    prob = random_linear(n, m, T, p, 100 * n + m)
    x0 = W.draw_x0(n, 7, scale=2.0)
    cs = E.ConvexSolver(E.DeviceProblem(prob, F64))
    z, J, info = (v.cpu().numpy() for v in cs.solve(dev(x0)))
    Po, qo, co = C.qp_form(prob, x0)
    np.testing.assert_allclose(cs.P.cpu().numpy(), Po, rtol=1e-11, atol=1e-11 * np.abs(Po).max())
    np.testing.assert_allclose(cs.q.cpu().numpy(), qo, rtol=1e-11, atol=1e-11 * np.abs(qo).max())
    np.testing.assert_allclose(cs.c.item(), co, rtol=1e-11)
    lo, hi = C.knot_bounds(prob)
    g = 2 * (Po @ z + qo)
    assert info[1] == 1 and np.all(z >= lo) and np.all(z <= hi)
    assert np.abs(z - np.clip(z - g, lo, hi)).max() < 1e-9 * max(1.0, np.abs(qo).max())
    np.testing.assert_allclose(J[0], C.qp_cost(Po, qo, co, z), rtol=1e-10)


def test_convex_pivots_outside_the_plain_range(E):
    """Weights of 1e210 make pivots whose reciprocals leave the fast square
    root's range: the factorization is repeated with the library's functions.
    Unbounded, so z = -P^-1 q (condition below 1e5: 1e-9)."""
    prob = random_linear(4, 3, 20, 5, 12)
    prob.u_min, prob.u_max = np.full(3, -1e250), np.full(3, 1e250)
    for k in ("q", "r", "qf"):
        setattr(prob, k, getattr(prob, k) * 1e210)
    cs = E.ConvexSolver(E.DeviceProblem(prob, F64), max_iter=3)
    z, _, _ = cs.solve(dev(np.full(4, 0.3)))
    P, q = cs.P.cpu().numpy() * 1e-210, cs.q.cpu().numpy() * 1e-210
    assert np.all(np.isfinite(P))
    np.testing.assert_allclose(z.cpu().numpy(), -np.linalg.solve(P, q), rtol=1e-9, atol=1e-9)


# (states, inputs, horizon, knots, candidates, dtype): every state-tile count
# and input-tile count of the matrix-core adjoint, ragged candidate tiles, one
# knot, a knot per step, horizons whose states do not fit in LDS (FP64 50 steps
# and up at two tiles), and more input than state tiles (the per-candidate
# kernel)
ADJOINT = [
    (1, 1, 1, 1, 1, F64), (3, 2, 9, 9, 17, F64), (16, 16, 20, 4, 16, F32), (17, 5, 21, 6, 15, F64),
    (28, 14, 60, 10, 33, F64), (32, 32, 12, 3, 40, F32), (33, 9, 25, 5, 31, F64),
    (48, 20, 14, 2, 16, F64), (40, 40, 18, 4, 20, F32), (64, 16, 30, 1, 18, F64),
    (64, 32, 60, 3, 16, F32), (64, 40, 11, 11, 5, F64), (28, 14, 300, 7, 48, F32),
    (5, 20, 10, 3, 7, F64),
]


@pytest.mark.parametrize("box", [False, True])
@pytest.mark.parametrize("n,m,T,p,ncand,dtype", ADJOINT)
def test_linear_adjoint_shapes(oracle_lib, E, n, m, T, p, ncand, dtype, box):
    """Costs and gradients against the FP64 oracle's: FP64 1e-9 of a column's
    largest entry; FP32 the method's 1e-4 (cost) and 2e-3 (gradient), the
    rounding of T dependent steps."""
    npd = np.float64 if dtype == F64 else np.float32
    prob = random_linear(n, m, T, p, 10 * n + m)
    if box:
        prob.x_min, prob.x_max = prob.x_goal - 0.3, prob.x_goal + 0.3
        prob.qb = np.linspace(0.5, 2.0, n)
    prob = prob.cast(npd)
    ld = ncand + 3
    x0 = W.draw_x0(n, 3).astype(npd).astype(np.float64)
    knots = W.draw_knots(prob, ncand, 5, ld=ld).astype(npd).astype(np.float64)
    dp, K = E.DeviceProblem(prob, dtype), dev(knots, dtype)
    dJ, cost = torch.full_like(K, float("nan")), dev(np.full(ncand, np.nan), dtype)
    E.empc_grad(dp, dev(x0, dtype), K, ncand, ld, dJ, cost)
    want, wcost = oracle_lib.grad(prob, x0, knots, ncand)
    got = dJ.cpu().numpy().astype(np.float64)
    assert np.all(np.isnan(got[:, ncand:]))  # nothing stored past the candidates
    err = np.abs(got[:, :ncand] - want[:, :ncand]).max(axis=0)
    scale = np.abs(want[:, :ncand]).max(axis=0)
    tg, tc = (1e-9, 1e-10) if dtype == F64 else (2e-3, 1e-4)
    assert (err <= tg * scale + 1e-30).all()
    np.testing.assert_allclose(cost.cpu().numpy(), wcost, rtol=tc)
    # refinement on the same tiles: a few Adam steps against the oracle's
    if dtype == F64:
        wk, wc = oracle_lib.refine(prob, x0, knots, wcost, lr=0.01, steps=3)
        C = dev(wcost, dtype)
        E.empc_refine(dp, dev(x0, dtype), K, ncand, ld, C, 0.01, 3)
        np.testing.assert_allclose(C.cpu().numpy(), wc, rtol=1e-9)
        np.testing.assert_allclose(K.cpu().numpy()[:, :ncand], wk[:, :ncand], rtol=0, atol=1e-9)


def test_linear_adjoint_blocks_equal_kept_states(E):
    """More candidate tiles than the chip holds with every state in LDS: the
    states are recomputed in blocks, by the same steps from the same stored
    states, so the first candidates' gradients are the same bits as in a
    small call that keeps them all; a candidate's NaN stays its own."""
    prob = W.linear_chain(14, 50, 10, seed=1).cast(np.float32)
    dp = E.DeviceProblem(prob, F32)
    n1, n2 = 64, 16 * 256 + 40
    x0 = dev(W.draw_x0(prob.n, 1), F32)
    K = dev(W.draw_knots(prob, n2, 2), F32)
    K[3, 5] = float("nan")
    out = []
    for nc in (n1, n2):
        dJ, cost = torch.zeros_like(K), torch.zeros(n2, device="cuda")
        E.empc_grad(dp, x0, K, nc, n2, dJ, cost)
        out.append((dJ[:, :n1].cpu(), cost[:n1].cpu()))
    for a, b in zip(*out):
        assert torch.equal(a.nan_to_num(123.0), b.nan_to_num(123.0))
        bad = torch.isnan(a).reshape(-1, n1).any(0)
        assert bad[5] and bad.sum() == 1


def spd(n, rng):
    Q, _ = np.linalg.qr(rng.normal(0, 1, (n, n)))
    return (Q * np.geomspace(1.0, 0.05, n)) @ Q.T


# (states, inputs, horizon, knots, candidates): state counts at both ends of
# every live-slice and tile count, input counts at the ends of the slice
# counts (and more input than state tiles), one knot, one step, a knot per step
FULL = [
    (1, 1, 1, 1, 1), (4, 2, 9, 3, 17), (5, 20, 12, 4, 16), (8, 4, 20, 20, 33), (9, 5, 15, 2, 15),
    (16, 8, 21, 6, 48), (16, 32, 8, 3, 5), (17, 9, 13, 4, 31), (32, 16, 25, 1, 18),
    (33, 17, 18, 5, 16), (48, 1, 30, 10, 40), (49, 32, 11, 11, 7), (64, 32, 40, 7, 65),
]


@pytest.mark.parametrize("weights", ["QRQf", "Q", "R", "Qf"])
@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("n,m,T,p,ncand", FULL)
def test_full_weights_shapes(oracle_lib, E, n, m, T, p, ncand, dtype, weights):
    """Costs with full weights against the FP64 oracle's, with the state box
    and its step charge (FP64) or without: relative 1e-9 and, as for the
    diagonal FP32 rollout, 1e-4."""
    npd = np.float64 if dtype == F64 else np.float32
    rng = np.random.default_rng(n + m)
    prob = random_linear(n, m, T, p, 100 * n + m)
    if "Q" in weights.replace("Qf", ""):
        prob.Q = spd(n, rng)
    if "R" in weights:
        prob.R = 0.05 * spd(m, rng)
    if "Qf" in weights:
        prob.Qf = 2.0 * spd(n, rng)
    if dtype == F64:
        prob.x_min, prob.x_max = prob.x_goal - 0.3, prob.x_goal + 0.3
        prob.qb, prob.sb = np.linspace(0.5, 2.0, n), np.linspace(0.1, 0.7, n)
    prob = prob.cast(npd)
    ld = ncand + 2
    x0 = W.draw_x0(n, 4).astype(npd).astype(np.float64)
    knots = W.draw_knots(prob, ncand, 6, ld=ld).astype(npd).astype(np.float64)
    cost = dev(np.full(ncand + 4, np.nan), dtype)
    E.empc_rollout_cost(E.DeviceProblem(prob, dtype), dev(x0, dtype), dev(knots, dtype), ncand, ld,
                        cost)
    got = cost.cpu().numpy()
    assert np.isnan(got[ncand:]).all()  # nothing stored past the candidates
    np.testing.assert_allclose(got[:ncand], oracle_lib.rollout_cost(prob, x0, knots, ncand),
                               rtol=1e-9 if dtype == F64 else 1e-4)


@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("pop,k", [(257, 256), (511, 40), (1000, 64), (1024, 32), (1024, 256),
                                   (4097, 64), (6000, 1), (16384, 64), (16385, 200), (40000, 256)])
def test_selection_short_cut_edges(oracle_lib, E, pop, k, dtype):
    """Selection through the wavefronts' threshold and through the passes that
    follow when it keeps too many costs: full and partly filled wavefronts,
    the lowest costs spread, all in the first slots, all in the last ones, and
    more equal costs at the threshold than a workgroup has threads.  Indices
    are exact."""
    from test_gpu_parity import gpu_generation

    prob = W.linear_chain(2, 10, 3, seed=0)
    ga = W.GA(pop=pop, n_elite=k, generations=1, sigma=0.1, seed=1)
    rng = np.random.default_rng(pop + k)
    spread = rng.normal(0, 1, pop).astype(np.float32).astype(np.float64)
    equal = np.where(rng.random(pop) < 0.002, -1.0, 2.0)
    knots = W.draw_knots(prob, pop, 1)
    for cost in (spread, np.sort(spread), np.sort(spread)[::-1].copy(), equal,
                 np.where(rng.random(pop) < 0.5, np.nan, spread)):
        _, eidx, best = gpu_generation(E, prob, ga, knots, cost, 0, 0, dtype)
        want_idx, want_best = oracle_lib.select(cost, k)
        np.testing.assert_array_equal(eidx, want_idx)
        assert best == want_best


@pytest.mark.parametrize("elitism", [True, False])
@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("m,p,pop,k", [(1, 1, 65, 1), (1, 7, 300, 65), (3, 5, 1000, 130),
                                       (5, 3, 64, 64), (31, 9, 129, 20), (33, 10, 4500, 256),
                                       (40, 4, 700, 70)])
def test_warm_population_shapes(oracle_lib, E, m, p, pop, k, dtype, elitism):
    """Children against the oracle's: parameter counts that leave a group of
    four partly filled, inputs that wrap inside a group and past a 32-bit word
    of mutation flags, bounds that differ by input, parents past the first
    tile of 64 slots.  The tolerances are those of the noise's rounding (1e-6
    at sigma 0.1 in FP32, 1e-14 in FP64)."""
    from test_gpu_parity import gpu_generation

    npd = np.float64 if dtype == F64 else np.float32
    prob = random_linear(4, m, 12, p, 70 + m)
    prob.u_max = np.linspace(0.5, 1.0, m)
    prob.u_min = -np.linspace(1.0, 0.7, m)
    prob = prob.cast(npd)
    ga = W.GA(pop=pop, n_elite=k, generations=1, sigma=0.1, seed=99, elitism=elitism)
    rng = np.random.default_rng(pop)
    knots = W.draw_knots(prob, pop, 2).astype(npd).astype(np.float64)
    cost = rng.uniform(0, 10, pop).astype(npd).astype(np.float64)
    got, eidx, _ = gpu_generation(E, prob, ga, knots, cost, tick=5, gen=3, dtype=dtype)
    want_idx, _ = oracle_lib.select(cost, k)
    np.testing.assert_array_equal(eidx, want_idx)
    want = oracle_lib.next_population(prob, ga, knots[:, want_idx].T.copy(), cold=False, tick=5,
                                      gen=3)
    np.testing.assert_allclose(got, want, rtol=0, atol=1e-6 if dtype == F32 else 1e-14)


@pytest.mark.parametrize("option", ["plain", "goal", "box"])
@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("n,m,T,p,ncand", [(1, 1, 1, 1, 1), (3, 2, 9, 4, 17), (4, 4, 20, 20, 64),
                                           (4, 8, 13, 1, 130), (5, 5, 12, 3, 16), (8, 1, 30, 6, 90),
                                           (8, 8, 21, 5, 15), (9, 4, 10, 2, 33)])
def test_few_states_rollout(oracle_lib, E, n, m, T, p, ncand, dtype, option):
    """Linear rollouts at both ends of the compile-time slice counts (up to 4,
    up to 8, more states), against the FP64 oracle: relative 1e-9 and 1e-4."""
    npd = np.float64 if dtype == F64 else np.float32
    prob = random_linear(n, m, T, p, 30 * n + m)
    if option == "plain":
        prob.x_goal = None
    if option == "box":
        prob.x_min, prob.x_max = prob.x_goal - 0.3, prob.x_goal + 0.3
        prob.qb = np.linspace(0.5, 2.0, n)
    prob = prob.cast(npd)
    x0 = W.draw_x0(n, 8).astype(npd).astype(np.float64)
    knots = W.draw_knots(prob, ncand, 9, ld=ncand + 1).astype(npd).astype(np.float64)
    cost = dev(np.full(ncand + 3, np.nan), dtype)
    E.empc_rollout_cost(E.DeviceProblem(prob, dtype), dev(x0, dtype), dev(knots, dtype), ncand,
                        ncand + 1, cost)
    got = cost.cpu().numpy()
    assert np.isnan(got[ncand:]).all()
    np.testing.assert_allclose(got[:ncand], oracle_lib.rollout_cost(prob, x0, knots, ncand),
                               rtol=1e-9 if dtype == F64 else 1e-4)
