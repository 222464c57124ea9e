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
