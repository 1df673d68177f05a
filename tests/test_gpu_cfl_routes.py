"""The time step's maximum on its routes (one block, several blocks, within the
one-launch steps), around the sizes at which they change: the oracle's dt to the
rounding of one rate (1e-14), the step's dt the same on every route, and a
non-finite node anywhere giving a non-finite dt."""
import numpy as np
import pytest
import torch

from gpu_util import say, to_dev, to_host

pytestmark = pytest.mark.gpu

SHAPES = [(9,), (320,), (321,), (4096,), (4097,), (9, 9), (64, 64), (17, 241), (363, 362),
          (9, 10, 11), (16, 16, 16), (65, 64, 64)]


@pytest.fixture(scope="module")
def lib():
    from paper_2306_09760_amd import solver
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return solver


@pytest.mark.parametrize("shape", SHAPES)
def test_dt_of_every_route(lib, ora, W, shape):
    prob, U = W.random_smooth_state(5, len(shape), shape, amp=0.2)
    P, O = lib.Plan(**prob, weights="z"), ora.Problem(**prob, weights="z")
    say("cfl route", shape)
    dt = P.cfl_dt(to_dev(U), 0.5).clone()
    assert abs(float(dt) - O.cfl_dt(U, 0.5)) <= 1e-14 * float(dt)
    Ua, Ub = to_dev(U), to_dev(U)
    P.rk3_step(Ua, cfl=0.5)
    P.rk3_step(Ub, dt=dt)
    assert torch.equal(Ua, Ub)
    n = int(np.prod(shape))
    for k in sorted({0, 1, 5, n // 2, n - 2, n - 1}):
        V = U.copy()
        V[0].flat[k] = np.nan
        assert not np.isfinite(float(P.cfl_dt(to_dev(V), 0.5))), k
        X = to_dev(V)
        P.rk3_step(X, cfl=0.5)
        assert not np.isfinite(to_host(X)).any(), k
