"""The WENO sweep at the edges of its tiles (127 nodes along x from lines
packed end to end with three ghosts per side, 31 nodes by four columns along y
and z): shortest lines, lengths around a tile's, several lines in one tile,
ragged last columns, against the oracle to the repository's one-residual bar
(1e-12 normwise, 1e-10 pointwise)."""
import numpy as np
import pytest
import torch

from gpu_util import rel_err, say, to_dev, to_host

pytestmark = pytest.mark.gpu

GRIDS = [(9,), (121,), (122,), (127,), (128,), (254,), (9, 9), (300, 24), (33, 62), (31, 63),
         (9, 10, 33), (13, 31, 9)]


@pytest.fixture(scope="module")
def lib():
    from paper_2306_09760_amd import solver
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return solver


@pytest.mark.parametrize("n", GRIDS)
@pytest.mark.parametrize("bc", ["periodic", "transmissive"])
@pytest.mark.parametrize("weights,charproj", [("fe", True), ("z", False)])
def test_weno_residual_at_tile_edges(lib, ora, W, n, bc, weights, charproj):
    prob, U = W.random_smooth_state(31, len(n), n, amp=0.2)
    U = U.copy()
    U[0].flat[::7] *= 1.4  # jumps, also at line ends
    prob["bc"] = bc
    opt = dict(weights=weights, xi=100.0, charproj=charproj)
    say("weno tiles", n, bc, opt)
    G = lib.Plan(**prob, scheme="weno", **opt)
    O = ora.Problem(**prob, family="weno", **opt)
    e = rel_err(to_host(G.residual(to_dev(U))), O.residual(U))
    assert e[0] <= 1e-12 and e[1] <= 1e-10, (n, bc, opt, e)
    dt = torch.full((1,), 1e-4, dtype=torch.float64, device="cuda")
    Ud = to_dev(U)
    G.rk3_step(Ud, dt=dt)
    e = rel_err(to_host(Ud), O.rk3_step(U, 1e-4)[0])
    assert e[0] <= 1e-12 and e[1] <= 1e-10, ("step", n, bc, opt, e)
