"""The WENO sweep's kernels with one lane per midpoint, which take a sweep of
more than 1408 tiles (two lanes per midpoint below): every weight kind on odd 1D,
2D and 3D grids just above that line against the oracle, and 1D grids of 1408 and
1409 tiles against each other bit for bit where their stencils agree.

Tolerance as in the other WENO weight tests: 1e-12 (normwise per variable), or
xi 2^-52 where a map's slope amplifies a weight's last bit, 100 times that
pointwise.  A state on which the oracle's own two roundings (plain and fused)
differ by more pins nothing and is passed over: the long 1D line with the FE maps,
whose differences are 1e-5 of its values (2e-10 between the two); there the
bitwise test stands alone."""
import numpy as np
import pytest
import torch

from gpu_util import rel_err, say, to_dev, to_host

pytestmark = pytest.mark.gpu

PATHS = [dict(weights="fe"), dict(weights="js"), dict(weights="z"), dict(weights="pfe"),
         dict(weights="fe", xi=1e6), dict(weights="z", zpow=3), dict(weights="linear")]


@pytest.fixture(scope="module")
def lib():
    from paper_2306_09760_amd import solver
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return solver


def _state(W, n, seed):
    prob, U = W.random_smooth_state(seed, len(n), n, amp=0.2)
    U = U.copy()
    U[0].flat[::5] *= 1.5
    return prob, U


@pytest.mark.parametrize("opt", PATHS, ids=str)
@pytest.mark.parametrize("n,charproj,bc", [((180001,), True, "transmissive"),
                                           ((461, 457), True, "periodic"),
                                           ((461, 457), False, "transmissive"),
                                           ((61, 58, 63), True, "transmissive")])
def test_residual(lib, ora, W, n, charproj, bc, opt):
    tol = max(1e-12, opt.get("xi", 100.0) * 2.0 ** -52)
    prob, U = _state(W, n, 14)
    opt = dict(opt, charproj=charproj)
    opt.setdefault("xi", 100.0)  # (the two sides' defaults differ)
    prob = dict(prob, bc=bc)
    say("weno large", n, opt, bc)
    ref, fused = (ora.Problem(**prob, family="weno", variant=v, **opt).residual(U)
                  for v in ("plain", "fma"))
    e = rel_err(fused, ref)
    if e[0] > tol or e[1] > 100 * tol:
        assert len(n) == 1 and opt["weights"] in ("fe", "pfe")
        return
    G = lib.Plan(**prob, scheme="weno", **opt)
    e = rel_err(to_host(G.residual(to_dev(U))), ref)
    assert e[0] <= tol and e[1] <= 100 * tol, e


@pytest.mark.parametrize("opt", PATHS, ids=str)
def test_both_sides_of_the_line(lib, W, opt):
    """1408 tiles (two lanes per midpoint) and 1409 (one): n + 6 slots in tiles
    of 127."""
    n = 1408 * 127 - 6
    _, U = _state(W, (n + 1,), 15)
    R = []
    for k in (0, 1):
        V = np.ascontiguousarray(U[:, :n + k])
        say("weno tiles", 1408 + k, opt)
        P = lib.Plan(ndim=1, n=(n + k,), h=(1.0 / n,), bc="transmissive", scheme="weno", **opt)
        R.append(to_host(P.residual(to_dev(V))))
    assert np.array_equal(R[0][:, :n - 3], R[1][:, :n - 3])
