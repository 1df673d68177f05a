"""The WENO sweep's specialised weights (JS, Z with p = 2, PFE, the steep FE
maps) and its run-time ones against the oracle: shock tubes, noise and jumps on
1D, 2D and 3D grids, on both sides of each rule that chooses a kernel.

Tolerance: the repository's 1e-12 (normwise per variable), or, where a map's
slope of up to xi / 2 amplifies a weight's last bit, xi 2^-52 if that is more;
100 times that pointwise.  A state on which the oracle's own two roundings (plain
and fused) differ by more than that pins nothing and is passed over: the noisy
tube where the maps act on projected fields (8e-10 between the two)."""
import numpy as np
import pytest
import torch

from gpu_util import rel_err, say, to_dev, to_host

pytestmark = pytest.mark.gpu

PATHS = [("js", 100.0, 1e-40, 2), ("js", 100.0, 1e-70, 2), ("js", 100.0, 1e-71, 2),
         ("z", 100.0, 1e-40, 2), ("z", 100.0, 1e-95, 2), ("z", 100.0, 1e-96, 2), ("z", 100.0, 1e-40, 3),
         ("pfe", 100.0, 1e-40, 2), ("pfe", 100.0, 1e-96, 2), ("pfe", 1e6, 1e-40, 2),
         ("fe", 980.0, 1e-40, 2), ("fe", 1000.0, 1e-40, 2), ("fe", 1e4, 1e-40, 2), ("fe", 1e6, 1e-40, 2)]


@pytest.fixture(scope="module")
def lib():
    from paper_2306_09760_amd import solver
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return solver


def _states(W):
    rng = np.random.default_rng(13)
    prob, U, _ = W.shock_tube(1.0, 0.75, 1.0, 0.125, 0.0, 0.1, 300)
    yield prob, U
    V = U.copy()
    V[:, 60:] *= 1.0 + 0.2 * rng.random((1, 240))
    yield prob, V
    for n in ((40, 37), (19, 21, 18)):
        prob, U = W.random_smooth_state(14, len(n), n, amp=0.2)
        U = U.copy()
        U[0].flat[::5] *= 1.5
        yield prob, U


@pytest.mark.parametrize("weights,xi,eps,zpow", PATHS)
@pytest.mark.parametrize("charproj", [True, False])
def test_residual_of_each_weno_path(lib, ora, W, weights, xi, eps, zpow, charproj):
    tol = max(1e-12, xi * 2.0 ** -52)
    checked = 0
    for prob, U in _states(W):
        opt = dict(weights=weights, xi=xi, eps=eps, zpow=zpow, charproj=charproj)
        say("weno weight path", opt, prob["n"])
        ref, fused = (ora.Problem(**prob, family="weno", variant=v, **opt).residual(U)
                      for v in ("plain", "fma"))
        n, p = rel_err(fused, ref)
        if n > tol or p > 100 * tol:
            continue
        checked += 1
        G = lib.Plan(**prob, scheme="weno", **opt)
        n, p = rel_err(to_host(G.residual(to_dev(U))), ref)
        assert n <= tol and p <= 100 * tol, (opt, prob["n"], n, p, tol)
    assert checked >= 3
