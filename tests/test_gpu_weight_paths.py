"""The specialised weights (JS, Z with p = 2, PFE, the steep FE maps) on the
device against the oracle: grids and a ragged batch with flat parts, jumps
and noise, on both sides of each rule that chooses a path (the size of eps;
the steepness from which the maps are staircases, where weights fall into the
bands around the null points).

Tolerance: the repository's 1e-12 (normwise per variable), or, where a map's
slope of up to xi / 2 amplifies a weight's last bit, xi 2^-52 if that is
more; 100 times that pointwise."""
import numpy as np
import pytest
import torch

from gpu_util import rel_err, say, to_dev, to_host

pytestmark = pytest.mark.gpu

PATHS = [("js", 100.0, 1e-40), ("js", 100.0, 1e-70), ("js", 100.0, 1e-71),
         ("z", 100.0, 1e-40), ("z", 100.0, 1e-95), ("z", 100.0, 1e-96),
         ("pfe", 100.0, 1e-40), ("pfe", 100.0, 1e-96), ("pfe", 1e6, 1e-40),
         ("fe", 980.0, 1e-40), ("fe", 1000.0, 1e-40), ("fe", 1e4, 1e-40), ("fe", 1e6, 1e-40)]


@pytest.fixture(scope="module")
def lib():
    from paper_2306_09760_amd import solver
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return solver


def _states(W):
    rng = np.random.default_rng(11)
    prob, U, _ = W.shock_tube(1.0, 0.75, 1.0, 0.125, 0.0, 0.1, 300)
    yield prob, U
    V = U.copy()
    V[:, 60:] *= 1.0 + 0.2 * rng.random((1, 240))
    yield prob, V
    for n in ((40, 37), (19, 21, 18)):
        prob, U = W.random_smooth_state(12, len(n), n, amp=0.2)
        U = U.copy()
        U[0].flat[::5] *= 1.5
        yield prob, U


def _check(got, ref, xi, what):
    n, p = rel_err(got, ref)
    tol = max(1e-12, xi * 2.0 ** -52)
    assert n <= tol and p <= 100 * tol, f"{what}: {n:.3e} / {p:.3e} (bar {tol:.1e})"


@pytest.mark.parametrize("weights,xi,eps", PATHS)
@pytest.mark.parametrize("diff,charproj", [("mnd6", True), ("md6", False)])
def test_residual_of_each_weight_path(lib, ora, W, weights, xi, eps, diff, charproj):
    for prob, U in _states(W):
        opt = dict(weights=weights, xi=xi, eps=eps, diff=diff, charproj=charproj)
        say("weight path", opt, prob["n"])
        G, O = lib.Plan(**prob, **opt), ora.Problem(**prob, **opt)
        _check(to_host(G.residual(to_dev(U))), O.residual(U), xi, f"{opt} {prob['n']}")


@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("weights,xi,eps", [("js", 100.0, 1e-40), ("z", 100.0, 1e-40),
                                            ("pfe", 100.0, 1e-40), ("fe", 1000.0, 1e-40)])
def test_batch_residual_of_each_weight_path(lib, ora, W, weights, xi, eps, tile):
    prob, U, meta = W.shock_tube_batch(seed=5, nprob=5, nmin=9, nmax=300)
    opt = dict(weights=weights, xi=xi, eps=eps)
    say("batch weight path", opt, tile)
    off = meta["offsets"]
    B = lib.BatchPlan(off, meta["h"], **opt)
    B.tile = tile
    R = to_host(B.residual(to_dev(U)))
    for p in range(5):
        s = slice(int(off[p]), int(off[p + 1]))
        O = ora.Problem(ndim=1, n=(s.stop - s.start,), h=(meta["h"][p],), bc="transmissive", **opt)
        _check(R[:, s], O.residual(U[:, s]), xi, f"problem {p}")
