"""FE weights (and steep PFE) with an eps so small that the product of the three
squared indicators of a flat stencil, eps^6, would underflow: the run-time
weights take over there.  Both sides of the line, for the WCNS and the WENO
sweep, on states with exactly uniform parts, against the oracle; and the adjoint
of such a plan against the oracle's JVP.

Tolerance as in the other weight tests: 1e-12 (normwise per variable), or xi
2^-52 where a map's slope amplifies a weight's last bit, 100 times that
pointwise.  A state on which the oracle's own two roundings (plain and fused)
differ by more pins nothing and is passed over."""
import numpy as np
import pytest
import torch

from gpu_util import rel_err, say, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2306_09760_amd import solver
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return solver


def _states(W):
    prob, U, _ = W.shock_tube(1.0, 0.75, 1.0, 0.125, 0.0, 0.1, 300)
    yield prob, U
    V = U.copy()
    V[:, 100:180] *= 1.5
    yield prob, V
    prob, U = W.random_smooth_state(12, 2, (40, 37), amp=0.2)
    U = U.copy()
    U[:, :12] = U[:, :1, :1]  # a uniform band
    yield prob, U


@pytest.mark.parametrize("scheme", ["wcns", "weno"])
@pytest.mark.parametrize("weights,xi", [("fe", 100.0), ("fe", 500.0), ("fe", 1e6), ("pfe", 1e6)])
@pytest.mark.parametrize("eps", [1e-45, 1.0001e-51, 9.999e-52, 1e-60, 1e-99])
def test_residual(lib, ora, W, scheme, weights, xi, eps):
    tol = max(1e-12, xi * 2.0 ** -52)
    checked = 0
    for prob, U in _states(W):
        opt = dict(weights=weights, xi=xi, eps=eps)
        say("small eps", scheme, opt, prob["n"])
        G = lib.Plan(**prob, scheme=scheme, **opt)
        got = to_host(G.residual(to_dev(U)))
        ref, fused = (ora.Problem(**prob, family=scheme, variant=v, **opt).residual(U)
                      for v in ("plain", "fma"))
        assert np.isfinite(got).all() and np.isfinite(ref).all()
        n, p = rel_err(fused, ref)
        if n > tol or p > 100 * tol:
            continue
        checked += 1
        n, p = rel_err(got, ref)
        assert n <= tol and p <= 100 * tol, (opt, prob["n"], n, p)
    assert checked >= 2


@pytest.mark.parametrize("xi", [100.0, 1e6])
def test_adjoint(lib, ora, W, xi):
    prob, U = W.random_smooth_state(24, 2, (16, 14), amp=0.25)
    opt = dict(weights="fe", xi=xi, eps=1e-60)
    say("small eps adjoint", opt)
    G, O = lib.Plan(**prob, **opt), ora.Problem(**prob, **opt)
    rng = np.random.default_rng(4)
    V, Rb = rng.standard_normal(U.shape), rng.standard_normal(U.shape)
    Ub = to_host(G.residual_adjoint(to_dev(U), to_dev(Rb)))
    _, JV = O.residual_jvp(U, V)
    scale = np.linalg.norm(Ub) * np.linalg.norm(V)
    assert abs(float(np.sum(Ub * V)) - float(np.sum(Rb * JV))) <= 1e-10 * scale
