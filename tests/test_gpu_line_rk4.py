"""The four-stage step of a short 1D problem in one launch against the scheme's
definition, bit for bit: each stage's residual from ``Plan.residual`` (the
sweep), combined on the host with the roundings of the sweeps' stage epilogue
(fused products by the C library's fma).  Sizes on both sides of what one
workgroup serves: 64 KB of LDS for Euler (573 nodes with MND6, 571 with MD6),
1024 lanes for advection; beyond it the sweeps take the step."""
import ctypes as C

import numpy as np
import pytest
import torch

from gpu_util import say, to_dev, to_host

pytestmark = pytest.mark.gpu

_fma = C.CDLL("libm.so.6").fma
_fma.restype, _fma.argtypes = C.c_double, [C.c_double] * 3
fma = np.vectorize(_fma, otypes=[np.float64])


@pytest.fixture(scope="module")
def lib():
    from paper_2306_09760_amd import solver
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return solver


def _step(P, u, dt):
    L = lambda x: to_host(P.residual(to_dev(x)))  # noqa: E731
    u1 = fma(0.5 * dt, L(u), u)
    u2 = u + 0.5 * dt * L(u1)  # (the stage adds dt/2 R, rounded, to u)
    u3 = u + dt * L(u2)
    acc = fma(-1.0 / 3.0, u, 1.0 / 3.0 * u1) + 2.0 / 3.0 * u2
    return acc + fma(1.0 / 6.0 * dt, L(u3), 1.0 / 3.0 * u3)


def _problem(W, system, n):
    if system == "euler":
        prob, U, _ = W.shock_tube(1.0, 0.75, 1.0, 0.125, 0.0, 0.1, n)
        rng = np.random.default_rng(n)
        U = U * (1.0 + 0.05 * rng.random((1, n)))
        return dict(prob, system="euler"), np.ascontiguousarray(U)
    x = np.linspace(-1.0, 1.0, n, endpoint=False)
    return dict(ndim=1, n=(n,), h=(2.0 / n,), system="advection", bc="periodic"), \
        np.ascontiguousarray(np.where(np.abs(x) < 0.4, 1.0, 0.2 * np.sin(3 * x))[None])


@pytest.mark.parametrize("system,n", [("euler", n) for n in (9, 60, 201, 570, 571, 572, 573, 574, 601)]
                         + [("advection", n) for n in (9, 200, 1023, 1024, 1025)])
@pytest.mark.parametrize("opt", [dict(weights="fe"), dict(weights="z"), dict(weights="z", zpow=3),
                                 dict(weights="fe", xi=1e6)], ids=str)
def test_four_stage_step(lib, W, system, n, opt):
    prob, U = _problem(W, system, n)
    for diff in ("mnd6", "md6"):
        P = lib.Plan(**{**prob, **opt, "diff": diff})
        say("line rk4", system, n, opt, diff)
        dt = 0.2 * prob["h"][0]
        X = to_dev(U)
        P.rk4_step(X, dt=torch.full((1,), dt, dtype=torch.float64, device="cuda"))
        assert np.array_equal(to_host(X), _step(P, U, dt))
