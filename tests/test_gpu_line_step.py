"""The one-launch step of short 1D problems: bitwise the step of a ragged batch of
one problem and of the sweeps, and the oracle's step, around the sizes at which
it pads to a wavefront, and on both sides of its size limit; with a given dt, a
CFL-limited one, kept stages, the four-stage scheme, and a non-physical state
reported."""
import numpy as np
import pytest
import torch

from gpu_util import rel_err, say, to_dev, to_host

pytestmark = pytest.mark.gpu

SIZES = [9, 59, 61, 62, 125, 201, 253, 320, 321, 509, 600, 601, 1100]
WEIGHTS = [("fe", 100.0), ("z", 100.0), ("js", 100.0), ("pfe", 100.0), ("fe", 1e6), ("fe", 500.0)]


@pytest.fixture(scope="module")
def lib():
    from paper_2306_09760_amd import solver
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return solver


def _tube(W, n, bc, seed):
    if bc == "periodic":
        return W.random_smooth_state(seed, 1, (n,), amp=0.2)
    prob, U, _ = W.shock_tube(1.0, 0.75, 1.0, 0.125, 0.0, 0.1, n)
    U = U * (1.0 + 0.1 * np.random.default_rng(seed).random(U.shape[1:]))
    return prob, np.ascontiguousarray(U)


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("bc", ["transmissive", "periodic"])
@pytest.mark.parametrize("weights,xi", WEIGHTS)
def test_step_equals_the_sweeps(lib, W, n, bc, weights, xi):
    prob, U = _tube(W, n, bc, n)
    for diff, charproj in (("mnd6", True), ("md6", False)):
        opt = dict(weights=weights, xi=xi, diff=diff, charproj=charproj, bc=bc)
        say("line step", n, opt)
        P = lib.Plan(**{**prob, **opt})
        B = lib.BatchPlan([0, n], [prob["h"][0]], **opt)
        Ua, Ub, Uc = to_dev(U), to_dev(U), to_dev(U)
        t = torch.zeros(1, dtype=torch.float64, device="cuda")
        for _ in range(3):
            P.rk3_step(Ua, cfl=0.5)
            B.rk3_step(Ub, t, 1e9, cfl=0.5)
            dt = B.last_dt()
            P.rk3_step(Uc, dt=dt)
        assert torch.equal(Ua, Ub) and torch.equal(Uc, Ub)


@pytest.mark.parametrize("n", SIZES)
def test_stages_and_oracle_steps(lib, ora, W, n):
    prob, U = _tube(W, n, "periodic", n + 1)
    opt = dict(weights="fe", xi=100.0)
    P, O = lib.Plan(**prob, **opt), ora.Problem(**prob, **opt)
    say("line stages", n)
    dt = O.cfl_dt(U, 0.3)
    dtd = torch.full((1,), dt, dtype=torch.float64, device="cuda")
    Ua, Ub, Uc = to_dev(U), to_dev(U), to_dev(U)
    U1, U2 = torch.empty_like(Ua), torch.empty_like(Ua)
    P.rk3_step(Ua, dt=dtd)
    P.rk3_step_stages(Ub, U1, U2, dt=dtd)
    assert torch.equal(Ua, Ub)
    R = P.residual(to_dev(U))
    assert torch.allclose(U1, to_dev(U) + dtd * R, rtol=1e-14, atol=0)
    la, lb = to_dev(U), to_dev(U)
    P.rk3_step_adjoint(to_dev(U), la, dtd)
    P.rk3_step_adjoint(to_dev(U), lb, dtd, stages=(U1, U2))
    assert torch.equal(la, lb)
    P.rk4_step(Uc, dt=dtd)
    for got, ref in ((Ua, O.rk3_step(U, dt)[0]), (Uc, O.rk4_step(U, dt)[0])):
        e = rel_err(to_host(got), ref)
        assert e[0] <= 1e-12 and e[1] <= 1e-10, (n, e)


@pytest.mark.parametrize("n", [9, 200, 1000, 1024, 1025, 1100])
@pytest.mark.parametrize("adv", [1.0, -0.7])
def test_advection_steps(lib, ora, W, n, adv):
    prob, U, _ = W.advection_sine(seed=3, n=n)
    prob["adv"] = (adv,)
    P, O = lib.Plan(**prob, weights="fe"), ora.Problem(**prob, weights="fe", xi=100.0)
    say("line advection", n, adv)
    for step, ostep, cfl in ((P.rk3_step, O.rk3_step, 0.5), (P.rk4_step, O.rk4_step, 0.3)):
        Ud = to_dev(U)
        step(Ud, cfl=cfl)
        e = rel_err(to_host(Ud), ostep(U, O.cfl_dt(U, cfl))[0])
        assert e[0] <= 1e-12 and e[1] <= 1e-10, (n, e)


@pytest.mark.parametrize("n", [100, 1100])
@pytest.mark.parametrize("method", ["rk3_step", "rk4_step"])
def test_node_without_energy_as_on_the_sweeps(lib, W, n, method):
    """p = 0 at one node: the flux takes the larger of the two sides' speeds (a
    NaN only if both are), so the stages stay finite and unflagged on the GPU,
    where the oracle's speeds and step are NaN; the step must do as the sweeps."""
    prob, U = _tube(W, n, "transmissive", 1)
    P = lib.Plan(**prob, weights="fe")
    for bad in (0, 1):
        V = U.copy()
        if bad:
            V[2, n // 2] = 0.0  # no energy at one node, before the stages
        dt = torch.full((1,), 1e-9, dtype=torch.float64, device="cuda")
        st = torch.zeros(1, dtype=torch.int32, device="cuda")
        say("line status", n, method, bad)
        Ua, Ub = to_dev(V), to_dev(V)
        getattr(P, method)(Ua, dt=dt, status=st)
        assert int(st.item()) == 0 and bool(torch.isfinite(Ua).all())
        if method == "rk3_step":
            B = lib.BatchPlan([0, n], [prob["h"][0]], weights="fe", bc="transmissive")
            t, sb = torch.zeros_like(dt), torch.zeros_like(st)
            B.rk3_step(Ub, t, 1e-9, cfl=0.5, status=sb)  # the end time caps dt at 1e-9
            assert int(sb.item()) == int(st.item()) and torch.equal(Ua, Ub)


@pytest.mark.parametrize("n", [100, 1100])
@pytest.mark.parametrize("method", ["rk3_step", "rk4_step"])
def test_negative_energy_is_reported(lib, W, n, method):
    prob, U = _tube(W, n, "transmissive", 1)
    U[2, n // 2] = -1.0  # of order one: the stages at dt = 1e-9 cannot mend it
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    say("line status, negative energy", n, method)
    getattr(lib.Plan(**prob, weights="fe"), method)(
        to_dev(U), dt=torch.full((1,), 1e-9, dtype=torch.float64, device="cuda"), status=st)
    assert int(st.item()) == 1
