"""The rounding of differentiated runs.

The derivative of the FE map amplifies the last bit of the states it is taken
at (one ulp moves single entries of a gradient by up to 1e-7 of its rms, see
wcns_plan_gradient), so the forward states of ``rollout`` are pinned bit for
bit: digests of U(T) on inputs made with exact operations only (random dyadic
numbers, sums and products rounded once), whatever tiles and kernels the
plan's own steps use.  The gradient plan's steps stay within rounding of the
plan's, and its stored and recomputed stages give the same gradient."""
import hashlib

import numpy as np
import pytest
import torch

from gpu_util import say, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mods():
    from paper_2306_09760_amd import rollout, solver
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return solver, rollout


def state(shape, system="euler", seed=3):
    """A periodic state from averaged random numbers: sums and products only."""
    rng = np.random.default_rng(seed)
    nv = 1 if system == "advection" else len(shape) + 2
    grid = tuple(reversed(shape))
    f = rng.random((nv,) + grid)
    for ax in range(1, f.ndim):
        for k in (1, 2, 1):
            f = 0.25 * np.roll(f, k, ax) + 0.5 * f + 0.25 * np.roll(f, -k, ax)
    if nv == 1:
        return f
    rho = 0.75 + 0.5 * f[0]
    vel = [0.5 * f[1 + k] for k in range(len(shape))]
    ke = vel[0] * vel[0]
    for v in vel[1:]:
        ke = ke + v * v
    E = 2.5 * (0.75 + 0.5 * f[-1]) + 0.5 * (rho * ke)
    return np.ascontiguousarray(np.stack([rho] + [rho * v for v in vel] + [E]))


def run(solver, rollout, shape, opt, tiles=None, stages=True, steps=2):
    opt = dict(opt)
    P = solver.Plan(ndim=len(shape), n=shape, h=(1 / 64,) * len(shape), **opt)
    if tiles is not None:
        P.tiles = tiles
    U = to_dev(state(shape, opt.get("system", "euler"))).requires_grad_(True)
    dt = torch.full((1,), 1 / 1024, dtype=torch.float64, device="cuda")
    V = rollout.rollout(P, U, dt, steps, snapshots=1, stages=stages)
    return P, U, dt, V


def digest(V):
    return hashlib.sha256(to_host(V.detach()).tobytes()).hexdigest()[:16]


MD6 = dict(diff="md6", charproj=False)
CASES = [
    ((201,), dict(weights="fe"), "f9ffa7ad8f5ed8c8"),
    ((201,), dict(weights="fe", system="advection"), "a436725ee5fec40d"),
    ((1100,), dict(weights="pfe", **MD6), "a9c670f46f660048"),
    ((61, 58), dict(weights="fe"), "6aebca9e6ea4d0f5"),
    ((61, 58), dict(weights="fe", bc="transmissive", **MD6), "fb4736eef327925f"),
    ((61, 58), dict(weights="pfe"), "67a8f3e42a413ef3"),
    ((400, 395), dict(weights="fe"), "3ffe3c9228130d2f"),
    ((61, 58), dict(weights="fe", xi=300.0, zpow=3), "aea8e8787d3cacc7"),
    ((24, 33, 40), dict(weights="fe"), "10b8195178a31076"),
    ((70, 66, 61), dict(weights="pfe"), "fcf1ac38a07abf89"),
]


@pytest.mark.parametrize("shape,opt,want", CASES)
def test_rollout_keeps_its_rounding(mods, shape, opt, want):
    solver, rollout = mods
    tiles = [None]
    if len(shape) > 1:
        tiles += [(256, 32, 8), (128, 128, 2), (256, 64, 4)]
    for t in tiles:
        if t is not None and opt.get("system") == "advection":
            continue
        for stages in (True, False):
            say("rollout digest", shape, opt, t, stages)
            P, U, dt, V = run(solver, rollout, shape, opt, t, stages)
            assert digest(V) == want
    # the plan's own steps: the same up to rounding
    W = U.detach().clone()
    for _ in range(2):
        P.rk3_step(W, dt=dt)
    d = (W - V.detach()).norm() / W.norm()
    assert float(d) <= 1e-14


@pytest.mark.parametrize("shape", [(201,), (61, 58), (24, 33, 40)])
@pytest.mark.parametrize("weights", ["fe", "pfe", "z"])
def test_stored_and_recomputed_stages_agree(mods, shape, weights):
    solver, rollout = mods
    grads = []
    for stages in (True, False):
        say("gradient plan stages", shape, weights, stages)
        P, U, dt, V = run(solver, rollout, shape, dict(weights=weights), None, stages, 3)
        grads.append(torch.autograd.grad(V, U, torch.ones_like(V) - 0.5 * V.detach())[0])
    assert torch.equal(*grads)


def test_plan_and_gradient_plan_live_apart(mods):
    """Each is destroyed on its own; tiles set later on one are not the other's."""
    solver, _ = mods
    P = solver.Plan(ndim=2, n=(61, 58), h=(1 / 64, 1 / 64))
    g = P.gradient_plan()
    ref = to_host(P.residual(to_dev(state((61, 58)))))
    P.tiles = (256, 32, 8)
    assert g.tiles == (128, 32, 4)
    h = g.gradient_plan()
    a = h.residual(to_dev(state((61, 58))))
    del P, g
    assert torch.equal(h.residual(to_dev(state((61, 58)))), a)
    d = np.linalg.norm(to_host(a) - ref) / np.linalg.norm(ref)
    assert 0 < d <= 1e-13


def test_rollout_of_a_subclass_calls_its_methods(mods):
    solver, rollout = mods
    calls = []

    class Counted(solver.Plan):
        def rk3_step(self, *a, **kw):
            calls.append("step")
            return super().rk3_step(*a, **kw)

        def rk3_step_adjoint(self, *a, **kw):
            calls.append("adjoint")
            return super().rk3_step_adjoint(*a, **kw)

    P = Counted(ndim=1, n=(201,), h=(1 / 64,))
    U = to_dev(state((201,))).requires_grad_()
    dt = torch.full((1,), 1e-3, dtype=torch.float64, device="cuda")
    V = rollout.rollout(P, U, dt, 2, 2)
    V.sum().backward()
    assert calls.count("step") >= 2 and calls.count("adjoint") == 2


def test_rollouts_follow_the_plan(mods):
    """The gradient plan kept for rollouts takes the plan's tiles and whatever was
    set on the plan since the rollout before."""
    solver, rollout = mods
    P = solver.Plan(ndim=2, n=(61, 58), h=(1 / 64, 1 / 64))
    g = P._rollout_plan()
    assert P._rollout_plan() is g and g.tiles == P.tiles == (128, 32, 4)
    P.tiles = (256, 32, 8)
    k = P._rollout_plan()
    assert k is not g and k.tiles == (256, 32, 8) and g.tiles == (128, 32, 4)
    P.work = torch.empty_like(P.work)
    assert P._rollout_plan() is k and k.work is P.work
    P.autotune(to_dev(state((61, 58))))
    assert P._rollout_plan() is not k and P._rollout_plan().tiles == P.tiles
    assert P.gradient_plan()._rollout is None and k._h.value != P._h.value
