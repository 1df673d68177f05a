"""The SSP-RK3 step with one launch per stage (small 2D and 3D problems):
bitwise the sweeps' step, for odd extents around the tiles', both differences, all weight kinds and boundary
types, given and CFL-limited dt, kept stages, the allocation-free step, and on
replays of a captured step."""
import pytest
import torch

from gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(11, 9), (29, 33), (61, 58), (117, 125), (130, 30), (11, 12, 9), (30, 28, 33), (35, 61, 27)]
WEIGHTS = [("fe", 100.0), ("z", 100.0), ("js", 100.0), ("pfe", 100.0), ("fe", 1e6), ("fe", 500.0)]


@pytest.fixture(scope="module")
def lib():
    from paper_2306_09760_amd import solver
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return solver


def _sweeps(P, U, dt):
    """Stage states and result of the sweeps, which serve a step whose stage
    arrays are the first two states of the plan's own workspace."""
    X, nb = U.clone(), U.numel() * 8
    al = (nb + 255) // 256 * 256
    U1, U2 = (P.work[k * al:k * al + nb].view(torch.float64).view(U.shape) for k in (0, 1))
    P.rk3_step_stages(X, U1, U2, dt=dt)
    return U1, U2, X


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("bc", ["transmissive", "periodic"])
@pytest.mark.parametrize("weights,xi", WEIGHTS)
def test_step_equals_the_sweeps(lib, W, shape, bc, weights, xi):
    prob, U = W.random_smooth_state(sum(shape), len(shape), shape, amp=0.2)
    for diff, charproj in (("mnd6", True), ("md6", False)):
        opt = dict(weights=weights, xi=xi, diff=diff, charproj=charproj, bc=bc)
        say("stage step", shape, opt)
        P = lib.Plan(**{**prob, **opt})
        Ua, Ub, Uc, Ud = (to_dev(U) for _ in range(4))
        U1, U2 = torch.full_like(Ua, float("nan")), torch.full_like(Ua, float("nan"))
        dt = P.cfl_dt(Ua, 0.5).clone()
        st = torch.zeros(1, dtype=torch.int32, device="cuda")
        P.rk3_step(Ua, cfl=0.5, status=st)
        P.rk3_step(Ub, dt=dt)
        P.rk3_step_stages(Uc, U1, U2, dt=dt)
        P.rk3_step_noalloc(Ud, dt=None, cfl=0.5)
        assert torch.equal(Ua, Ub) and torch.equal(Ua, Uc) and torch.equal(Ua, Ud)
        assert int(st.item()) == 0
        for got, ref in zip((U1, U2, Ua), _sweeps(P, to_dev(U), dt)):
            assert torch.equal(got, ref) and bool(torch.isfinite(ref).all())


@pytest.mark.parametrize("shape", [(61, 58), (30, 28, 33)])
def test_status_capture_and_workspace_stages(lib, W, shape):
    prob, U = W.random_smooth_state(3, len(shape), shape, amp=0.2)
    P = lib.Plan(**prob, weights="fe")
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    V = U.copy()
    V[(-1,) + tuple(n // 2 for n in U.shape[1:])] = -1.0
    P.rk3_step(to_dev(V), dt=torch.full((1,), 1e-9, dtype=torch.float64, device="cuda"), status=st)
    assert int(st.item()) == 1
    X, ref = to_dev(U), to_dev(U)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            P.rk3_step(X, cfl=0.4)
    X.copy_(to_dev(U))
    for k in range(4):
        say("replay", shape, k)
        with torch.cuda.stream(s):
            g.replay()
        torch.cuda.synchronize()
        Q = lib.Plan(**prob, weights="fe")
        Q.rk3_step(ref, cfl=0.4)
        assert torch.equal(X, ref)
