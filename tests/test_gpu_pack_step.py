"""The one-launch step of small ragged batches: bitwise the sweeps' steps (which
a capped call runs on), for problems shorter than a stage's reach, tiles across
many problems, both boundary types and differences, all weight kinds, one to
five steps, problems that finish or are non-physical on the way, and a captured
step."""
import numpy as np
import pytest
import torch

from gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

BATCHES = [[9], [9] * 40, [9, 10, 11, 12, 13, 14, 15, 16, 17, 24, 25, 33], [85, 86, 108, 109, 110, 133],
           [1000, 9, 400, 61, 62], [300] * 30]
WEIGHTS = [("fe", 100.0), ("z", 100.0), ("js", 100.0), ("pfe", 100.0), ("fe", 1e6), ("fe", 500.0)]


@pytest.fixture(scope="module")
def lib():
    from paper_2306_09760_amd import solver
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return solver


def _batch(W, lengths, seed):
    U = np.concatenate([W.random_smooth_state(seed + k, 1, (n,), amp=0.15)[1]
                        for k, n in enumerate(lengths)], axis=1)
    return np.concatenate([[0], np.cumsum(lengths)]), [1.0 / n for n in lengths], U


def _run(lib, args, opt, U, t_end, steps, capped, status):
    B = lib.BatchPlan(*args, **opt)
    X = to_dev(U)
    t = torch.zeros(len(args[1]), dtype=torch.float64, device="cuda")
    for n in steps:
        B.rk3_steps(X, t, t_end, cfl=0.5, nsteps=n, status=status,
                    max_live=1 << 20 if capped else None)
    return X, t, B.last_dt().clone(), int(status.item())


@pytest.mark.parametrize("lengths", BATCHES, ids=lambda l: f"{len(l)}x{l[0]}")
@pytest.mark.parametrize("bc", ["transmissive", "periodic"])
@pytest.mark.parametrize("weights,xi", WEIGHTS)
def test_steps_equal_the_sweeps(lib, W, lengths, bc, weights, xi):
    off, h, U = _batch(W, lengths, len(lengths))
    for diff, charproj in (("mnd6", True), ("md6", False)):
        opt = dict(weights=weights, xi=xi, diff=diff, charproj=charproj, bc=bc)
        # the second end time: short problems take fewer steps than long ones
        for t_end, steps in ((1e9, (1, 2, 5)), (0.02, (3, 4))):
            say("packed steps", lengths[:4], opt, t_end)
            got, ref = (_run(lib, (off, h), opt, U, t_end, steps, capped,
                             torch.zeros(1, dtype=torch.int32, device="cuda")) for capped in (0, 1))
            assert torch.equal(got[0], ref[0]) and bool(torch.isfinite(ref[0]).all())
            assert torch.equal(got[1], ref[1]) and torch.equal(got[2], ref[2]) and got[3] == ref[3]


def test_non_physical_problem_stops_alone(lib, W):
    lengths = [40, 30, 200, 50]
    off, h, U = _batch(W, lengths, 7)
    U[2, off[1] + 3] = -1.0
    opt = dict(weights="fe", bc="transmissive")
    got, ref = (_run(lib, (off, h), opt, U, 1e9, (1, 3), capped,
                     torch.zeros(1, dtype=torch.int32, device="cuda")) for capped in (0, 1))
    assert got[3] == ref[3] == 1
    for a, b in zip(got[:3], ref[:3]):
        assert torch.equal(a.nan_to_num(7.0), b.nan_to_num(7.0))
    keep = [i for p in (0, 2, 3) for i in range(off[p], off[p + 1])]
    assert bool(torch.isfinite(got[0][:, keep]).all())


def test_graph_and_capture(lib, W):
    lengths = [300, 40, 500]
    off, h, U = _batch(W, lengths, 9)
    B, C = (lib.BatchPlan(off, h, weights="fe", bc="transmissive") for _ in range(2))
    t, tc = (torch.zeros(3, dtype=torch.float64, device="cuda") for _ in range(2))
    X, ref = to_dev(U), to_dev(U)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            B.rk3_steps(X, t, 1e9, cfl=0.4, nsteps=3)
    for k in range(4):
        say("replay", k)
        with torch.cuda.stream(s):
            g.replay()
        torch.cuda.synchronize()
        C.rk3_steps(ref, tc, 1e9, cfl=0.4, nsteps=3, max_live=1 << 20,
                    status=torch.zeros(1, dtype=torch.int32, device="cuda"))
        assert torch.equal(X, ref) and torch.equal(t, tc)
