"""Ragged batches whose FE or PFE maps are neither the shared exponential's nor
staircases, around the numbers of windows up to which the one-launch step serves
calls of one step (768) and of more (1024): calls of both kinds on one plan, bit
for bit the sweeps' steps (a capped call takes those)."""
import numpy as np
import pytest
import torch

from gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


def _windows(nprob, n):
    # the problems, each with its 12 ghosts a side, end to end in windows of 109 slots
    return -(-nprob * (n + 24) // 109)


@pytest.mark.parametrize("nprob,n", [(691, 97), (692, 97), (922, 97), (923, 97), (2536, 9), (2537, 9)])
@pytest.mark.parametrize("opt", [dict(weights="fe", xi=500.0), dict(weights="pfe", zpow=3)],
                         ids=["fe", "pfe"])
def test_calls_on_both_sides_of_the_lines(W, nprob, n, opt):
    from paper_2306_09760_amd import solver
    say("run-time maps", nprob, n, _windows(nprob, n), opt)
    one = W.random_smooth_state(n, 1, (n,), amp=0.15)[1]
    U = np.concatenate([one * (1.0 + 1e-3 * (p % 17)) for p in range(nprob)], axis=1)
    off, h = np.arange(nprob + 1) * n, np.full(nprob, 1.0 / n)
    out = []
    for cap in (None, 1 << 20):
        B = solver.BatchPlan(off, h, bc="transmissive", **opt)
        X, t = to_dev(U), torch.zeros(nprob, dtype=torch.float64, device="cuda")
        status = torch.zeros(1, dtype=torch.int32, device="cuda")
        for k in (1, 3, 1, 2):
            B.rk3_steps(X, t, 1e9, cfl=0.5, nsteps=k, status=status, max_live=cap)
        out.append((X, t, B.last_dt().clone(), status))
    for a, b in zip(*out):
        assert torch.equal(a, b)
    assert bool(torch.isfinite(out[0][0]).all()) and not int(out[0][3].item())
