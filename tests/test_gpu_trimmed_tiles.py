"""The 3D Euler y and z tiles of four and eight columns, which keep a field's
states in registers and two variables' node fluxes in the nodes' place: bitwise
the residual of the 32 x 4 tiles, for odd extents around the tiles' edges, both
differences and boundary types, and every kernel of weights."""
import ctypes as C

import pytest
import torch

from gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2306_09760_amd import solver
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return solver


def _residual(lib, prob, opt, U, tiles):
    from paper_2306_09760_amd import _lib
    P = lib.Plan(**{**prob, **opt})
    lib.check(_lib.lib().wcns_plan_set_tiles(P._h, (C.c_int32 * 3)(*tiles)), "wcns_plan_set_tiles")
    return P.residual(to_dev(U))


@pytest.mark.parametrize("shape", [(9, 10, 11), (15, 29, 30), (17, 61, 62), (13, 33, 58)])
@pytest.mark.parametrize("bc", ["transmissive", "periodic"])
@pytest.mark.parametrize("weights,xi", [("fe", 100.0), ("z", 100.0), ("js", 100.0), ("pfe", 100.0),
                                        ("fe", 1e6), ("fe", 500.0)])
def test_residual_of_every_tile(lib, W, shape, bc, weights, xi):
    prob, U = W.random_smooth_state(sum(shape), 3, shape, amp=0.2)
    for diff, charproj in (("mnd6", True), ("md6", True), ("mnd6", False)):
        opt = dict(weights=weights, xi=xi, diff=diff, charproj=charproj, bc=bc)
        say("trimmed tiles", shape, opt)
        ref = _residual(lib, prob, opt, U, (128, 32, 4))
        assert bool(torch.isfinite(ref).all())
        for tiles in ((256, 32, 8), (256, 64, 4), (256, 128, 2)):
            assert torch.equal(_residual(lib, prob, opt, U, tiles), ref), tiles
