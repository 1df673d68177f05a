"""The exponential of the FE maps (exp2_tab, wcns_probe_math) against its bound:
e^(2 xi w) within 2.7e-15 of x86 extended precision over |w| <= 1, exact at 0, a
NaN for a NaN."""
import ctypes as C
from decimal import Decimal, getcontext

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_map_exponential_within_its_bound():
    from paper_2306_09760_amd import _lib as L
    assert np.finfo(np.longdouble).nmant >= 63, "the reference needs x86 extended precision"
    rng = np.random.default_rng(12)
    w = np.concatenate([rng.uniform(-1.0, 1.0, 400000), rng.uniform(0.0, 1.0, 400000),
                        rng.uniform(-1e-3, 1e-3, 100000), [1.0, -1.0, 1e-300, 0.0, np.nan]])
    x = torch.from_numpy(w).cuda()
    out = torch.empty_like(x)
    L.check(L.lib().wcns_probe_math(C.c_void_p(x.data_ptr()), C.c_void_p(out.data_ptr()), w.size,
                                    6, None), "probe")
    y = out.cpu().numpy()
    assert np.isnan(y[-1]) and y[-2] == 1.0 and y[-3] == 1.0
    # X = 2^(w a / 64) with the rounded a
    getcontext().prec = 40
    a = np.longdouble(float(Decimal(2 * 100 * 64) / Decimal(2).ln()))
    ref = np.exp2(w[:-1].astype(np.longdouble) * a / 64)
    rel = np.abs((y[:-1].astype(np.longdouble) - ref) / ref)
    assert float(rel.max()) <= 2.7e-15, float(rel.max())
