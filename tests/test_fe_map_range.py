"""Range of the three maps' denominators in the device's FE fast path: with
X_0, X_1 = 2^-s e^(2 xi w_k), X_2 = X_0 X_1 and the terms X + k_j, the log of
the product of the ten terms stays within +-600 over the simplex of weights,
for the shift s that centres its bounds, at every steepness the fast path
takes (the vertex bound B below 600, see test_fe_product_bound)."""
import numpy as np
import pytest

PSI = {"wcns": ((0, 1 / 16, 1 / 11, 1), (0, 10 / 16, 2 / 3, 10 / 11, 1), (0, 5 / 16, 1 / 3, 1)),
       "weno": ((0, 1 / 10, 1 / 7, 1), (0, 6 / 10, 2 / 3, 6 / 7, 1), (0, 3 / 10, 1 / 3, 1))}


def _null_points(family, kappa=0.5):
    return [[kappa * (p[j] + p[j - 1]) for j in range(1, len(p))] for p in PSI[family]]


def _log_product(w, nu, xi, s):
    """ln prod (X_m + k_j) at the weights w (3, n)."""
    ln2 = np.log(2.0)
    t = 0.0
    for m in range(3):
        x = 2 * xi * w[m] - s * ln2 if m < 2 else 2 * xi * (w[0] + w[1]) - 2 * s * ln2
        for v in nu[m]:
            k = 2 * xi * v - s * ln2 if m < 2 else 2 * xi * (1 - v) - 2 * s * ln2
            t = t + np.logaddexp(x, k)
    return t


@pytest.mark.parametrize("family", ["wcns", "weno"])
@pytest.mark.parametrize("xi", [10.0, 100.0, 127.0])
def test_denominator_product_stays_in_range(family, xi):
    nu = _null_points(family)
    corners = np.eye(3)
    top = _log_product(corners, nu, xi, 0).max()
    low = sum(np.logaddexp(0.0, 2 * xi * v) for m in (0, 1) for v in nu[m]) + \
        sum(np.logaddexp(0.0, 2 * xi * (1 - v)) for v in nu[2])
    s = np.rint((top + low) / (26 * np.log(2.0)))
    w = np.random.default_rng(3).dirichlet((0.3, 0.3, 0.3), 200000).T
    w = np.concatenate([w, corners, np.full((3, 1), 1 / 3)], axis=1)
    t = _log_product(w, nu, xi, s)
    assert t.max() <= top - 13 * s * np.log(2.0) + 1e-9     # the vertex is the peak
    assert t.min() >= low - 13 * s * np.log(2.0) - 1e-9
    assert t.max() < 600 and t.min() > -600
