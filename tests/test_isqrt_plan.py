"""The stages of A^(-1/2) (isqrt_plan.hpp) on scalars: every row of the table
must map each eigenvalue of its interval [1/kappa, 1] to its inverse square
root (CPU only; the coefficients as the kernels read them)."""
import os
import re

import numpy as np
import pytest

PLAN = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1310_5954_amd", "csrc", "isqrt_plan.hpp")
PRODUCTS = {1: 0, 2: 1, 4: 2, 6: 3}


def _rows():
    text = open(PLAN).read()
    rows = []
    for n, products, deg, body in re.findall(r"\{(\d+), (\d+), \{([\d, ]+)\}, \{(.*?)\n    \}\},", text, re.S):
        coef = [[np.longdouble(v) for v in line.split(",")] for line in re.findall(r"\{([^{}]+)\}", body)]
        rows.append((int(n), int(products), [int(v) for v in deg.split(",")], coef))
    return rows


ROWS = _rows()


def test_every_row_is_there():
    assert len(ROWS) == int(re.search(r"kIsqrtRows = (\d+);", open(PLAN).read()).group(1))


@pytest.mark.parametrize("r", range(1, len(ROWS)))
def test_row_gives_the_inverse_square_root(r):
    n, products, deg, coef = ROWS[r]
    assert len(coef) == n and all(deg[:n]) and not any(deg[n:])
    # a stage: its polynomial, P Z (not in the first), P (P M) (not in the last)
    assert products == sum(PRODUCTS[k] for k in deg[:n]) + 3 * (n - 1)
    x = np.longdouble(2) ** (-np.linspace(0, 1, 4001).astype(np.longdouble) * r / 2)  # eigenvalues of A / beta
    m, z = x.copy(), np.ones_like(x)
    for s in range(n):
        t = m - 1 if s + 1 == n else m
        p = sum(c * t ** k for k, c in enumerate(coef[s]))
        z, m = z * p, m * p * p
    # the generator's 1e-15, the coefficients' rounding to 20 digits, and this
    # replay's: up to 16000 eps of the first stages' alternating sums
    assert np.max(np.abs(z * np.sqrt(x) - 1)) < 1e-15 + 11 * 16000 * float(np.finfo(np.longdouble).eps)
