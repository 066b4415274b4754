"""The tables of isqrt_plan.hpp as the kernels take them: coefficients rounded to
binary64, degrees that the kernels have code for, and the property that the
stages rely on when the condition number was underestimated: an eigenvalue
below a stage's interval stays in (0, 1) and gains at least what its lower end
does; none passes 1 for the rounding of the coefficients (CPU only)."""
import os
import re

import numpy as np
import pytest

PLAN = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1310_5954_amd", "csrc", "isqrt_plan.hpp")
TEXT = open(PLAN).read()
L = np.longdouble


def _values(line):
    return [L(float(v)) for v in line.split(",")]  # as the compiler rounds them


ROWS = [([int(v) for v in deg.split(",")][:int(n)], [_values(line) for line in re.findall(r"\{([^{}]+)\}", body)])
        for n, _, deg, body in re.findall(r"\{(\d+), (\d+), \{([\d, ]+)\}, \{(.*?)\n    \}\},", TEXT, re.S)]
ENTRIES = [(int(n), _values(c)) for n, c in
           re.findall(r"\{(\d+), \{([^}]*)\}\},", re.search(r"kIsqrtStage4\[kIsqrtEntries\] = \{\n(.*?)\n\};", TEXT, re.S).group(1))]
LAST = [_values(c) for c in re.findall(r"\{([^}]*)\}", re.search(r"kIsqrtLast\[3\]\[7\] = \{\n(.*?)\n\};", TEXT, re.S).group(1))]
RHO = [float(v) for v in re.search(r"kIsqrtRho\[3\] = \{([^}]*)\}", TEXT).group(1).split(",")]
EPS = 2.0 ** -53


def poly(c, t):
    return sum(v * t ** k for k, v in enumerate(c))


def kappa(r):
    return 2.0 ** (r / 2) if r else 1.05


def test_sizes():
    assert len(ROWS) == int(re.search(r"kIsqrtRows = (\d+);", TEXT).group(1))
    assert len(ENTRIES) == int(re.search(r"kIsqrtEntries = (\d+);", TEXT).group(1)) == 2 * (len(ROWS) - 1)
    assert max(len(d) for d, _ in ROWS) <= int(re.search(r"kIsqrtStages = (\d+);", TEXT).group(1))
    assert [len(c) for c in LAST] == [3, 5, 7]


@pytest.mark.parametrize("k", [0, 1, 2])
def test_last_stage_is_exact_to_rounding(k):
    """(1 + R)^(-1/2) for R in [-rho, 0]: the generator's 2e-16, and the rounding of
    coefficients that sum to 1 + rho / 2 and little more."""
    R = -np.linspace(0, 1, 4001).astype(L) * L(RHO[k])
    assert np.max(np.abs(poly(LAST[k], R) * np.sqrt(1 + R) - 1)) < 2e-16 + 1.1 * EPS


@pytest.mark.parametrize("r", range(len(ROWS)))
def test_row(r):
    deg, coef = ROWS[r]
    assert len(deg) >= 2 and set(deg[:-1]) == {4} and deg[-1] in (2, 4, 6)
    assert [len(c) for c in coef] == [d + 1 for d in deg]
    assert coef[-1] == LAST[deg[-1] // 2 - 1]
    low = L(1) / L(kappa(r))
    x = low ** np.linspace(0, 1, 4001).astype(L)
    m, z = x.copy(), np.ones_like(x)
    below = low * np.array([0.9, 0.3, 1e-2, 1e-4], dtype=L)
    for c in coef[:-1]:
        p = poly(c, m)
        z, m = z * p, m * p * p
        gain = np.min(m) / low
        q = poly(c, below)
        below, low = below * q * q, np.min(m)
        assert np.all(m > 0) and np.max(m) < 1
        assert np.all(below > 0) and np.max(below) < 1
        assert gain > 1
    assert 1 - low <= RHO[deg[-1] // 2 - 1] / 2  # room for the kernels' bound of the norm
    p = poly(coef[-1], m - 1)
    assert np.max(np.abs(z * p * np.sqrt(x) - 1)) < 1e-15


@pytest.mark.parametrize("i", range(1, len(ENTRIES) + 1))
def test_entry_of_degree_four(i):
    nxt, c = ENTRIES[i - 1]
    assert nxt < i and len(c) == 5
    low = L(2) ** (-L(i) / 4)
    x = low ** np.linspace(0, 1, 4001).astype(L)
    m = x * poly(c, x) ** 2
    assert np.max(m) < 1
    assert np.min(m) >= (L(2) ** (-L(nxt) / 4) if nxt else 1 - RHO[1] / 2)
    below = low * np.array([0.9, 0.3, 1e-2, 1e-4], dtype=L)
    left = below * poly(c, below) ** 2
    assert np.all(left > 0) and np.max(left) < 1
    assert np.all(left / below >= np.min(m) / low * (1 - 1e-12))
