"""Eigenvalues of a debug record past 128 members: the requested domain's alone
are computed, whichever it is and however often."""
import numpy as np
import pytest

from paper_1310_5954_amd import FP64, Filter, Problem
from workload.configs import build_case

pytestmark = pytest.mark.gpu


def test_each_domain_s_eigenvalues_in_any_order():
    case = build_case(1, m=130)
    f = Filter(Problem.from_case(case), case.X0, precision=FP64, debug=True)
    f.step(case.slopes(0))
    shift = (case.m - 1) / case.inflation
    for l in (15, 0, 6, 15):
        g = f.debug_domain(l)
        want = np.linalg.eigvalsh(g["C"] + shift * np.eye(case.m))
        # both are backward stable: m rounding errors of the largest eigenvalue
        assert np.abs(g["lam"] - want).max() <= 10 * case.m * 2.0 ** -53 * want.max()
    f.close()
