"""A^(-1/2) by polynomial stages over the condition numbers and sizes where its
stages, tiles and padding change: T against the FP64 oracle, every domain."""
import pytest

import oracle
from paper_1310_5954_amd import FP64, Filter, Problem
from workload.configs import build_case

from _helpers import rel, sparse_D

pytestmark = pytest.mark.gpu


def check_T(m, scale):
    """scale multiplies R^-1, so that kappa(A) runs from 1 to a few 1e7.  Bound:
    forming A rounds each entry by at most (p_l + 2) u, an error of A that both
    sides carry and that A^(-1/2) and A^-1 b turn into kappa times as much of T;
    32 kappa u covers it for the square root of the p_l <= 50 roundings on
    both sides, and 1e-12 the well-conditioned end."""
    case = build_case(1, m=m)
    case.r_inv = case.r_inv * scale
    f = Filter(Problem.from_case(case), case.X0, precision=FP64, debug=True)
    y = case.slopes(0)
    f.analyse(y)
    _, doms = oracle.analysis(case.X0, y, sparse_D(case), case.dmap, case.r_inv, case.inflation, keep_domains=True)
    for l in sorted({0, 1, len(doms) // 2, len(doms) - 1}):
        g, o = f.debug_domain(l), doms[l]
        kappa = float(o["lam"].max() / o["lam"].min())
        assert rel(g["T"], o["T"]) < 1e-12 + 32 * kappa * 2.0 ** -53, (l, kappa)
        assert rel(g["lam"], o["lam"]) < 1e-10
    assert f.unconverged() == 0
    f.close()


@pytest.mark.parametrize("m", [129, 144, 145, 208, 256])
@pytest.mark.parametrize("scale", [1e-6, 1e-2, 1.0, 1e3, 1e8])
def test_T_over_condition_numbers_large_ensembles(m, scale):
    check_T(m, scale)
