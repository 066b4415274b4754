"""A^(-1/2) by polynomial stages over the condition numbers and sizes where its
stages, tiles and padding change: T against the FP64 oracle, every domain."""
import numpy as np
import pytest

import oracle
from paper_1310_5954_amd import FP64, Filter, Problem, Server
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


@pytest.mark.parametrize("m", [2, 15, 16, 17, 32, 33, 48, 49, 64, 65, 80, 81, 96, 97, 112, 113, 128])
@pytest.mark.parametrize("scale", [1e-6, 1e-2, 1.0, 1e3])
def test_T_over_condition_numbers(m, scale):
    check_T(m, scale)


@pytest.mark.parametrize("m", [16, 64, 128])
def test_batch_of_both_solvers_equals_the_plain_path(m):
    """Instances that observe phi_k and phi_{k-1} share a class but not an
    analysis kernel; served together they give the plain path's states."""
    case = build_case(1, m=m)
    problems = [Problem.from_case(case, obs_instant=o) for o in (0, 1, 0)]
    plain = []
    for p in problems:
        f = Filter(p, case.X0, precision=FP64)
        for k in range(2):
            f.step(case.slopes(k))
        plain.append(f.get_state()[0])
        f.close()
    srv = Server(sum(p.workspace_size(FP64) + (1 << 16) for p in problems) + (64 << 20), max_batch=3)
    inst = [srv.add(p, case.X0, FP64) for p in problems]
    for k in range(2):
        for i, x in enumerate(inst):
            assert srv.submit(x, case.slopes(k), 3 * k + i) == 0
    srv.drain()
    for x, want in zip(inst, plain):
        assert np.array_equal(x.get_state()[0], want)
    srv.close()
