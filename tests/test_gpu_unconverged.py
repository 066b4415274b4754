"""Domains whose A rounds to an indefinite matrix are counted: the stages end at
their cap or at a value that is not finite, and say so, on both FP64 paths."""
import pytest

from paper_1310_5954_amd import FP64, Filter, Problem
from workload.configs import build_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [100, 128, 130])
def test_numerically_indefinite_domains_are_counted(m):
    """Fewer slopes than members leave A's null directions at (m-1)/rho; under
    slope weights of 1e25 times their size its rounding errors are far above
    that, and of either sign.  The same domains converge at their own weights."""
    case = build_case(1, m=m)
    ptr = case.dmap.obs_ptr
    deficient = sum(2 * int(ptr[l + 1] - ptr[l]) < m - 8 for l in range(case.dmap.n_domains))
    assert deficient > 0
    for scale in (1.0, 1e25):
        case.r_inv = case.r_inv * scale
        f = Filter(Problem.from_case(case), case.X0, precision=FP64)
        f.analyse(case.slopes(0))
        n = f.unconverged()
        f.close()
        print(f"m={m} scale={scale:g}: {n} unconverged, {deficient} deficient", flush=True)
        assert n == 0 if scale == 1.0 else n > 0
