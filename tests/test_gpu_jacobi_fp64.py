"""The FP64 Jacobi kernel against the oracle at every padded size and its
remainders.  Plain FP64 filters run the polynomial stages, so the kernel is
reached through obs_instant = 1."""
import pytest

from paper_1310_5954_amd import FP64
from test_gpu_parity import _check_step, oracle_spin_up
from workload.configs import build_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [2, 27, 33, 64, 65, 100, 128])
def test_fp64_jacobi_sizes(m):
    case = build_case(1, m=m)
    X, k = oracle_spin_up(case, 2)
    _check_step(case, X, k, FP64, debug=True, obs_instant=1)
