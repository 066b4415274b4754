"""The analysis launch is sized by the kernel that it runs: the polynomial
stages of the plain FP64 path have other registers and LDS than the Jacobi
kernel of the remaining forms, and at 65..128 members a grid of their own."""
import pytest

from paper_1310_5954_amd import FP64, Filter, Problem
from paper_1310_5954_amd import _lib as L
from test_kernel_resources import LDS_PER_CU, _resources
from workload.configs import build_case

pytestmark = pytest.mark.gpu


def _resident(kernel, waves):
    """Workgroups a CU holds at once, by the build's record of the kernel."""
    names = [n for n in _resources() if kernel in n]
    assert len(names) == 1, names
    r = _resources()[names[0]]
    return min(r["waves_per_simd"] * 4 // waves, LDS_PER_CU // r["lds_bytes"])


@pytest.mark.parametrize("m", [16, 32, 64, 100])
@pytest.mark.parametrize("obs_instant", [0, 1])
def test_blocks_per_cu_is_that_of_the_kernel_that_runs(m, obs_instant):
    case = build_case(1, m=m)
    f = Filter(Problem.from_case(case, obs_instant=obs_instant), case.X0, precision=FP64)
    f.step(case.slopes(0))
    M = next(k for k in (16, 32, 64, 128) if m <= k)
    kernel = f"k_analysisILi0ELi{M}E" if obs_instant else f"k_analysis_polyILi{M}E"
    assert f.autotune(reps=1)["blocks_per_cu"] == _resident(kernel, 8 if M == 128 else 4)
    f.close()


def test_no_grid_beyond_the_parking_slots_is_tuned_or_reported():
    """At 65..128 members the polynomial stages run at most 256 workgroups: on
    a map of more domains the candidates are half the CUs and one each (by the
    four orders), not one a domain as well, which would be the same launch."""
    case = build_case(3, m=66)
    assert case.dmap.n_domains > 256
    f = Filter(Problem.from_case(case), case.X0, precision=FP64)
    f.step(case.slopes(0))
    t = f.autotune(reps=1)
    assert t["blocks_per_cu"] == 1 and t["candidates"] == 8 and t["grid"] <= 256, t
    f.set_tuning(4096, L.ORDER_MAP)  # accepted as before; launched with the slots there are
    a = f.step(case.slopes(1))
    assert f.unconverged() == 0 and a.shape == (f.problem.n_act,)
    f.close()
