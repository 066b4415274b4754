"""Slopes that the slope kernel reads where the caller has them: what it must
leave behind for the calls that use the frame's slopes again, and memory that
it must not read in place."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_1310_5954_amd import FP64, Filter, Problem
from paper_1310_5954_amd import _lib as L
from workload.configs import build_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("obs_instant", [0, 1])
def test_autotune_analyses_the_frame_s_slopes_in_every_form(obs_instant):
    """letkf_autotune analyses the current state with the slopes of the last
    frame: the debug record it leaves is the same whether they came by a copy
    command, in pinned memory or on the GPU (an older frame's lie behind them)."""
    case = build_case(1)
    p = Problem.from_case(case, obs_instant=obs_instant)
    got = []
    for on_gpu, mean in [(False, False), (False, True), (True, False), (True, True)]:
        f = Filter(p, case.X0, precision=FP64, debug=True)
        f.step(case.slopes(0), pred=False)  # by a copy command
        y = case.slopes(1)
        f.analyse(torch.from_numpy(y).cuda() if on_gpu else y, mean=mean)
        f.autotune(1)
        got.append([f.debug_domain(l)["T"] for l in (0, 5, 15)])
        f.close()
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.isfinite(a).all() and np.array_equal(a, b)
