"""The forms a frame's slopes and means may take: slopes on the host (read in
pinned memory where the call waits for its means and there are few of them,
copied otherwise) or on the GPU, means wanted or not, launches or a graph.
Every form runs the same kernels on the same numbers, so states and means are
equal to the last bit, in any mixture."""
import numpy as np
import pytest
import torch

from paper_1310_5954_amd import FP32, FP64, Filter, Problem
from workload.configs import build_case

pytestmark = pytest.mark.gpu

# (slopes on the GPU, means wanted) of each frame
FORMS = [[(False, False)] * 6, [(False, True)] * 6, [(True, True)] * 6,
         [(False, True), (True, False), (False, False), (True, True), (False, False), (False, True)]]


# config 1: 450 slopes, 256 actuators; 2: 2528 and 1345; 3: 11088 (copied, too many to read in pinned memory) and 5713
@pytest.mark.parametrize("config,m,precision", [(1, 7, FP64), (2, 33, FP32), (3, 9, FP32), (1, 130, FP64)])
@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("graph", [False, True])
def test_every_form_gives_the_same_frames(config, m, precision, split, graph):
    case = build_case(config, m=m)
    got = []
    for forms in FORMS:
        f = Filter(Problem.from_case(case), case.X0, precision=precision, graph=graph)
        means = []
        for k, (dev, want) in enumerate(forms):
            y = np.ascontiguousarray(case.slopes(k % 3))
            given = torch.from_numpy(y).cuda() if dev else y.copy()
            if split:
                means.append(f.analyse(given, mean=want))
                f.forecast()
            else:
                means.append(f.step(given, pred=want))
            if not dev:
                given[:] = np.nan  # the caller's memory is its own again
        got.append((f.get_state(), means))
        f.close()
    (X, frame), _ = got[0]
    assert frame == len(FORMS[0]) and np.isfinite(X).all()
    for (Xi, fi), mi in got[1:]:
        assert fi == frame and np.array_equal(Xi, X)
        for a, b in zip(mi, got[1][1]):
            assert a is None or np.array_equal(a, b)
