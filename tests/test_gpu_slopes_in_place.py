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


def _step(f, pointer, out):
    return L.lib().letkf_step(f.handle, C.c_void_p(pointer), 1, out.ctypes.data_as(C.POINTER(C.c_double)) if out is not None else None,
                              C.c_void_p(torch.cuda.current_stream().cuda_stream))


def test_pinned_host_memory_passed_as_device_slopes_is_copied():
    case = build_case(1)
    p = Problem.from_case(case)
    ref, f = (Filter(p, case.X0, precision=FP64) for _ in range(2))
    y = torch.empty(p.p, dtype=torch.float64, pin_memory=True)
    y.copy_(torch.from_numpy(case.slopes(0)))
    want, got = ref.step(case.slopes(0)), np.empty(p.n_act)
    assert _step(f, y.data_ptr(), got) == L.OK
    assert np.array_equal(got, want)
    ref.close()
    f.close()


def test_device_slopes_that_end_before_their_count_are_refused():
    """One value short of the frame's 450 (3592 of the 3600 bytes, within a
    page): the copy command that takes what cannot be read in place refuses
    it, and the state stays."""
    case = build_case(1)
    p = Problem.from_case(case)
    f = Filter(p, case.X0, precision=FP64)
    before = f.get_state()[0]
    loaded = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    hip = C.CDLL(loaded)
    short = C.c_void_p()
    assert p.p == 450 and hip.hipMalloc(C.byref(short), C.c_size_t(8 * (p.p - 1))) == 0
    for out in (np.empty(p.n_act), None):
        assert _step(f, short.value, out) == L.EDEVICE
    assert np.array_equal(f.get_state()[0], before)
    assert hip.hipFree(short) == 0
    f.close()


def test_a_refused_call_leaves_no_error_for_the_next():
    case = build_case(1)
    p = Problem.from_case(case)
    f = Filter(p, case.X0, precision=FP64)
    loaded = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    hip = C.CDLL(loaded)
    short = C.c_void_p()
    assert hip.hipMalloc(C.byref(short), C.c_size_t(8 * (p.p - 1))) == 0
    assert _step(f, short.value, None) == L.EDEVICE
    assert np.isfinite(f.step(case.slopes(0))).all()
    assert hip.hipFree(short) == 0
    f.close()
