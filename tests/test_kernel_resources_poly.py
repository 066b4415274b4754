"""Register and LDS figures of the polynomial-stage kernels, which the plain
FP64 path runs (CPU only, by the build's record): three workgroups per CU at
M = 64, two wavefronts per SIMD (one workgroup of eight) at M = 128."""
import pytest

from test_kernel_resources import LDS_PER_CU, _resources


@pytest.mark.parametrize("m, groups, waves, vgprs", [(16, 4, 4, 128), (32, 4, 4, 128), (64, 3, 3, 168), (128, 1, 2, 256)])
def test_poly_kernels_keep_their_residency(m, groups, waves, vgprs):
    ks = _resources()
    names = [n for n in ks if n.startswith(f"_ZN5letkf15k_analysis_polyILi{m}E")]
    assert len(names) == 1, names
    r = ks[names[0]]
    assert r["waves_per_simd"] >= waves and r["vgprs"] + r["agprs"] <= vgprs, r
    assert groups * r["lds_bytes"] <= LDS_PER_CU, r
    assert r["scratch_bytes"] == 0 and r["vgpr_spill"] == 0, r
