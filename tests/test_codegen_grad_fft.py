"""CPU-only checks of the gradient and the register transforms as hipcc builds
them for gfx950: no register spills in any precision, storage form, gauge or
direction. (Asked for four waves a SIMD in every float form, the gradient of
8-real links spilled 197 registers and took twice its time.)"""
import shutil

import pytest

from test_codegen import device_asm, kernel_meta

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")


@pytest.mark.parametrize("src,kernel,count", [("grad.hip", "k_functional_grad", 12), ("fft.hip", "k_fft_line", 12)])
def test_no_spills(src, kernel, count, tmp_path):
    meta = {k: v for k, v in kernel_meta(device_asm(src, tmp_path)).items() if kernel in k}
    assert len(meta) >= count
    for name, m in meta.items():
        assert m["scratch"] == 0 and m["vgpr_spill"] == 0, (name, m)


def test_float_gradients_fit_their_waves(tmp_path):
    """Four waves a SIMD (128 registers) for full and 12-real links, three (168) for 8-real ones."""
    meta = {k: v for k, v in kernel_meta(device_asm("grad.hip", tmp_path)).items() if "k_functional_gradIf" in k}
    assert len(meta) == 6
    for name, m in meta.items():
        assert m["vgpr"] <= (168 if "IfLi4E" in name else 128), (name, m)
