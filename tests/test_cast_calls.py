"""The kernels a current-scaling cast launches, read from its calls on the fake HIP runtime."""
import re

import pytest

from tests.fake_hip import ADDR, calls


def launched(qe, hip, entry, rows, cols):
    hip.clear()
    meta = qe.FP8Meta(ADDR, ADDR, ADDR, 1, 0, qe.E4M3, 0, 0)
    assert getattr(qe, entry)(ADDR, qe.F32, rows, cols, meta, ADDR, cols, ADDR, max(rows, 1), ADDR, 0, stream=0) == "OK"
    return [re.search(r"\d+([a-z_]+_kernel)", w[2])[1] for w in hip.log("launch")]


AMAX_UPDATE_CAST = ["amax_kernel", "scale_update_kernel", "quantize_kernel"]


@pytest.mark.parametrize("rows", [1, 4095, 4096])
def test_noalloc_takes_two_launches_up_to_64_mb(rows):
    assert calls(launched, "qe_quantize_fp8_current_noalloc", rows, 4096) == ["amax_kernel", "quantize_current_kernel"]


def test_noalloc_takes_four_launches_beyond():
    assert calls(launched, "qe_quantize_fp8_current_noalloc", 4097, 4096) == ["fill_zero_kernel"] + AMAX_UPDATE_CAST


def test_noalloc_of_an_empty_tensor_updates_and_casts():
    """No amax pass: the scale stays and the snapshot is written."""
    assert calls(launched, "qe_quantize_fp8_current_noalloc", 0, 4096) == ["fill_zero_kernel", "scale_update_kernel", "quantize_kernel"]


def test_current_cast_takes_three_launches():
    assert calls(launched, "qe_quantize_fp8_current", 4096, 4096) == AMAX_UPDATE_CAST
