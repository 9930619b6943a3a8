"""bcsr_spmv where one wave of a workgroup would have more than half of its
blocks, at both sides of the two limits that send the rows to all its waves
(256 and 512 blocks for FP64 and FP32 values; half of the workgroup's 16 and
32 rows), under the bound of the tests of the other splits."""

import pytest

import test_gpu_spmv_rows as rows

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = {
    "f64_wave": [64, 64, 64, 64] + [3] * 12 + [64, 64, 64, 65] + [3] * 12,
    "f64_half": [300, 0, 0, 0] + [25] * 12 + [300, 0, 0, 0] + [25] * 11 + [26] + [0, 0, 0, 301] + [25] * 11 + [24],
    "f32_wave": [512] + [0] * 7 + [3] * 24 + [513] + [0] * 7 + [3] * 24,
    "f32_half": [600] + [0] * 7 + [25] * 24 + [600] + [0] * 7 + [25] * 23 + [24] + [0] * 7 + [601] + [25] * 24,
    "ragged": [7] * 16 + [5, 290, 0],
}


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("name", list(CASES))
def test_spmv_uneven_waves(name, dtype, monkeypatch):
    monkeypatch.setattr(rows, "CASES", CASES)
    rows.test_spmv_row_split(name, dtype)
