"""LDS-poison debug build, the kernels that came after the first list of cases: the
direct coarsest solve over several workgroups (k_direct_plane, k_direct_axis) and in
the coarse tail, the column form of the tail with its ragged and short segments
(k_tail_col) and the convergence test inside it, the one-launch strokes of small 3-D
and of 2-D levels (k_brick_down / up with both segment lengths, k_win2_down / up), the
residual march (k_defect), and the stage chunks in packed strips."""
import pytest

import test_gpu_lds_poison as first

pytestmark = pytest.mark.gpu

CASES = [
    "tests/test_gpu_direct.py",
    "tests/test_gpu_tail_column.py",
    "tests/test_gpu_tail_check.py",
    "tests/test_gpu_windows.py",
    "tests/test_gpu_windows_2d.py",
    "tests/test_gpu_defect.py",
    "tests/test_gpu_chunk_forms.py",
]


@pytest.mark.timeout(900)
def test_stroke_kernels_read_only_what_they_wrote(monkeypatch):
    monkeypatch.setattr(first, "CASES", CASES)
    first.test_lds_kernels_read_only_what_they_wrote()
