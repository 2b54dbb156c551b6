"""Periodic compatibility with one mean removal per cycle: V-cycles whose
right-hand side has a mean (used as given on level 0, removed below) against
the oracle's, which removes it on every coarse level, with two to four coarse
levels above the tail; tolerances of the other V-cycle tests."""
import numpy as np
import pytest

from oracle import multigrid as omg
from oracle import operators as oop

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(16, 16, 16), (40, 24, 64), (96, 48, 80), (128, 64, 96)])
@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-11), (torch.float32, 1e-5)])
def test_vcycle_of_a_right_hand_side_with_a_mean(shape, dtype, tol):
    import paper_2306_05332_amd as R
    rng = np.random.default_rng(sum(shape))
    h = tuple(1.0 / n for n in shape[::-1])
    f = rng.standard_normal(shape) * 50 + 7.0
    u = rng.standard_normal(shape) * 0.01
    nz, ny, nx = shape
    want = omg.vcycle(u, f, oop.build_hierarchy(oop.Grid(nx, ny, nz, *h, "periodic")), omg.Options(), None)
    phi = torch.from_numpy(u).to("cuda", dtype)
    R.vcycle(torch.from_numpy(f).to("cuda", dtype), phi, h, "periodic")
    assert np.abs(phi.double().cpu().numpy() - want).max() < tol * np.abs(want).max()
