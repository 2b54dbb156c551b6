"""Stage chunks of large-s tau-steps (rkl_relax_solve, App. B) on float64 grids
large enough for the four-row strips: remainder columns packed into shared
wavefronts (130 = 2 x 60 + 10, 64 = 60 + 4), several planes a chunk (a grid with
more strips than the device has slots for one-plane chunks) and remainder rows.
Smaller grids (test_gpu_chunks.py) take the two-row strips.  Same comparison and
tolerance as there: identical tau-step counts against the oracle's stage-by-stage
recurrence, 1e-10 of the max norm."""
import numpy as np
import pytest

from oracle import multigrid as omg
from oracle import operators as oop

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(40, 90, 130), (170, 66, 64)])
@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("s,steps", [(5, 3), (6, 3)])
def test_four_row_chunks_match_oracle(shape, bc, s, steps):
    import paper_2306_05332_amd as R
    nz, ny, nx = shape
    h = (0.05, 0.04, 0.06)
    rng = np.random.default_rng(29 + s)
    f = rng.standard_normal(shape) * 100.0
    if bc == "periodic":
        f -= f.mean()
    faces = None
    if bc == "dirichlet":
        faces = tuple(rng.standard_normal(q) for q in ((nz, ny), (nz, ny), (nz, nx), (nz, nx), (ny, nx), (ny, nx)))
    g = oop.Grid(nx, ny, nz, *h, bc)
    u, it, _, _ = omg.relax_solve(f, g, "rkl", faces=faces, tol_max=0.0, max_iters=steps, s=s, theta=0.9)
    assert it == steps
    phi, st = R.relax_solve(torch.from_numpy(f).cuda(), h, bc, "rkl", faces=R.pack_faces(faces) if faces else None,
                            s=s, tol_max=0.0, max_iters=steps, raise_on_error=False)
    assert st.cycles == steps
    assert np.abs(phi.cpu().numpy() - u).max() < 1e-10 * np.abs(u).max()
