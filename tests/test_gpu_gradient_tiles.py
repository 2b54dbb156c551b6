"""The acceleration kernel at the edges of its tiles: chunks of several planes
with a short last one, rows and columns past the last full tile, axes shorter
than the stencil beside long ones, and a wide single plane; against the oracle
at the tolerance of its other tests (a few rounding errors of the differences,
1e-13 of the largest component)."""
import numpy as np
import pytest

from oracle import gradient as ogr

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(90, 130, 200), (131, 65, 257), (3, 500, 66), (41, 2, 129), (37, 300, 3)])
@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
def test_gradient_tiles_match_oracle(shape, bc):
    import paper_2306_05332_amd as R
    rng = np.random.default_rng(sum(shape))
    h = (0.11, 0.07, 0.13)
    nz, ny, nx = shape
    phi = rng.standard_normal(shape)
    faces = None
    if bc == "dirichlet":
        faces = tuple(rng.standard_normal(s) for s in ((nz, ny),) * 2 + ((nz, nx),) * 2 + ((ny, nx),) * 2)
    want = ogr.acceleration(phi, h, bc, faces)
    got = R.gradient(torch.from_numpy(phi).cuda(), h, bc, R.pack_faces(faces) if faces else None)
    for g, w in zip(got, want):
        assert np.abs(g.cpu().numpy() - w).max() <= 1e-13 * np.abs(w).max()
