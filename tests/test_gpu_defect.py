"""Residual of 3-D grids against the oracle at the edges of its tiles: rows of 1
to 130 columns around the 64 of a wavefront (a last tile that ends at the last
column overlaps the one before it), row counts around the 16 of a workgroup, one
to many chunks of planes, face data, and the norm.  Tolerances: float64 as the
other residual tests (1e-13 of the largest residual, 1e-12 of the norm); float32
2e-6 (about ten roundings of 6e-8 in M u at the size of its largest value, which
is the residual's), the norm being summed in float64 of float32 residuals."""
import numpy as np
import pytest

from oracle import operators as oop

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(4, 5, 63), (18, 16, 64), (33, 17, 65), (3, 40, 128), (40, 15, 129), (2, 2, 2), (70, 64, 130)]


def relmax(a, b):
    return np.abs(a - b).max() / max(np.abs(b).max(), 1e-300)


@pytest.mark.parametrize("bc", ["periodic", "dirichlet", "faces"])
@pytest.mark.parametrize("shape", SHAPES)
def test_residual_tiles_match_oracle(shape, bc):
    import paper_2306_05332_amd as R
    nz, ny, nx = shape
    rng = np.random.default_rng(sum(shape))
    h = (0.11, 0.07, 0.13)
    u, f = rng.standard_normal(shape), rng.standard_normal(shape)
    faces = None
    if bc == "faces":
        bc = "dirichlet"
        faces = tuple(rng.standard_normal(q) for q in ((nz, ny), (nz, ny), (nz, nx), (nz, nx), (ny, nx), (ny, nx)))
    want = -oop.residual(u, f, h, bc, faces)
    norm = np.linalg.norm(want)
    cu = lambda a, dt: torch.from_numpy(a).to("cuda", dt)
    packed = R.pack_faces(faces) if faces else None
    r, n = R.residual(cu(f, torch.float64), cu(u, torch.float64), h, bc, faces=packed)
    assert relmax(r.cpu().numpy(), want) < 1e-13 and abs(n - norm) < 1e-12 * norm
    r, n = R.residual_noalloc(cu(f, torch.float64), cu(u, torch.float64), h, bc, faces=packed)
    assert relmax(r.cpu().numpy(), want) < 1e-13 and abs(float(n) - norm) < 1e-12 * norm
    if faces is None:
        r, n = R.residual(cu(f, torch.float32), cu(u, torch.float32), h, bc)
        assert relmax(r.double().cpu().numpy(), want) < 2e-6 and abs(n - norm) < 2e-6 * norm
