"""One-launch strokes of two-dimensional levels, through V-cycles against the
oracle's: windows of 64 columns by 32 rows (levels up to about 1024^2) and by 48
rows (beyond), boxes smaller than a window, windows that overhang the box, every
stage count they accept, and strokes of more stages, which keep the separate
passes.  Tolerances of the other V-cycle tests (1e-11 float64, 1e-5 float32): both
sides run the same recurrence and solve the coarsest system to 1e-13 of its
right-hand side.  The coarsest level of 160 x 1100 (40 x 275, periodic) is too
ill-conditioned for the direct solve's rule and iterates, in float32 to 1e-6 of
its right-hand side, which 275^2 modes amplify beyond any such bound (1.0e-4,
with or without the one-launch strokes): float64 only."""
import numpy as np
import pytest

from oracle import multigrid as omg
from oracle import operators as oop

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (ny, nx) of the finest level
SHAPES = [(12, 20), (20, 104), (64, 64), (130, 66), (160, 1100), (1440, 1504)]


def relmax(a, b):
    return np.abs(a - b).max() / max(np.abs(b).max(), 1e-300)


def _check(shape, bc, **opt):
    import paper_2306_05332_amd as R
    rng = np.random.default_rng(sum(shape))
    h = (0.11, 0.07)
    f = rng.standard_normal(shape) * 50
    if bc == "periodic":
        f -= f.mean()
    u = rng.standard_normal(shape)
    g = oop.grid2d(shape[1], shape[0], *h, bc)
    want = omg.vcycle(u[None], f[None], oop.build_hierarchy(g), omg.Options(**opt), None)[0]
    dtypes = [(torch.float64, 1e-11)] + ([] if shape == (160, 1100) else [(torch.float32, 1e-5)])
    for dt, tol in dtypes:
        phi = torch.from_numpy(u).to("cuda", dt)
        R.vcycle(torch.from_numpy(f).to("cuda", dt), phi, h, bc, opts=R.Options(**opt))
        assert relmax(phi.double().cpu().numpy(), want) < tol


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("shape", SHAPES)
def test_window_strokes_2d_match_oracle(shape, bc):
    _check(shape, bc)


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("s,n_pre,n_post", [(1, 1, 1), (1, 4, 3), (2, 1, 2), (3, 1, 1), (4, 1, 1), (2, 3, 3), (2, 2, 0)])
def test_window_sweeps_2d_match_oracle(s, n_pre, n_post, bc):
    _check((144, 176), bc, s=s, n_pre=n_pre, n_post=n_post)
