"""Column form of the coarse tail, through V-cycles against the oracle's.

The finest level runs kernels of its own, so a tail starts at half its shape.
Shapes cover each cells-per-thread count (8^3: one; 12^3: two; 12 x 16 x 16:
three; 16^3: four), marches that leave a short last segment (10 and 14 planes of
256 cells, 58 rows of 52), planes that fill no wavefront (10 x 14), and both
coarsest solves (at most 64 cells and more).  Tolerances are those of the other
V-cycle tests (1e-11 float64, 1e-5 float32): both sides smooth with the same
recurrence and solve the coarsest system to 1e-13 of its right-hand side."""
import numpy as np
import pytest

from oracle import multigrid as omg
from oracle import operators as oop

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (nz, ny, nx) or (ny, nx) of the finest level
SHAPES = [(16, 16, 16), (24, 24, 24), (24, 32, 32), (32, 32, 32), (20, 32, 32), (28, 32, 32), (32, 20, 28),
          (128, 128), (116, 104), (56, 40)]


def relmax(a, b):
    return np.abs(a - b).max() / max(np.abs(b).max(), 1e-300)


def _check(shape, bc, **opt):
    import paper_2306_05332_amd as R
    rng = np.random.default_rng(sum(shape))
    h = (0.11, 0.07, 0.13)[: len(shape)]
    f = rng.standard_normal(shape) * 50
    if bc == "periodic":
        f -= f.mean()
    u = rng.standard_normal(shape)
    if len(shape) == 2:
        g = oop.grid2d(shape[1], shape[0], *h, bc)
        want = omg.vcycle(u[None], f[None], oop.build_hierarchy(g), omg.Options(**opt), None)[0]
    else:
        g = oop.Grid(shape[2], shape[1], shape[0], *h, bc)
        want = omg.vcycle(u, f, oop.build_hierarchy(g), omg.Options(**opt), None)
    for dt, tol in ((torch.float64, 1e-11), (torch.float32, 1e-5)):
        phi = torch.from_numpy(u).to("cuda", dt)
        R.vcycle(torch.from_numpy(f).to("cuda", dt), phi, h, bc, opts=R.Options(**opt))
        assert relmax(phi.double().cpu().numpy(), want) < tol


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("shape", SHAPES)
def test_tail_shapes_match_oracle(shape, bc):
    _check(shape, bc)


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("s,n_pre,n_post", [(1, 1, 1), (2, 2, 0), (3, 1, 2), (4, 3, 1)])
def test_tail_sweeps_match_oracle(s, n_pre, n_post, bc):
    _check((28, 32, 32), bc, s=s, n_pre=n_pre, n_post=n_post)
