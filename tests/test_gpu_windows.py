"""One-launch strokes of small levels (a workgroup per window with its halo),
through V-cycles against the oracle's.

Levels of 20^3 to 64 x 48 x 80 take them (the finest one too, from the given
iterate, up to about 48^3); shapes cover
windows that overhang the box on every axis, boxes shorter than a window, both
segment lengths (64 x 48 x 80 needs the longer one) and every stage count they
accept (n_pre s and n_post s of 1 to 4), with strokes of more stages falling back
to the strip kernels.  Tolerances of the other V-cycle tests (1e-11 float64, 1e-5
float32): both sides run the same recurrence and solve the coarsest system to
1e-13 of its right-hand side."""
import numpy as np
import pytest

from oracle import multigrid as omg
from oracle import operators as oop

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (nz, ny, nx) of the finest level
SHAPES = [(32, 32, 32), (56, 24, 40), (40, 40, 40), (80, 80, 80), (72, 44, 100), (24, 200, 56), (160, 96, 128)]


def relmax(a, b):
    return np.abs(a - b).max() / max(np.abs(b).max(), 1e-300)


def _check(shape, bc, **opt):
    import paper_2306_05332_amd as R
    rng = np.random.default_rng(sum(shape))
    h = (0.11, 0.07, 0.13)
    f = rng.standard_normal(shape) * 50
    if bc == "periodic":
        f -= f.mean()
    u = rng.standard_normal(shape)
    g = oop.Grid(shape[2], shape[1], shape[0], *h, bc)
    want = omg.vcycle(u, f, oop.build_hierarchy(g), omg.Options(**opt), None)
    for dt, tol in ((torch.float64, 1e-11), (torch.float32, 1e-5)):
        phi = torch.from_numpy(u).to("cuda", dt)
        R.vcycle(torch.from_numpy(f).to("cuda", dt), phi, h, bc, opts=R.Options(**opt))
        assert relmax(phi.double().cpu().numpy(), want) < tol


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("shape", SHAPES)
def test_window_strokes_match_oracle(shape, bc):
    _check(shape, bc)


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("s,n_pre,n_post", [(1, 1, 1), (1, 4, 3), (2, 1, 2), (3, 1, 1), (4, 1, 1), (2, 3, 3)])
def test_window_sweeps_match_oracle(s, n_pre, n_post, bc):
    _check((80, 56, 72), bc, s=s, n_pre=n_pre, n_post=n_post)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_batches_that_overfill_the_windows_equal_single_solves(prec):
    """Twelve members run strips where one runs windows: the same arithmetic, so
    the same answers (the bound of the other batch tests)."""
    import paper_2306_05332_amd as R
    rng = np.random.default_rng(4)
    rhos, hs = [], []
    for _ in range(12):
        r = rng.standard_normal((80, 80, 80))
        rhos.append(torch.from_numpy(r - r.mean()).cuda())
        hs.append((1.0 / 80,) * 3)
    o = R.Options(tol=1e-9, prec=prec)
    phis, stats = R.solve_batched(rhos, hs, "periodic", opts=o)
    for k in (0, 11):
        ref, sr = R.solve(rhos[k], hs[k], "periodic", opts=o)
        assert stats[k].cycles == sr.cycles
        np.testing.assert_allclose(stats[k].history, sr.history, rtol=1e-12, atol=0)
        assert relmax(phis[k].cpu().numpy(), ref.cpu().numpy()) < 1e-13
