"""Direct coarsest solve (the default when the caller leaves the coarse
tolerance alone): V-cycles against the oracle's, whose coarsest level runs the
accelerated RKL iteration to 1e-13 (float64) or is compared at float32's
tolerance.  Shapes cover every form: one tile per axis (4^3), several tiles in
one workgroup (6^3, 14 x 6 x 10, 2-D), tables too long for LDS (4 x 4 x 100),
the plane form (22 x 30 x 50) and one launch per axis (planes of 100 x 100).
Tolerances: both sides solve the coarsest system to 1e-13 of its right-hand
side or better, so the V-cycle bounds of the other tests hold (1e-11 float64,
1e-5 float32)."""
import math

import numpy as np
import pytest

from oracle import exact
from oracle import multigrid as omg
from oracle import operators as oop

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (nz, ny, nx) of the finest level
SHAPES = [(16, 16, 16), (48, 48, 48), (56, 24, 40), (8, 8, 200), (44, 60, 100), (20, 200, 200)]


def _lib():
    import paper_2306_05332_amd as R
    return R


def relmax(a, b):
    return np.abs(a - b).max() / max(np.abs(b).max(), 1e-300)


def _case(shape, bc, seed):
    rng = np.random.default_rng(seed)
    h = (0.11, 0.07, 0.13)
    f = rng.standard_normal(shape) * 50
    if bc == "periodic":
        f -= f.mean()
    u = rng.standard_normal(shape)
    return h, f, u


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("shape", SHAPES)
def test_vcycle_with_direct_coarsest_matches_oracle(shape, bc):
    R = _lib()
    h, f, u = _case(shape, bc, sum(shape))
    nz, ny, nx = shape
    g = oop.Grid(nx, ny, nz, *h, bc)
    want = omg.vcycle(u, f, oop.build_hierarchy(g), omg.Options(), None)
    for dt, tol in ((torch.float64, 1e-11), (torch.float32, 1e-5)):
        phi = torch.from_numpy(u).to("cuda", dt)
        R.vcycle(torch.from_numpy(f).to("cuda", dt), phi, h, bc)
        assert relmax(phi.double().cpu().numpy(), want) < tol


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("shape", [(20, 28), (96, 40), (600, 40)])
def test_2d_vcycle_with_direct_coarsest_matches_oracle(shape, bc):
    """Coarsest levels of 10 x 14, 12 x 10 (6 x 5 is odd) and 150 x 10."""
    R = _lib()
    ny, nx = shape
    h, f, u = _case((1, ny, nx), bc, ny + nx)
    g = oop.grid2d(nx, ny, h[0], h[1], bc)
    want = omg.vcycle(u, f, oop.build_hierarchy(g), omg.Options(), None)
    phi = torch.from_numpy(u[0]).cuda()
    R.vcycle(torch.from_numpy(f[0]).cuda(), phi, h[:2], bc)
    assert relmax(phi.cpu().numpy(), want[0]) < 1e-11


@pytest.mark.parametrize("n", [16, 44])
def test_a_tolerance_of_the_callers_own_keeps_the_iteration(n):
    """A loose coarse tolerance, or a cap below what the default needs, runs the
    accelerated RKL steps: the result is the oracle's with the same options."""
    R = _lib()
    h, f, u = _case((n, n, n), "periodic", n)
    lv = oop.build_hierarchy(oop.Grid(n, n, n, *h, "periodic"))
    for kw in ({"coarse_tol": 1e-2}, {"coarse_max_steps": 2}):
        want = omg.vcycle(u, f, lv, omg.Options(**kw), None)
        full = omg.vcycle(u, f, lv, omg.Options(), None)
        phi = torch.from_numpy(u).cuda()
        R.vcycle(torch.from_numpy(f).cuda(), phi, h, "periodic", opts=R.Options(**kw))
        assert relmax(want, full) > 1e-8
        assert relmax(phi.cpu().numpy(), want) < 1e-11


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_batched_classes_without_a_small_coarsest_level(prec):
    """Classes whose coarsest level is 10^3 (80^3: the tail is that level alone)
    and 22 x 30 x 50 run batched: every member against its single solve and
    the exact discrete solution."""
    R = _lib()
    rng = np.random.default_rng(3)
    rhos, hs = [], []
    for shape, nb in (((80, 80, 80), 3), ((44, 60, 100), 2)):
        for _ in range(nb):
            r = rng.standard_normal(shape)
            rhos.append(r - r.mean())
            hs.append(tuple(1.0 / n for n in shape[::-1]))
    o = R.Options(tol=1e-10, prec=prec)
    phis, stats = R.solve_batched([torch.from_numpy(r).cuda() for r in rhos], hs, "periodic", opts=o)
    for r, h, phi, st in zip(rhos, hs, phis, stats):
        ref, sr = R.solve(torch.from_numpy(r).cuda(), h, "periodic", opts=o)
        assert st.status == 0 and st.cycles == sr.cycles
        assert relmax(phi.cpu().numpy(), ref.cpu().numpy()) < 1e-13
        assert relmax(phi.cpu().numpy(), exact.exact_solution(4 * math.pi * r, h, "periodic")) < 1e-9


def test_non_finite_sources_end_as_before():
    R = _lib()
    rho = torch.zeros((32, 32, 32), dtype=torch.float64, device="cuda")
    rho[3, 4, 5] = float("inf")
    _, st = R.solve(rho, (1.0, 1.0, 1.0), "dirichlet", raise_on_error=False)
    assert st.status == R.RKL_ENONFINITE
