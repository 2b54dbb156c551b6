"""The convergence test inside the coarse tail (small grids, whose first stroke is
one launch) against the test in its own launch, which the separate passes
(fuse = 0) keep: the same decisions at the same cycles for convergence, cycle
limits (none, one, an even and an odd number), exactly max_cycles at tol = 0 and
non-finite data, on one and on several grids.  History: both paths run the same
algorithm, so the residual norms differ by rounding, at most 1e-13 of the norm of
f (a few hundred roundings of M u against f), beside 1e-9 of their value.  Mixed: a
float32 correction's rounding, 6e-8 of it, reaches the next residual times the
condition number of M (about 700 on 40 cells), 4e-5 of the last residual and ten
times that of the next: 1e-2 with the roundings of a cycle; 1e-6 of phi."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [dict(tol=1e-10), dict(tol=1e-10, max_cycles=0), dict(tol=1e-10, max_cycles=1), dict(tol=1e-10, max_cycles=4),
         dict(tol=0.0, max_cycles=3)]


def _rho(shape, seed):
    r = np.random.default_rng(seed).standard_normal(shape)
    return torch.from_numpy(r - r.mean()).cuda()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("shape", [(32, 32, 32), (24, 40, 28), (64, 48)])
@pytest.mark.parametrize("opt", CASES)
def test_decisions_match_the_separate_check(opt, shape, prec):
    import paper_2306_05332_amd as R
    h = (0.05, 0.04, 0.06)[: len(shape)]
    rho = _rho(shape, 5)
    got = [R.solve(rho, h, "periodic", opts=R.Options(prec=prec, fuse=f, **opt), raise_on_error=False) for f in (3, 0)]
    (phi, a), (ref, b) = got
    assert (a.status, a.cycles) == (b.status, b.cycles)
    np.testing.assert_allclose(a.history, b.history, rtol=1e-9 if prec == "fp64" else 1e-2, atol=1e-13)
    d = (phi - ref).abs().max()
    assert float(d) <= (1e-11 if prec == "fp64" else 1e-6) * max(float(ref.abs().max()), 1e-300)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_batch_members_stop_on_their_own(prec):
    import paper_2306_05332_amd as R
    rhos = [_rho((32, 32, 32), 7), 0 * _rho((32, 32, 32), 8), _rho((32, 32, 32), 9)]
    h = (0.05, 0.04, 0.06)
    o = R.Options(tol=1e-9, prec=prec)
    phis, stats = R.solve_batched(rhos, [h] * 3, "periodic", opts=o)
    for rho, phi, st in zip(rhos, phis, stats):
        ref, sr = R.solve(rho, h, "periodic", opts=o)
        assert (st.status, st.cycles) == (sr.status, sr.cycles)
        assert float((phi - ref).abs().max()) <= 1e-13 * max(float(ref.abs().max()), 1e-300)


def test_non_finite_data_is_reported():
    import paper_2306_05332_amd as R
    rho = _rho((32, 32, 32), 3)
    rho[3, 4, 5] = float("inf")
    codes = []
    for f in (3, 0):
        _, st = R.solve(rho, (0.05,) * 3, "dirichlet", opts=R.Options(fuse=f), raise_on_error=False)
        codes.append(st.status)
    assert codes[0] == codes[1] != 0
