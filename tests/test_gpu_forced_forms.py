"""A tile entry set by hand reaches the V-cycle's strokes: with a strip variant
forced onto a level, its prolongation runs in the strips' fused form (or apart from
them where the variant has none), not in the one-launch strokes that small levels
take otherwise; and what it computes is the same to the last bit, since both spell
out the same operations.  The kernels that ran are read from a device trace."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPE, H = (40, 24, 136), (0.11, 0.07, 0.13)  # levels (40, 24, 136), (20, 12, 68), (10, 6, 34)
# variant: (float64, float32) fused prolongation, s = 2: rows per wavefront, wavefronts
FORMS = {"strip4x4": ((4, 4), (4, 4)), "stripyx4x8": ((4, 8), (4, 8)), "stripyx2x8": ((2, 8), (2, 8)),
         "stripyx8x4": ((2, 8), (8, 4))}


@pytest.fixture(autouse=True)
def _restore_table():
    import paper_2306_05332_amd as R
    R.load_library()
    yield
    R.tune_clear()
    R.install_default_tuning()


def _trace(fn):
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        fn()
        torch.cuda.synchronize()
    return [e.name for e in p.events() if "rkl::" in e.name]


def _cycle(R, dtype, shape=SHAPE, h=H, bc="dirichlet"):
    g = torch.Generator(device="cuda")
    g.manual_seed(17)
    f = torch.randn(shape, generator=g, dtype=torch.float64, device="cuda").to(dtype)
    phi = torch.zeros_like(f)
    names = _trace(lambda: R.vcycle(f, phi, h, bc, opts=R.Options(n_post=1)))
    return phi, names


@pytest.mark.parametrize("prec,dtype", [("fp64", torch.float64), ("mixed", torch.float32)])
@pytest.mark.parametrize("variant", sorted(FORMS))
def test_forced_variant_runs_the_fused_prolongation(variant, prec, dtype):
    import paper_2306_05332_amd as R
    entries = [{"nx": nx, "ny": ny, "nz": nz, "bc": "dirichlet", "prec": prec, "s": 2, "variant": variant,
                "target": 512} for nz, ny, nx in R.level_shapes(SHAPE, bc="dirichlet", h=H)[:2]]
    R.tune_clear()
    free, names = _cycle(R, dtype)
    assert any("k_brick_up" in n for n in names) and not any("k_tau_strip_pro" in n for n in names), names
    R.tune_set(entries)
    got, names = _cycle(R, dtype)
    rows, waves = FORMS[variant][0 if prec == "fp64" else 1]
    name = "double" if prec == "fp64" else "float"
    pro = [n for n in names if f"k_tau_strip_pro<{name}, 2, {rows}, {waves}," in n]
    assert len(pro) == 2 and not any("k_brick" in n for n in names), names
    assert torch.equal(got, free)
    # with a time the entry names a shape only: the strokes stay in one launch
    R.tune_set([dict(e, us=10.0) for e in entries])
    _, names = _cycle(R, dtype)
    assert any("k_brick_up" in n for n in names), names


@pytest.mark.parametrize("prec,dtype", [("fp64", torch.float64), ("mixed", torch.float32)])
def test_forced_two_dimensional_variant_keeps_the_separate_passes(prec, dtype):
    import paper_2306_05332_amd as R
    shape, h = (64, 104), (0.11, 0.07)
    R.tune_clear()
    free, names = _cycle(R, dtype, shape, h)
    assert any("k_win2_up" in n for n in names), names
    R.tune_set([{"nx": nx, "ny": ny, "nz": 1, "bc": "dirichlet", "prec": prec, "s": s, "variant": "strip2d4",
                 "target": 512} for _, ny, nx in R.level_shapes(shape, bc="dirichlet", h=h) for s in (2, 4)])
    got, names = _cycle(R, dtype, shape, h)
    assert any("k_prolong_2d" in n for n in names) and not any("k_win2" in n for n in names), names
    # the passes round once more in between than a window does
    eps = 1e-13 if prec == "fp64" else 1e-5
    assert float((got - free).abs().max()) <= eps * float(free.abs().max())


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("shape", [(100, 100, 100), (72, 130, 160), (300, 300, 300)])
def test_the_query_names_the_kernel_that_runs(shape, prec, bc):
    """Levels without an entry: the tau-step that kernel_info names is the one a
    sweep launches, also after the recorded choice was read and installed again."""
    import paper_2306_05332_amd as R
    R.tune_clear()
    f = torch.ones(shape, dtype=torch.float64 if prec == "fp64" else torch.float32, device="cuda")
    phi = torch.zeros_like(f)

    def sweep():
        return [n for n in _trace(lambda: R.smooth(f, phi, 1.0, bc, s=2, n_steps=2)) if "k_tau" in n]

    want = R.kernel_info(shape, 2, bc, prec)["kernel"].rstrip(">") + ","
    names = sweep()
    assert len(names) == 2 and all(want in n for n in names), (want, names)
    R.tune_set([R.tune_get(shape, 2, bc, prec)])
    assert sweep() == names
