"""The tile query that says what runs (host only): entries as installed, fitted
shapes on levels without one, and round trips of both queries through the table."""
import pytest

SHAPES = [((300, 300, 300), 1.0), ((100, 100, 100), 1.0), ((160, 96, 224), 1.0), ((130, 4000), (1.0, 1.0)),
          ((8, 8, 8), 1.0)]


@pytest.fixture()
def L():
    from paper_2306_05332_amd import _lib
    _lib.tune_clear()
    yield _lib
    _lib.tune_clear()
    _lib.install_default_tuning()


def _keys(shape):
    nz, ny, nx = (1,) * (3 - len(shape)) + shape
    return {"nx": nx, "ny": ny, "nz": nz}


@pytest.mark.parametrize("query", ["tune_get", "tune_launched"])
@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("s", [1, 2, 3])
def test_installing_a_query_s_answer_changes_nothing(L, query, bc, prec, s):
    for shape, h in SHAPES:
        before = L.tune_launched(shape, s, bc, prec, h)
        L.tune_set([getattr(L, query)(shape, s, bc, prec, h)])
        assert L.tune_launched(shape, s, bc, prec, h) == before, shape


@pytest.mark.parametrize("us", [0.0, 17.5])
def test_entries_are_reported_as_installed(L, us):
    shape = (300, 300, 300)
    fitted = L.tune_launched(shape, 2, "periodic", "fp64")
    assert fitted["variant"] == "stripyx2x8" and fitted["us"] == -1.0
    base = L.tune_get(shape, 2, "periodic", "fp64")
    assert base["variant"] == "strip8x4" and base["us"] == -1.0
    e = dict(_keys(shape), bc="periodic", prec="fp64", s=2, variant="strip4x4", target=700, us=us)
    L.tune_set([e])
    assert L.tune_get(shape, 2, "periodic", "fp64") == e == L.tune_launched(shape, 2, "periodic", "fp64")
    L.tune_set([base])
    assert L.tune_launched(shape, 2, "periodic", "fp64") == fitted


def test_launched_strips_state_their_workgroups(L):
    """A fitted target is the workgroup count it comes to: z chunks times the
    column tiles, which the tuner times too (stacked two-row strips: 60 columns by
    16 rows)."""
    e = L.tune_launched((300, 300, 300), 2, "periodic", "fp64")
    per = 5 * 19
    assert e["target"] % per == 0
    chunks = e["target"] // per
    assert any(chunks == -(-300 // zc) for zc in range(1, 65))


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("shape", [(300, 300, 300), (160, 160, 160), (40, 40, 40)])
def test_float64_steps_of_one_stage_keep_the_base_choice(L, shape, bc):
    """The fitted shapes were timed on two stages; with one they lose as often as
    they win."""
    base, got = L.tune_get(shape, 1, bc, "fp64"), L.tune_launched(shape, 1, bc, "fp64")
    assert got["variant"] == base["variant"]
