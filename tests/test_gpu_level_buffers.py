"""Level-0 buffers of the level entry points: odd numbers of passes end in the
caller's array without a copy, and a call whose phi is its own right-hand side
takes f as it was on entry; against the same call with the passes made one by
one, or on separate arrays (the same kernels, so the same bits)."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
H = (0.11, 0.07, 0.13)


def _fields(shape, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(shape))
    f, u = (torch.randn(shape, generator=g, device="cuda", dtype=torch.float64).to(dtype) for _ in range(2))
    return f, u


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("shape", [(20, 11, 130), (9, 6, 5), (40, 24, 64)])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
def test_smooth_steps_together_are_the_steps_one_by_one(shape, n, dtype):
    import paper_2306_05332_amd as R
    f, u = _fields(shape, dtype)
    a, b = u.clone(), u.clone()
    R.smooth(f, a, H, "periodic", s=2, n_steps=n)
    for _ in range(n):
        R.smooth(f, b, H, "periodic", s=2, n_steps=1)
    assert torch.equal(a, b)


@pytest.mark.parametrize("smoother", ["rkl", "gsrb"])
@pytest.mark.parametrize("pre,post", [(1, 1), (2, 1), (4, 1), (2, 2), (3, 1)])
def test_vcycle_on_its_own_right_hand_side(pre, post, smoother):
    import paper_2306_05332_amd as R
    f, _ = _fields((40, 24, 64), torch.float64)
    o = R.Options(n_pre=pre, n_post=post, smoother=smoother)
    a, b = f.clone(), f.clone()
    R.vcycle(f, a, H, "dirichlet", opts=o)
    R.vcycle(b, b, H, "dirichlet", opts=o)
    assert torch.equal(a, b)
    a, b = f.clone(), f.clone()
    R.gsrb_smooth(f, a, H, "dirichlet", n_iter=3)
    R.gsrb_smooth(b, b, H, "dirichlet", n_iter=3)
    assert torch.equal(a, b)
