"""Device memory of batched solves whose coarsest level is larger than the
one-workgroup iteration takes (more than 256 cells): they hold arrays for every
member, where single solves need one member's."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GIB = 1 << 30


def test_batch_without_room_for_its_class_is_solved_member_by_member():
    """24 boxes of 200 x 120 x 88 cells (coarsest level 50 x 30 x 22): their class
    takes over 2 GiB, of which the device has 1.25 left.  The members are solved
    one by one: the single solves, bit for bit."""
    import paper_2306_05332_amd as R
    shape, h, nb = (88, 120, 200), (0.005,) * 3, 24
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    rhos = [torch.randn(shape, generator=g, dtype=torch.float64, device="cuda") for _ in range(nb)]
    o = R.Options(tol=1e-8)
    R.release_all()
    ref = [R.solve(rhos[k], h, "dirichlet", opts=o) for k in (0, nb - 1)]
    outs = [torch.empty(shape, dtype=torch.float64, device="cuda") for _ in range(nb)]
    del outs  # the batch's results come from these cached blocks
    torch.cuda.synchronize()
    held = []
    try:
        while True:
            left = torch.cuda.mem_get_info()[0] - int(1.25 * GIB)
            if left < GIB // 8:
                break
            held.append(torch.empty(min(left, 16 * GIB), dtype=torch.uint8, device="cuda"))
        print("free:", torch.cuda.mem_get_info()[0] / GIB, "GiB", flush=True)
        phis, stats = R.solve_batched(rhos, [h] * nb, "dirichlet", opts=o)
        torch.cuda.synchronize()
    finally:
        del held
        torch.cuda.empty_cache()
    assert all(st.status == 0 for st in stats)
    for k, (phi, st) in zip((0, nb - 1), ref):
        assert torch.equal(phis[k], phi) and stats[k].cycles == st.cycles
        np.testing.assert_array_equal(stats[k].history, st.history)


def test_classes_kept_between_calls_are_bounded():
    """Three batches of about 64 million cells (boxes of 40^3, coarsest level 10^3)
    that differ in their member count, each a class of its own: 43 bytes a cell, so
    one class is 2.6 GiB, and what the library holds stays below two of them."""
    import paper_2306_05332_amd as R
    n, h = 40, (1.0 / 40,) * 3
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    rho = torch.randn((n, n, n), generator=g, dtype=torch.float64, device="cuda")
    o = R.Options(tol=1e-3)
    ref, st = R.solve(rho, h, "dirichlet", opts=o)
    R.release_all()
    R.solve_batched([rho] * 3, [h] * 3, "dirichlet", opts=o)
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    for nb in (1000, 1001, 1002):
        phis, stats = R.solve_batched([rho] * nb, [h] * nb, "dirichlet", opts=o)
        for k in (0, nb - 1):
            assert stats[k].cycles == st.cycles
            assert float((phis[k] - ref).abs().max()) <= 1e-13 * float(ref.abs().max())
        del phis
        torch.cuda.empty_cache()
        held = free - torch.cuda.mem_get_info()[0]
        print(f"{nb} members: {held / GIB:.2f} GiB held", flush=True)
        assert held < 2 * 43 * 1000 * n ** 3
    R.release_all()
