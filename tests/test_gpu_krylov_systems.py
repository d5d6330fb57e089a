"""GMRES over several systems that leave a cycle at different steps: a system that stops
while another launch still works on its vectors must not disturb the others, nor the
bits of the results from one run to the next (every sum has a fixed order)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import workloads as wl  # noqa: E402
from paper_2107_09879_amd import tmhip  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def setup(nx, ny, lmax, seed=7):
    ctx = tmhip.Context(0)
    ctx.set_geometry(wl.lattice_positions(nx, ny), wl.K, lmax)
    ctx.set_spheres(torch.tensor(wl.uniform_radii(nx * ny, 0.15, 0.2, seed), device=DEV), wl.N_REL)
    return ctx


def rhs(ctx, R, seed):
    rng = np.random.default_rng(seed)
    return torch.tensor(rng.normal(size=(R, ctx.n, ctx.L)) + 1j * rng.normal(size=(R, ctx.n, ctx.L)), device=DEV)


@pytest.mark.parametrize("nx,ny,precision", [(17, 13, "fp64"), (40, 37, "mixed")])
def test_systems_that_stop_at_different_steps(nx, ny, precision):
    """From start vectors of different accuracy, so that the systems stop steps apart."""
    print(f"[case] {nx}x{ny} {precision}", flush=True)
    ctx = setup(nx, ny, 2)
    a0 = rhs(ctx, 5, 1)
    s, _ = ctx.solve(a0, tol=1e-12, precision=precision)
    x0 = s + rhs(ctx, 5, 2) * torch.tensor([1e-10, 1e-8, 1e-5, 1e-2, 1.0], device=DEV)[:, None, None]
    first = None
    for rep in range(4):
        got, info = ctx.solve(a0, x0=x0.clone(), tol=1e-11, restart=60, precision=precision)
        assert all(i["status"] == 0 and i["rel_residual"] <= 1e-11 for i in info)
        assert len({i["iters"] for i in info}) >= 4
        if first is None:
            first = got, info
        assert torch.equal(torch.view_as_real(got), torch.view_as_real(first[0])) and info == first[1]
    ctx.close()


def test_bits_do_not_depend_on_free_memory():
    """Twelve bases of 1001 vectors (61 GB), with the card empty, with two fifths of it
    taken, and with too little left for all twelve (then solved in two halves, whose sums
    are cut otherwise: equal to rounding)."""
    ctx = setup(100, 100, 3)
    a0 = rhs(ctx, 12, 3)

    def solve():
        s, info = ctx.solve(a0, tol=1e-30, restart=1000, max_iter=25)
        assert all(i["iters"] == 25 and i["status"] == tmhip.TM_NOT_CONVERGED for i in info)
        return s

    ref = solve()
    hold = torch.empty(torch.cuda.mem_get_info()[1] * 2 // 5, dtype=torch.uint8, device=DEV)
    assert torch.equal(torch.view_as_real(solve()), torch.view_as_real(ref))
    del hold
    torch.cuda.empty_cache()
    hold = torch.empty(torch.cuda.mem_get_info()[0] - (44 << 30), dtype=torch.uint8, device=DEV)
    s = solve()
    del hold
    torch.cuda.empty_cache()
    assert float(torch.linalg.vector_norm(s - ref)) < 1e-11 * float(torch.linalg.vector_norm(ref))
    ctx.close()


@pytest.mark.parametrize("product", ["staged", "direct", "pairwise", "dense"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_solved_right_hand_sides_cost_no_product(product, precision):
    """One right-hand side of four is not zero: the products of a solve take what its own
    would, and not four times that (twice, at most), and the solution is its own."""
    n, lmax = 48, 3
    print(f"[case] {product} {precision}", flush=True)
    pos = wl.lattice_positions(n, n)
    if product == "pairwise":
        pos[:, :2] += np.random.default_rng(1).uniform(-0.03, 0.03, (n * n, 2))
    ctx = tmhip.Context(0)
    ctx.set_geometry(pos, wl.K, lmax)
    ctx.set_spheres(torch.full((n * n,), 0.17, dtype=torch.float64, device=DEV), wl.N_REL)
    if product == "dense":
        ctx.set_tmatrix_dense(torch.diag_embed(ctx.get_tmatrix_diag()[0]).contiguous())
    if product != "pairwise":
        for prec in ("fp64", "mixed"):
            ctx.set_matvec_config(prec, 3 if product == "direct" else 8, 0)
    one = rhs(ctx, 1, 5)
    four = torch.zeros(4, ctx.n, ctx.L, dtype=torch.complex128, device=DEV)
    four[2] = one[0]

    def timed(a0):
        ms = []
        for _ in range(3):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            s, info = ctx.solve(a0, tol=1e-10, precision=precision)
            e[1].record()
            e[1].synchronize()
            ms.append(e[0].elapsed_time(e[1]))
        return s, info, min(ms)

    s1, i1, t1 = timed(one)
    s4, i4, t4 = timed(four)
    print(f"[info] {t1:.2f} ms alone, {t4:.2f} ms of four", flush=True)
    assert i1[0]["status"] == 0 and [i["status"] for i in i4] == [0] * 4
    assert float(torch.linalg.vector_norm(s4[2] - s1[0])) < 1e-7 * float(torch.linalg.vector_norm(s1[0]))
    assert float(s4[[0, 1, 3]].abs().max()) == 0.0
    assert t4 < 2.0 * t1
    ctx.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_products_are_counted(precision):
    """One product per step, one more in a cycle that ends early (its last step's second
    Gram-Schmidt pass), one FP64 residual per cycle and one for a start vector; the
    profiler records as many."""
    print(f"[case] {precision}", flush=True)
    ctx = setup(14, 9, 2)
    a0 = rhs(ctx, 1, 6)
    which = {"fp64": 0, "mixed": 1}[precision]

    def check(early, x0=None, **opts):
        ctx.profile_reset()
        ctx.profile_enable(True)
        s, info = ctx.solve(a0, x0=x0, precision=precision, **opts)
        ctx.profile_enable(False)
        i = info[0]
        arnoldi, residuals = i["iters"] + early(i), i["cycles"] + (x0 is not None)
        want = (arnoldi + residuals, 0) if precision == "fp64" else (residuals, arnoldi)
        assert (i["matvecs_fp64"], i["matvecs_lowp"]) == want, i
        assert ctx.profile_query(which)[1] == want[which]
        assert ctx.profile_query(1 - which)[1] == want[1 - which]
        return s

    # cycles that converge (in mixed precision, to the inner tolerance)
    s = check(lambda i: i["cycles"], tol=1e-12, restart=200)
    check(lambda i: i["cycles"], x0=s + 1e-3 * rhs(ctx, 1, 7), tol=1e-12, restart=200)
    # cycles that run to their end: 5, 5 and 2 steps
    check(lambda i: 0, tol=1e-30, restart=5, max_iter=12)
    ctx.close()
