"""The transformed product on the longest columns it takes, where twiddle factors,
positions and constants no longer fit in LDS beside the column (FP64: 257 sites and more
at lmax 3, 271 at lmax 2, 289 at lmax 1), at sizes that fit in complex64 alone, in the
position gradient and in batches of every lmax, against the block kernels; and 300x300,
both axes at their longest, against rows of the oracle.

Tolerances as for every matvec kernel: FP64 1e-12, complex64 2e-5."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import workloads as wl  # noqa: E402
from paper_2107_09879_amd import tmhip  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
TOL = {"fp64": 1e-12, "mixed": 2e-5}


def contexts(nx, ny, lmax):
    """One with the default products, one with the block kernels."""
    r = torch.tensor(wl.uniform_radii(nx * ny, 0.15, 0.25, nx + ny), dtype=torch.float64, device=DEV)
    out = []
    for blocks in (False, True):
        ctx = tmhip.Context(0)
        ctx.set_geometry(wl.lattice_positions(nx, ny), wl.K, lmax)
        ctx.set_spheres(r, wl.N_REL)
        if blocks:
            ctx.set_matvec_config("fp64", 9, 0)
            ctx.set_matvec_config("mixed", 8, 0)
        out.append(ctx)
    return out


def vec(rng, *shape):
    return torch.tensor(rng.normal(size=shape) + 1j * rng.normal(size=shape), device=DEV)


def rel(a, b):
    return float(torch.linalg.vector_norm(a - b)) / float(torch.linalg.vector_norm(b))


@pytest.mark.parametrize("nx,ny,lmax,rhs", [(2, 300, 3, 2), (3, 257, 3, 1), (3, 256, 3, 1), (2, 300, 2, 1), (2, 271, 2, 1),
                                            (2, 300, 1, 1), (3, 289, 1, 2), (300, 3, 3, 1), (2, 320, 3, 1), (2, 300, 4, 1),
                                            (2, 151, 4, 1), (2, 200, 5, 1), (2, 200, 6, 1), (2, 100, 6, 1), (2, 100, 5, 2)])
def test_longest_columns(nx, ny, lmax, rhs):
    print(f"[case] {nx}x{ny} lmax {lmax} rhs {rhs}", flush=True)
    ctx, ref = contexts(nx, ny, lmax)
    x = vec(np.random.default_rng(ny), rhs, nx * ny, ctx.L)
    for op in ("forward", "coupling", "adjoint", "coupling_t"):
        want = ref.apply_operator(x, op, "fp64")
        for prec in ("fp64", "mixed"):
            assert rel(ctx.apply_operator(x, op, prec), want) < TOL[prec], (op, prec)
    ctx.close()
    ref.close()


@pytest.mark.parametrize("nx,ny,lmax", [(2, 300, 3), (3, 257, 3), (2, 271, 2), (2, 289, 1)])
def test_position_gradient_on_long_columns(nx, ny, lmax):
    print(f"[case] {nx}x{ny} lmax {lmax}", flush=True)
    ctx, ref = contexts(nx, ny, lmax)
    rng = np.random.default_rng(ny)
    mu, s, a0 = (vec(rng, 1, nx * ny, ctx.L) for _ in range(3))
    w = rng.normal(size=(1, 3)) + 1j * rng.normal(size=(1, 3))
    a, b = (c.grad_position(mu, s, a0, np.array([[0.6, 0.0, 0.8]]), np.array([0.3, 0.4, 3.0]), w) for c in (ctx, ref))
    assert rel(a, b) < 1e-12
    ctx.close()
    ref.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("lmax,tall", [(1, 290), (2, 272), (3, 258), (4, 40), (5, 9), (6, 7)])
def test_batches(lmax, tall, precision):
    """Subregions of several heights in one batch share their launches, and so their LDS."""
    print(f"[case] lmax {lmax} {precision}", flush=True)
    ctx, ref = contexts(12, tall + 2, lmax)
    kh, po = wl.incidences(["x", "p10"])
    subs = [(0, 1, 2, tall), (1, 0, 5, 4), (4, 3, 1, 1), (2, 2, 8, 5)]
    out = []
    for c in (ctx, ref):
        s, info = c.solve_batched(subs, kh, po, tol=1e-11, restart=60, max_iter=3000, precision=precision)
        assert all(i["status"] == 0 for q in info for i in q)
        out.append(s)
    # residuals of 1e-11 on systems of condition below 1e3
    for a, b in zip(*out):
        assert rel(a, b) < 2e-8
    ctx.close()
    ref.close()


def test_300x300_rows_of_the_default_product():
    print("[case] 300x300", flush=True)
    n, lmax = 300, 3
    pos = wl.lattice_positions(n, n)
    ctx = tmhip.Context(0)
    ctx.set_geometry(pos, wl.K, lmax)
    rng = np.random.default_rng(301)
    x = rng.normal(size=(2, n * n, ctx.L)) + 1j * rng.normal(size=(2, n * n, ctx.L))
    for op, r, rows in (("coupling", 0, [0, n * n - 1]), ("coupling", 1, [n * 150 + 149]),
                        ("coupling_t", 1, [n - 1, n * 297 + 3])):
        ref = torch.tensor(oracle.rows_A(pos, wl.K, lmax, x[r], rows, transpose=op == "coupling_t"), device=DEV)
        for prec in ("fp64", "mixed"):
            y = ctx.apply_operator(torch.tensor(x, device=DEV), op, prec)[r][rows]
            e = rel(y, ref)
            print(f"[info] {op} {prec} rows {rows}: {e:.2e}", flush=True)
            assert e < TOL[prec]
    ctx.close()
