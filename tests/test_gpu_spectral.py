"""The transformed block matvec (the default on lattices it fits) against the
direct block matvec, at the sizes where its index maps can go wrong: single rows,
columns and sites, every padded length up to two stages' radices, odd and even
lengths, the largest lattice it takes and the first it does not, one and several
right-hand sides, every lmax and operator.

Tolerances: FP64 1e-12 and complex64 2e-5 as for every matvec kernel (the direct
FP64 product is good to about 4e-15; its complex64 sums to about 2e-6).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import workloads as wl  # noqa: E402
from paper_2107_09879_amd import tmhip  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
TOL = {"fp64": 1e-12, "mixed": 2e-5}
SIZES = [(1, 1, 1, 2), (2, 1, 3, 1), (1, 7, 2, 3), (5, 5, 6, 1), (13, 9, 5, 2), (26, 31, 4, 1)]
SIZES += [(k, 3 + k % 5, 1 + k % 3, 1) for k in (3, 4, 8, 10, 12, 14, 16, 18, 20, 23, 25, 30, 36, 38, 40, 45, 48, 50,
                                                60, 64, 75, 80, 100, 113, 120, 125, 128)]
SIZES += [(3, 160, 3, 1), (250, 4, 2, 1), (320, 2, 1, 1), (2, 320, 3, 1), (321, 2, 1, 1), (2, 321, 1, 1),
          (2, 101, 6, 1), (2, 103, 6, 1), (3, 150, 4, 1)]


@pytest.mark.parametrize("nx,ny,lmax,rhs", SIZES)
def test_transformed_product_matches_blocks(nx, ny, lmax, rhs):
    print(f"[case] {nx}x{ny} lmax {lmax} rhs {rhs}", flush=True)
    ctx, ref = tmhip.Context(0), tmhip.Context(0)
    r = torch.tensor(wl.uniform_radii(nx * ny, 0.15, 0.25, nx + ny), dtype=torch.float64, device=DEV)
    for q in (ctx, ref):
        q.set_geometry(wl.lattice_positions(nx, ny), wl.K, lmax)
        q.set_spheres(r, wl.N_REL)
    rng = np.random.default_rng(nx * 1000 + ny)
    x = torch.tensor(rng.normal(size=(rhs, nx * ny, ctx.L)) + 1j * rng.normal(size=(rhs, nx * ny, ctx.L)), device=DEV)
    for prec in ("fp64", "mixed"):
        ref.set_matvec_config(prec, 8, 0)
        for op in ("forward", "coupling", "adjoint", "coupling_t"):
            y = ctx.apply_operator(x, op, prec)
            want = ref.apply_operator(x, op, "fp64")
            torch.cuda.synchronize()
            err = float(torch.linalg.vector_norm(y - want))
            scale = float(torch.linalg.vector_norm(want))
            assert err <= TOL[prec] * scale, (prec, op, err, scale)
    ctx.close()
    ref.close()


def test_new_geometry_replaces_the_transform():
    """The same context on a second lattice, and T-matrices set after its first product."""
    ctx, ref = tmhip.Context(0), tmhip.Context(0)
    for nx, ny, lmax in ((12, 17, 3), (33, 6, 2), (12, 17, 4)):
        x = torch.randn(1, nx * ny, 2 * lmax * (lmax + 2), 2, dtype=torch.float64, device=DEV)
        x = torch.view_as_complex(x)
        r = torch.full((nx * ny,), 0.2, dtype=torch.float64, device=DEV)
        for q in (ctx, ref):
            q.set_geometry(wl.lattice_positions(nx, ny), wl.K, lmax)
            q.set_matvec_config("mixed", 8, 0)
        a = ctx.apply_operator(x, "coupling", "fp64")
        ref.set_matvec_config("fp64", 8, 0)
        b = ref.apply_operator(x, "coupling", "fp64")
        assert float(torch.linalg.vector_norm(a - b)) <= 1e-12 * float(torch.linalg.vector_norm(b))
        for q in (ctx, ref):
            q.set_spheres(r, wl.N_REL)
        a, b = (q.apply_operator(x, "adjoint", "fp64") for q in (ctx, ref))
        assert float(torch.linalg.vector_norm(a - b)) <= 1e-12 * float(torch.linalg.vector_norm(b))
    ctx.close()
    ref.close()


@pytest.mark.parametrize("nx,ny,lmax,rhs", [(2, 1, 1, 1), (1, 6, 3, 2), (9, 14, 2, 1), (31, 18, 3, 2), (12, 11, 4, 1), (7, 8, 6, 3)])
def test_position_gradient_by_transform_and_by_tables(nx, ny, lmax, rhs):
    """The derivative products by transform against those by derivative tables (which
    the oracle's gradient checks), FP64 in both."""
    ctx, ref = tmhip.Context(0), tmhip.Context(0)
    r = torch.tensor(wl.uniform_radii(nx * ny, 0.15, 0.25, 5), dtype=torch.float64, device=DEV)
    for q in (ctx, ref):
        q.set_geometry(wl.lattice_positions(nx, ny), wl.K, lmax)
        q.set_spheres(r, wl.N_REL)
    ref.set_matvec_config("fp64", 9, 0)
    rng = np.random.default_rng(nx + ny)

    def vec():
        return torch.tensor(rng.normal(size=(rhs, nx * ny, ctx.L)) + 1j * rng.normal(size=(rhs, nx * ny, ctx.L)), device=DEV)

    mu, s, a0 = vec(), vec(), vec()
    kh = np.tile([[0.6, 0.0, 0.8]], (rhs, 1))
    w = rng.normal(size=(rhs, 3)) + 1j * rng.normal(size=(rhs, 3))
    xd = np.array([0.3, 0.4, 3.0])
    for q in range(2):  # the second call finds the symbols built
        a, b = (c.grad_position(mu, s, a0, kh, xd, w) for c in (ctx, ref))
        assert float(torch.linalg.vector_norm(a - b)) <= 1e-12 * float(torch.linalg.vector_norm(b))
    ctx.close()
    ref.close()
