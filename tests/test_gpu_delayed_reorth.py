"""GMRES with its second Gram-Schmidt pass one step late, where its kernels split:
one cycle of more steps than rows that three waves share (256; 128 from step 512 on) and than rotations
loaded ahead (128), long after convergence (the basis has to stay orthogonal), and
vectors on both sides of the switch between elements shared by four waves and one
per thread (131072 in all).

Condition numbers are below 1e3 on these lattices (radii 0.15 to 0.2): a residual of
1e-12 gives 1e-9 in the solution.  A long cycle's residual is the least one of its
Krylov space, taken here from modified Gram-Schmidt, twice, in numpy.
"""
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


def setup(nx, ny, lmax):
    pos = wl.lattice_positions(nx, ny)
    radii = wl.uniform_radii(nx * ny, 0.15, 0.2, 7)
    ctx = tmhip.Context(0)
    ctx.set_geometry(pos, wl.K, lmax)
    ctx.set_spheres(torch.tensor(radii, device=DEV), wl.N_REL)
    return ctx, pos, radii


def least_residual(B, b, steps):
    """of B x = b over the Krylov space of that many steps, relative to |b|"""
    V = np.zeros((steps + 1, len(b)), complex)
    H = np.zeros((steps + 1, steps), complex)
    beta = np.linalg.norm(b)
    V[0] = b / beta
    for j in range(steps):
        w = B @ V[j]
        for _ in range(2):
            for q in range(j + 1):
                h = np.vdot(V[q], w)
                H[q, j] += h
                w -= h * V[q]
        H[j + 1, j] = np.linalg.norm(w)
        V[j + 1] = w / H[j + 1, j]
    rhs = np.zeros(steps + 1, complex)
    rhs[0] = beta
    y = np.linalg.lstsq(H, rhs, rcond=None)[0]
    return np.linalg.norm(b - B @ (y @ V[:steps])) / beta


@pytest.mark.parametrize("steps", [64, 65, 129, 130, 255, 256, 257, 300, 512, 513])
def test_long_cycles(steps):
    print(f"[case] {steps} steps", flush=True)
    ctx, pos, radii = setup(12, 11, 2)
    rng = np.random.default_rng(steps)
    a = rng.normal(size=(2, ctx.n, ctx.L)) + 1j * rng.normal(size=(2, ctx.n, ctx.L))
    s, info = ctx.solve(torch.tensor(a, device=DEV), tol=1e-300, restart=steps, max_iter=steps)
    assert [(i["iters"], i["cycles"]) for i in info] == [(steps, 1)] * 2
    t, _ = oracle.mie_tmatrix_diag_many(2, wl.K, radii, wl.N_REL)
    B, _, T = oracle.system_dense(pos, wl.K, 2, t)
    for r in range(2):
        b = T @ a[r].ravel()
        assert info[r]["rel_residual"] <= least_residual(B, b, steps) * (1 + 1e-6) + 1e-13
        x = s[r].cpu().numpy().ravel()
        err = np.linalg.norm(x - np.linalg.solve(B, b)) / np.linalg.norm(x)
        assert err < 1e3 * info[r]["rel_residual"] + 1e-12
    ctx.close()


@pytest.mark.parametrize("nx,ny", [(64, 32), (64, 33), (61, 64)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_elements_shared_and_not(nx, ny, precision):
    """Two right-hand sides together (2 * 32 * sites elements each) and one by one."""
    print(f"[case] {nx}x{ny} {precision}", flush=True)
    ctx, _, _ = setup(nx, ny, 2)
    kh, po = wl.incidences(["x", "p10"])
    a0 = ctx.plane_wave_rhs(kh, po)
    s, info = ctx.solve(a0, tol=1e-12, precision=precision)
    assert all(i["status"] == 0 and i["rel_residual"] <= 1e-12 for i in info)
    for r in range(2):
        one, i1 = ctx.solve(a0[r:r + 1].clone(), tol=1e-12, precision=precision)
        assert i1[0]["status"] == 0
        assert float(torch.linalg.vector_norm(one[0] - s[r])) < 1e-9 * float(torch.linalg.vector_norm(s[r]))
    ctx.close()
