"""What a context still holds after calls whose workspaces were large, in bytes of device
memory beyond what its results and tables need."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import workloads as wl  # noqa: E402
from paper_2107_09879_amd import tmhip  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
MB = 1 << 20


def free():
    """Device memory that nobody but torch's allocator holds."""
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0] + torch.cuda.memory_reserved()


def spheres(ctx, pos, lmax):
    ctx.set_geometry(pos, wl.K, lmax)
    ctx.set_spheres(torch.full((len(pos),), 0.17, dtype=torch.float64, device=DEV), wl.N_REL)


def test_tables_of_a_large_lattice():
    """7.8 GB of tables and T; the workspace that built them is 82 MB."""
    n = 400
    with tmhip.Context(0) as ctx:
        ctx.set_geometry(wl.lattice_positions(3, 3), wl.K, 1)
        before = free()
        ctx.set_geometry(wl.lattice_positions(n, n), wl.K, 1)
        tables = (2 * n - 1) ** 2 * 2 * 256 * 24 + n * n * 2 * 16 * (16 + 8 + 16)
        assert before - free() < tables + 40 * MB


def test_transforms_are_released_off_the_lattice():
    n = 300
    pos = wl.lattice_positions(n, n)
    with tmhip.Context(0) as ctx:
        spheres(ctx, wl.lattice_positions(3, 3), 3)
        before = free()
        spheres(ctx, pos, 3)
        x = torch.zeros(1, n * n, ctx.L, dtype=torch.complex128, device=DEV)
        ctx.apply_operator(x, "coupling", "fp64")
        off = pos[:40].copy()
        off[3, 1] += 0.01
        spheres(ctx, off, 3)
        # T (three copies) and the operator's two packed vectors may stay
        kept = n * n * 2 * 16 * (16 + 8 + 16 + 2 * 16)
        assert before - free() < kept + 40 * MB


def test_batch_of_many_systems():
    """2400 systems at restart 200: 3 GB of Hessenberg matrices."""
    with tmhip.Context(0) as ctx:
        spheres(ctx, wl.lattice_positions(20, 15), 1)
        before = free()
        kh, po = wl.incidences(["x", "y"] * 4)
        _, info = ctx.solve_batched([(i, j, 1, 1) for i in range(20) for j in range(15)], kh, po, tol=1e-10, restart=200)
        assert all(i["status"] == 0 for q in info for i in q)
        assert before - free() < 2100 * MB


def test_a_solve_that_fails():
    """Two bases of 1001 vectors (10 GB) are given back when a right-hand side is not
    finite as when the solve succeeds."""
    with tmhip.Context(0) as ctx:
        spheres(ctx, wl.lattice_positions(100, 100), 3)
        a0 = torch.zeros(2, ctx.n, ctx.L, dtype=torch.complex128, device=DEV)
        a0[:, 5, 0] = 1.0
        before = free()
        ctx.solve(a0, tol=1e-2, restart=1000)
        assert before - free() < 1000 * MB
        a0[1, 7, 2] = np.nan
        with pytest.raises(tmhip.TmError) as e:
            ctx.solve(a0, tol=1e-2, restart=1000)
        assert e.value.code == -6
        assert before - free() < 1000 * MB
        a0[1, 7, 2] = 0.0
        _, info = ctx.solve(a0, tol=1e-2, restart=50)
        assert [i["status"] for i in info] == [0, 0]
