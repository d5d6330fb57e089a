"""Readout calls take no workspace that grows with the readout, and none at all inside a
graph: captured as a context's first calls, replayed after other calls have replaced the
context's workspaces."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import workloads as wl  # noqa: E402
from paper_2107_09879_amd import tmhip  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def rel(a, b):
    return float(torch.linalg.vector_norm(a - b)) / float(torch.linalg.vector_norm(b))


def cvec(rng, *shape):
    return torch.tensor(rng.normal(size=shape) + 1j * rng.normal(size=shape), device=DEV)


def directions(rng, n):
    d = rng.normal(size=(n, 3))
    return torch.tensor(d / np.linalg.norm(d, axis=1)[:, None], device=DEV)


@pytest.mark.parametrize("lmax", [1, 3, 6])
def test_far_field_of_many_directions(lmax):
    """1e5 directions and four right-hand sides: partial sums would take up to 614 MB.
    The first, middle and last directions against calls of their own (split sums)."""
    print(f"[case] lmax {lmax}", flush=True)
    rng = np.random.default_rng(lmax)
    ctx = tmhip.Context(0)
    ctx.set_geometry(wl.lattice_positions(31, 9), wl.K, lmax)
    s, d = cvec(rng, 4, ctx.n, ctx.L), directions(rng, 100000)
    pick = [0, 50001, 99999]
    ref = ctx.far_field(s, d[pick].contiguous())
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0] + torch.cuda.memory_reserved()
    F = ctx.far_field(s, d)
    torch.cuda.synchronize()
    held = before - torch.cuda.mem_get_info()[0] - torch.cuda.memory_reserved()
    assert held < 32 << 20, held
    assert rel(F[:, pick], ref) < 1e-12
    ctx.close()


def test_readouts_in_a_graph():
    rng = np.random.default_rng(0)
    st = torch.cuda.Stream(device=DEV)
    with torch.cuda.stream(st):
        ctx = tmhip.Context(0)
        ctx.set_geometry(wl.lattice_positions(23, 19), wl.K, 3)
        s, w = cvec(rng, 2, ctx.n, ctx.L), cvec(rng, 2, 33, 3)
        pts = torch.tensor(rng.uniform(2.0, 5.0, (33, 3)), device=DEV)
        d = directions(rng, 5)
        big = torch.tensor(rng.uniform(2.0, 5.0, (60000, 3)), device=DEV)
        st.synchronize()

        def readouts():
            return (ctx.far_field(s, d), ctx.near_field(s, pts), ctx.near_field(s, pts, "mixed"),
                    ctx.near_field_adjoint(pts, w))

        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            out = readouts()
        for rep in range(4):
            s.copy_(cvec(rng, 2, ctx.n, ctx.L))
            w.copy_(cvec(rng, 2, 33, 3))
            ctx.near_field(s, big[:15000 * (rep + 1)].contiguous())  # replaces the context's workspace
            graph.replay()
            ref = readouts()
            st.synchronize()
            # the sums' order differs: FP64 to 1e-12, the FP32 basis to 2e-5
            for a, b, tol in zip(out, ref, (1e-12, 1e-12, 2e-5, 1e-12)):
                assert rel(a, b) < tol
        ctx.close()
