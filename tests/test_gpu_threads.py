"""Several threads, each with its own context and stream: products whose kernels need
different amounts of LDS, solves, batches, readouts; every result as alone.  (Batches without
graphs: while one thread captures, the runtime refuses other threads' synchronous copies.)"""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import workloads as wl  # noqa: E402
from paper_2107_09879_amd import tmhip  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
# columns of 154, 144, 92 and 41 KB at lmax 3 and FP64, one of each beside another
LATTICES = [(2, 300, 3), (3, 280, 3), (4, 180, 3), (12, 80, 3)]


def outputs(k, reps):
    nx, ny, lmax = LATTICES[k]
    st = torch.cuda.Stream(device=DEV)
    out = []
    with torch.cuda.stream(st), tmhip.Context(0) as ctx:
        for rep in range(reps):
            ctx.set_geometry(wl.lattice_positions(nx, ny), wl.K, lmax)
            ctx.set_spheres(torch.full((nx * ny,), 0.16, dtype=torch.float64, device=DEV), wl.N_REL)
            rng = np.random.default_rng(k)
            x = torch.tensor(rng.normal(size=(2, ctx.n, ctx.L)) + 1j * rng.normal(size=(2, ctx.n, ctx.L)), device=DEV)
            got = [ctx.apply_operator(x, op, prec) for op in ("forward", "adjoint") for prec in ("fp64", "mixed")]
            got.append(ctx.solve(x, tol=1e-6, restart=30)[0])
            kh, po = wl.incidences(["x"])
            got += ctx.solve_batched([(0, 0, 2, 7), (1, 3, 1, 9)], kh, po, tol=1e-6, use_graph=False)[0]
            got.append(ctx.far_field(x, torch.tensor([[0.0, 0.6, 0.8]], dtype=torch.float64, device=DEV)))
            st.synchronize()
            out.append([g.clone() for g in got])
            st.synchronize()
    return out


def test_threads_with_contexts_of_their_own():
    alone = [outputs(k, 1)[0] for k in range(len(LATTICES))]
    got, errors = [None] * len(LATTICES), []

    def work(k):
        try:
            got[k] = outputs(k, 12)
        except Exception as e:  # reported by the test's own thread
            errors.append((k, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(LATTICES))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k, ref in enumerate(alone):
        for rep in got[k]:
            for a, b in zip(rep, ref):
                assert torch.equal(torch.view_as_real(a), torch.view_as_real(b)), k
