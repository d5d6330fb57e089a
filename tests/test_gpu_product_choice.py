"""Which product runs (transformed or by block kernels) is what was last chosen for the
lattice's size: a configuration read back selects the same product, and a choice made on
one lattice does not follow the context to another.  The products differ in rounding, so
equal bits mean the same product."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import workloads as wl  # noqa: E402
from paper_2107_09879_amd import tmhip  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
PRECISIONS = ["fp64", "mixed"]


def set_lattice(ctx, nx, ny, lmax):
    ctx.set_geometry(wl.lattice_positions(nx, ny), wl.K, lmax)
    ctx.set_spheres(torch.tensor(wl.uniform_radii(nx * ny, 0.15, 0.2, 3), device=DEV), wl.N_REL)


def vec(ctx, seed=1):
    rng = np.random.default_rng(seed)
    return torch.tensor(rng.normal(size=(1, ctx.n, ctx.L)) + 1j * rng.normal(size=(1, ctx.n, ctx.L)), device=DEV)


def outputs(ctx, precision):
    """What each path that has the choice computes, as bits."""
    x, y = vec(ctx, 1), vec(ctx, 2)
    kh, po = wl.incidences(["x"])
    got = [ctx.apply_operator(x, "coupling", precision), ctx.grad_position(x, y)]
    got += ctx.solve_batched([(0, 0, 9, 8), (1, 2, 5, 5)], kh, po, use_graph=False, tol=1e-6, precision=precision)[0]
    return [torch.view_as_real(g).clone() if g.is_complex() else g.clone() for g in got]


def same(a, b):
    return [torch.equal(p, q) for p, q in zip(a, b)]


@pytest.mark.parametrize("precision", PRECISIONS)
def test_a_configuration_read_back_selects_the_same_product(precision):
    print(f"[case] {precision}", flush=True)
    ctx = tmhip.Context(0)
    set_lattice(ctx, 21, 18, 3)
    transformed = outputs(ctx, precision)
    conf = ctx.get_matvec_config(precision)
    ctx.set_matvec_config(precision, *conf)
    assert ctx.get_matvec_config(precision) == conf and conf[1] < 0
    assert all(same(outputs(ctx, precision), transformed))
    for items in (0, 40):
        ctx.set_matvec_config(precision, 8, items)
        assert ctx.get_matvec_config(precision) == (8, items)
        blocks = outputs(ctx, precision)
        differ = same(blocks, transformed)
        assert not differ[0] and not any(differ[2:]) and (precision == "mixed" or not differ[1])
        ctx.set_matvec_config(precision, *ctx.get_matvec_config(precision))
        assert all(same(outputs(ctx, precision), blocks))
        ctx.set_matvec_config(precision, *conf)
        assert all(same(outputs(ctx, precision), transformed))
    # the work split under the transformed product is kept for the block kernels
    ctx.set_matvec_config(precision, 8, -1 - 40)
    assert ctx.get_matvec_config(precision) == (8, -41)
    assert all(same(outputs(ctx, precision), transformed))
    ms, tuned = ctx.autotune(1, precision)
    first = outputs(ctx, precision)
    ctx.set_matvec_config(precision, *tuned)
    assert ctx.get_matvec_config(precision) == tuned
    assert all(same(outputs(ctx, precision), first))
    ctx.close()


@pytest.mark.parametrize("precision", PRECISIONS)
def test_a_choice_holds_for_its_lattice_size(precision):
    print(f"[case] {precision}", flush=True)
    ctx, fresh = tmhip.Context(0), tmhip.Context(0)
    ctx.set_matvec_config(precision, 8, 0)  # for the first geometry
    set_lattice(ctx, 9, 8, 2)
    set_lattice(fresh, 9, 8, 2)
    blocks, transformed = outputs(ctx, precision), outputs(fresh, precision)
    assert not same(blocks, transformed)[0]
    set_lattice(ctx, 9, 8, 2)  # the same size again
    assert all(same(outputs(ctx, precision), blocks))
    for nx, ny, lmax in ((21, 18, 2), (9, 8, 3), (9, 10, 3), (9, 8, 2)):
        set_lattice(ctx, nx, ny, lmax)
        set_lattice(fresh, nx, ny, lmax)
        assert ctx.get_matvec_config(precision) == (8, -1)
        assert all(same(outputs(ctx, precision), outputs(fresh, precision)))
        if lmax == 3:
            ctx.set_matvec_config(precision, 8, 0)
            assert not same(outputs(ctx, precision), outputs(fresh, precision))[0]
    ctx.close()
    fresh.close()


@pytest.mark.parametrize("precision", PRECISIONS)
@pytest.mark.parametrize("graph", [False, True])
def test_batch_autotuner_of_the_block_kernels(precision, graph):
    """With the block kernels chosen the batched autotuner really times and re-plans: a
    candidate's configuration, and the solution of the default one and of the transform."""
    print(f"[case] {precision} graph {graph}", flush=True)
    kh, po = wl.incidences(["x", "p10", "y"])
    subs = [(0, 0, 9, 20), (3, 2, 1, 1), (5, 4, 16, 7), (0, 0, 24, 20)]
    out = []
    for blocks, autotune in ((True, True), (True, False), (False, True)):
        ctx = tmhip.Context(0)
        set_lattice(ctx, 24, 20, 3)
        if blocks:
            ctx.set_matvec_config("fp64", 9, 0)
            ctx.set_matvec_config("mixed", 8, 0)
        ctx.set_batch_autotune(autotune)
        s, info = ctx.solve_batched(subs, kh, po, use_graph=graph, tol=1e-12, restart=40, precision=precision)
        assert all(i["status"] == 0 for q in info for i in q) and ctx.batch_graph_used() == graph
        prefetch, items = ctx.batch_config(precision)
        assert 1 <= prefetch <= (3 if precision == "mixed" else 2)
        assert items in ([wg // 6 for wg in (16384, 32768, 65536)] if blocks and autotune else [32768 // 6])
        out.append(torch.cat([q.reshape(-1) for q in s]))
        ctx.close()
    for o in out[1:]:
        assert float(torch.linalg.vector_norm(o - out[0])) < 1e-9 * float(torch.linalg.vector_norm(out[0]))
