"""bench.py names the product that ran from the context's configuration (no GPU), and not
from how fast it was: a transformed product slower than the matrix cores' peak is still no
matrix-core fraction."""
import types

import pytest

import bench


def context(lmax, nx, ny, items):
    return types.SimpleNamespace(lmax=lmax, get_matvec_config=lambda prec: (8, items),
                                 get_lattice=lambda: (nx, ny, 0.6))


@pytest.mark.parametrize("lmax,nx,ny,fp64,mixed", [(3, 20, 20, True, True), (3, 320, 300, True, True),
                                                   (1, 4, 301, False, True), (3, 321, 4, False, False),
                                                   (4, 9, 151, False, True), (6, 100, 101, False, True),
                                                   (6, 100, 201, False, False), (2, 5, 321, False, False)])
def test_product_follows_the_configuration_and_the_lattice(lmax, nx, ny, fp64, mixed):
    for prec, fits in (("fp64", fp64), ("mixed", mixed)):
        assert bench.transformed(context(lmax, nx, ny, -1), prec) == fits
        assert not bench.transformed(context(lmax, nx, ny, 0), prec)
        # subregions of a larger lattice
        assert bench.transformed(context(lmax, 900, 900, -1), prec, [(3, 4), (nx, ny)]) == fits


def test_slow_transformed_product_is_not_a_matrix_core_fraction():
    dom = {"tflops": 3.0, "avg_launch_ms": 0.03, "flops_per_launch": 1e8}
    assert bench.fraction(3.0, bench.PEAK_FP32_MFMA, True) is None
    r = bench.matvec_roofline(dom, 3, 20, 20, 1, "20x20", ["block_matvec_lds_kernel"], True)
    assert r["bound"] == "hbm" and r["kernel"].startswith("spec_rows")
    r = bench.matvec_roofline(dom, 3, 20, 20, 1, "20x20", ["block_matvec_lds_kernel"], False)
    assert r["bound"] == "mfma" and r["kernel"] == "block_matvec_lds_kernel"
