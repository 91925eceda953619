"""cbs_spmv over many products with the same values: the first ones read the
block CSR, later ones the sliced copy, and replaced values start over."""
import numpy as np
import pytest

import oracle as O
from workloads import jacobian_box, jacobian_graph, pressure_velocity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("mesh", ["box", "graph", "two cells"])
def test_every_product_is_the_oracles(n, mesh):
    """Rows of 2 to 60 blocks, remainders of four among them.  Sums of m terms
    round to at most m eps of their magnitudes: bar 1e-14 times 8 to 66 terms'
    largest products, as for the single product."""
    print("products", n, mesh, flush=True)
    s = {"box": lambda: jacobian_box(7, 6, 5, n=n, seed=80 + n),
         "graph": lambda: jacobian_graph(N=300, n=n, hubs=3, hub_degree=40, seed=81),
         "two cells": lambda: jacobian_box(2, 1, 1, n=n, seed=82)}[mesh]()
    A = O.from_system(s)
    x = np.random.default_rng(83).standard_normal((s["N"], n))
    width = int(np.diff(A.row_ptr).max()) + 1
    scale = np.abs(A.vals).max() * np.abs(x).max() * width
    with P.System.from_dict(s) as sysm:
        for tr, ref in ((False, O.spmv(A, x)), (True, O.spmv_t(A, x))):
            for k in range(19):
                y = sysm.spmv(x, transpose=tr).cpu().numpy()
                assert np.abs(y - ref).max() <= 1e-14 * scale, (tr, k)
        sysm.update_values(2.0 * s["diag"], 2.0 * s["upper"], 2.0 * s["lower"])
        for tr, ref in ((False, O.spmv(A, x)), (True, O.spmv_t(A, x))):
            y = sysm.spmv(x, transpose=tr).cpu().numpy()
            assert np.abs(y - 2.0 * ref).max() <= 2e-14 * scale, tr


def test_products_before_and_after_setup_agree():
    """A setup that names a schedule uses the sliced copy at once."""
    s = pressure_velocity(9, 8, 7, seed=84)
    x = np.random.default_rng(85).standard_normal((s["N"], 4))
    with P.System.from_dict(s) as sysm:
        y0 = sysm.spmv(x).cpu().numpy()
        sysm.setup(precond=P.PREC_NONE, schedule=3)
        y1 = sysm.spmv(x).cpu().numpy()
    assert np.abs(y0 - y1).max() <= 1e-14 * 8 * np.abs(y0).max()
