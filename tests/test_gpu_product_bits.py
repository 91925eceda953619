"""cbs_spmv gives the same bits for the same values and vector in every call,
whichever kernel the call takes: the block-CSR product or the sliced one, with
whole rows and with rows split over threads."""
import numpy as np
import pytest

from workloads import jacobian_box, jacobian_graph

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("mesh", ["two cells", "box", "graph", "whole rows", "32767 rows", "32768 rows"])
def test_every_product_has_the_same_bits(n, mesh):
    """Rows of 2 to 60 blocks; 1 to 8 threads per row."""
    print("product bits", n, mesh, flush=True)
    s = {"two cells": lambda: jacobian_box(2, 1, 1, n=n, seed=220),
         "box": lambda: jacobian_box(9, 8, 7, n=n, seed=221),
         "graph": lambda: jacobian_graph(N=300, n=n, hubs=60, hub_degree=55, seed=222),
         # 98,304 scalar rows and just under: 4x4 24,576 and 24,575 rows
         "whole rows": lambda: jacobian_box(983, 25, 1, n=n, seed=226) if n % 2 else jacobian_box(32, 32, 24, n=n, seed=226),
         "32767 rows": lambda: jacobian_box(217, 151, 1, n=n, seed=223),
         "32768 rows": lambda: jacobian_box(32, 32, 32, n=n, seed=224)}[mesh]()
    x = torch.tensor(np.random.default_rng(225).standard_normal((s["N"], n)), device="cuda")
    with P.System.from_dict(s) as sysm:
        for tr in (False, True):
            y = sysm.spmv(x, transpose=tr)
            for k in range(19):
                assert torch.equal(sysm.spmv(x, transpose=tr), y), (tr, k)
