"""BiCGStab iterations whose two products come with A x, on both sides of the
number of workgroups up to which they do, one thread to a scalar row and
several, forward and transposed, and a batch, which keeps a launch for them."""
import numpy as np
import pytest

import oracle as O
from workloads import concat_systems, jacobian_box, jacobian_graph

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


def _transposed(A):
    vals = np.ascontiguousarray(A.vals[_mirror(A)].transpose(0, 2, 1))
    return O.BCSR(A.N, A.vals.shape[1], A.row_ptr, A.col, vals)


def _mirror(A):
    rows = np.repeat(np.arange(A.N), np.diff(A.row_ptr))
    key = rows.astype(np.int64) * A.N + A.col
    order = np.argsort(key)
    return order[np.searchsorted(key[order], A.col.astype(np.int64) * A.N + rows)]


@pytest.mark.parametrize("mesh,n", [(m, n) for m in ("two cells", "ragged", "graph") for n in (1, 2, 3, 4, 5)] +
                         [(m, n) for m in ("4096 workgroups", "4097 workgroups") for n in (1, 4)])
def test_bicgstab_iterate_matches_oracle(mesh, n):
    """x after two iterations.  Sums of m terms differ by at most m * 1.1e-16
    relative to the sum of magnitudes, 1.2e-10 for the largest, 1.05M; the usual
    sqrt(m) growth is 1.1e-13.  Bar 1e-10."""
    print("products", mesh, n, flush=True)
    s = {"two cells": lambda: jacobian_box(2, 1, 1, n=n, seed=130), "ragged": lambda: jacobian_box(9, 7, 5, n=n, seed=131),
         "graph": lambda: jacobian_graph(N=700, n=n, hubs=3, hub_degree=40, seed=132),
         "4096 workgroups": lambda: jacobian_box(64, 64, 64, n=n, seed=133),
         "4097 workgroups": lambda: jacobian_box(241, 64, 17, n=n, seed=134)}[mesh]()
    assert mesh[0] != "4" or -(-s["N"] // 64) == int(mesh[:4])
    A = O.from_system(s)
    its = 1 if mesh == "two cells" else 2
    for tr in (False, True):
        xo, _ = O.bicgstab(_transposed(A) if tr else A, s["b"], prec=O.PREC_BJACOBI, tol=1e-14, maxit=its)
        with P.System.from_dict(s) as sysm:
            sysm.setup(precond=P.PREC_BJACOBI, tol=1e-14, max_iter=its)
            x, _ = sysm.solve_transpose(s["b"]) if tr else sysm.solve(s["b"])
        x = x.cpu().numpy()
        assert np.linalg.norm(x - xo) <= 1e-10 * np.linalg.norm(xo), (tr, np.linalg.norm(x - xo) / np.linalg.norm(xo))


def test_batch_matches_solo_iterates():
    systems = [jacobian_box(2, 1, 1, n=3, seed=135), jacobian_box(9, 8, 7, n=3, seed=136), jacobian_box(5, 5, 5, n=3, seed=137)]
    cat = concat_systems(systems)
    with P.System.from_dict(cat) as bs:
        bs.setup(precond=P.PREC_BJACOBI, tol=1e-14, max_iter=1)
        x, _ = bs.solve(cat["b"])
    x = x.cpu().numpy()
    for k, sk in enumerate(systems):
        xo, _ = O.bicgstab(O.from_system(sk), sk["b"], prec=O.PREC_BJACOBI, tol=1e-14, maxit=1)
        xk = x[cat["cell_off"][k]:cat["cell_off"][k + 1]]
        assert np.linalg.norm(xk - xo) <= 1e-10 * np.linalg.norm(xo), k
