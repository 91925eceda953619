"""A setup that keeps the hierarchy's pattern after new coefficients: the levels'
values are the Galerkin products of the new level 0, which a block-Jacobi level
0 reads from the caller's blocks through slot maps and a coloured one from its
own copy; aggregates of up to more than 64 rows."""
import numpy as np
import pytest

import oracle as O
from workloads import jacobian_box, jacobian_graph, pressure_velocity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


def _np(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("kw", [dict(), dict(precision=1), dict(smoother=P.SMOOTH_DILU, dilu_levels=1),
                                dict(renumber=0), dict(match_passes=7, coarse_max=8)], ids=str)
def test_levels_are_galerkin_products_of_the_new_values(n, kw):
    """Sums of at most some hundred blocks in the oracle's order: bar 1e-13 of
    the largest value (the same sums differ by no more than their fused
    multiply-adds, of which there are none)."""
    print("re-setup", n, kw, flush=True)
    s = jacobian_graph(N=900, n=n, hubs=2, hub_degree=20, seed=170) if kw.get("renumber") == 0 else (
        pressure_velocity(13, 12, 11, seed=171) if n == 4 else jacobian_box(13, 12, 11, n=n, seed=171))
    rng = np.random.default_rng(172)
    with P.System.from_dict(s) as sysm:
        sysm.setup(precond=P.PREC_AMG, **{"coarse_max": 30, **kw})
        for _ in range(2):
            f = 1.0 + 0.1 * rng.random((s["N"], 1, 1))
            d = s["diag"].reshape(s["N"], n, n) * f
            sysm.update_values(d, 1.1 * s["upper"], 0.9 * s["lower"])
            sysm.setup(precond=P.PREC_AMG, reuse_aggregates=1, **{"coarse_max": 30, **kw})
            nlev = sysm.info()["levels"]
            assert nlev >= 2
            lv = [sysm.get_level(l) for l in range(nlev)]
            A = O.BCSR(lv[0]["N"], n, *(_np(lv[0][k]) for k in ("row_ptr", "col", "vals")))
            user = O.from_system({**s, "diag": d, "upper": 1.1 * s["upper"], "lower": 0.9 * s["lower"]})
            order = _np(lv[0]["order"])
            x = rng.standard_normal((A.N, n))
            xu = np.empty_like(x)
            xu[order] = x
            assert np.abs(O.spmv(A, x) - O.spmv(user, xu)[order]).max() <= 1e-13 * 64 * np.abs(user.vals).max()
            for l in range(nlev - 1):
                C = O.rap(A, _np(lv[l]["agg"]), lv[l + 1]["N"])
                assert np.array_equal(C.row_ptr, _np(lv[l + 1]["row_ptr"]))
                assert np.array_equal(C.col, _np(lv[l + 1]["col"]))
                assert np.abs(C.vals - _np(lv[l + 1]["vals"])).max() <= 1e-13 * np.abs(C.vals).max()
                A = C
        xs, st = sysm.solve(s["b"])
        r = s["b"] - O.spmv(user, _np(xs))
    assert np.linalg.norm(r) <= 1.1e-6 * np.linalg.norm(s["b"])
