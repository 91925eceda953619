"""Solves that end at the half step of a BiCGStab iteration, at tolerances within
rounding of the norm that decides it."""
import numpy as np
import pytest

import oracle as O
from workloads import jacobian_box

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


@pytest.mark.parametrize("n", [1, 3, 4, 5])
def test_tolerances_at_the_half_steps_norm(n):
    """The recursive residual of a solve is that of its last update; tolerances
    of a few units in its last place around it end at the half step, in the same
    iteration after the second half, or (the true residual, which differs by
    eps |A||x| / |r| relatively, can lie above) after a restart."""
    print("half step", n, flush=True)
    s = jacobian_box(11, 10, 9, n=n, seed=180 + n)
    A = O.from_system(s)
    kw = dict(precond=P.PREC_BJACOBI if n == 1 else P.PREC_AMG, max_iter=200)
    with P.System.from_dict(s) as sysm:
        for tol in (1e-4, 3e-6, 1e-7):
            sysm.setup(tol=tol, **kw)
            _, st = sysm.solve(s["b"])
            for k in range(-4, 5):
                t = st["rel_res_recursive"] * (1.0 + k * 2.0 ** -52)
                sysm.setup(tol=t, reuse_aggregates=1, **kw)
                x, q = sysm.solve(s["b"])
                assert q["status"] == P.OK and q["iterations"] <= st["iterations"] + 2, (tol, k, q)
                assert O.relres(A, s["b"], x.cpu().numpy()) <= t * (1.0 + 1e-6), (tol, k)
