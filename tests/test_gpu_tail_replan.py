"""A setup on kept aggregates whose values let a level that had stalled coarsen
further: the hierarchy gets more levels below the same first level of the
V-cycle tail, whose operators are then planned again."""
import numpy as np
import pytest

from workloads import box_faces

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


@pytest.mark.parametrize("n", [1, 4])
@pytest.mark.parametrize("precision", [P.PRECISION_FP64, P.PRECISION_MIXED])
def test_levels_appended_below_the_tails_first_level(n, precision):
    """A chain of 240 cells coupled in pairs stops at 120 rows; coupled all
    along it goes on.  Against the same cycle step by step: 1e-11, FP32 1e-5."""
    print("tail replan", n, precision, flush=True)
    N = 240
    la, ua, _ = box_faces(N, 1, 1)
    rng = np.random.default_rng(210 + n)
    off = rng.uniform(0.5, 1.0, N - 1)[:, None, None] * (np.eye(n) + 0.2 * rng.standard_normal((N - 1, n, n)))
    off[::2] *= 2.0                                   # the pairs are the stronger couplings

    def values(c):
        diag = np.tile(np.eye(n), (N, 1, 1))
        np.add.at(diag, la, c)
        np.add.at(diag, ua, c)
        return diag, -c, -c

    pairs = off.copy()
    pairs[1::2] = 0.0
    f = rng.standard_normal((N, n))
    kw = dict(precond=P.PREC_AMG, precision=precision, coarse_max=8)
    z = {}
    for tail in (0, -1):
        with P.System(N, n, la, ua, *values(pairs)) as sysm:
            sysm.setup(tail_rows=tail, **kw)
            assert sysm.info()["levels"] == 2
            sysm.update_values(*values(off))
            sysm.setup(tail_rows=tail, reuse_aggregates=1, **kw)
            assert sysm.info()["levels"] > 2
            z[tail] = [sysm.apply_precond(f, transpose=t).cpu().numpy() for t in (False, True)]
            x, st = sysm.solve(f)
            assert st["status"] == P.OK
    for a, b in zip(z[0], z[-1]):
        assert np.abs(a - b).max() <= (1e-5 if precision == P.PRECISION_MIXED else 1e-11) * np.abs(b).max()
