"""A W-cycle whose second run starts on a level large enough to prolong in a
pass of its own, with odd and even numbers of sweeps there: the pass also moves
the iterate between the level's two vectors."""
import numpy as np
import pytest

import oracle as O
from workloads import jacobian_box

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


def _np(t):
    return t.detach().cpu().numpy()


@pytest.fixture(scope="module")
def system():
    return jacobian_box(59, 57, 53, n=2, seed=180)


@pytest.mark.parametrize("pre,post", [(1, 2), (2, 1), (1, 1), (3, 0), (0, 3), (2, 2)])
@pytest.mark.parametrize("precision", [P.PRECISION_FP64, P.PRECISION_MIXED])
def test_w_cycle_on_a_large_level_matches_oracle(system, precision, pre, post):
    """Bars of the cycles elsewhere: 1e-11 (FP64) and 1e-5 (FP32) of the largest value."""
    print("large W-cycle", precision, pre, post, flush=True)
    s = system
    f = np.random.default_rng(181).standard_normal((s["N"], 2))
    with P.System.from_dict(s) as sysm:
        sysm.setup(precond=P.PREC_AMG, precision=precision, omega=0.9, match_passes=1, w_levels=1,
                   pre_sweeps=pre, post_sweeps=post)
        lv = [sysm.get_level(l) for l in range(sysm.info()["levels"])]
        assert lv[1]["N"] >= 65536
        order = _np(lv[0]["order"])
        A = O.BCSR(lv[0]["N"], 2, *(_np(lv[0][k]) for k in ("row_ptr", "col", "vals")))
        z = _np(sysm.apply_precond(f))
    aggs = [_np(v["agg"]) for v in lv[:-1]]
    ref = np.empty_like(f)
    ref[order] = O.AMG(A, nu1=pre, nu2=post, omega=0.9, aggs=aggs, w_levels=1).apply(f[order])
    assert np.abs(z - ref).max() <= (1e-5 if precision == P.PRECISION_MIXED else 1e-11) * np.abs(ref).max()
