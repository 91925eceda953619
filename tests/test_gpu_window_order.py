"""A level below the finest with more than 32,768 rows, whose sliced copies
hold the rows of each window of 64 longest first: its kernels, the cycle and
the transposed cycle, for every block size in both precisions, the last window
not full."""
import numpy as np
import pytest

import oracle as O
from workloads import jacobian_box

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


def _np(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("precision,scaled", [(P.PRECISION_FP64, 1), (P.PRECISION_MIXED, 1), (P.PRECISION_MIXED, 0)])
def test_window_ordered_level_matches_oracle(n, precision, scaled):
    """Bars of the level kernels and cycles elsewhere: 1e-14 (FP32: 1e-6) of
    the sums' magnitudes for a residual, 1e-13 (1e-5) for a sweep, 1e-11
    (1e-5) for a cycle; the adjoint identity as a cycle."""
    print("window order", n, precision, scaled, flush=True)
    mixed = precision == P.PRECISION_MIXED
    s = jacobian_box(53, 47, 43, n=n, seed=120 + n)
    rng = np.random.default_rng(121)
    with P.System.from_dict(s) as sysm:
        sysm.setup(precond=P.PREC_AMG, precision=precision, omega=0.9, match_passes=1,
                   pre_sweeps=1, post_sweeps=1, scaled_sweeps=scaled)
        nlev = sysm.info()["levels"]
        lv = sysm.get_level(1)
        A = O.BCSR(lv["N"], n, _np(lv["row_ptr"]), _np(lv["col"]), _np(lv["vals"]))
        assert A.N >= 32768 and A.N % 64 and np.diff(A.row_ptr).max() > np.diff(A.row_ptr).min()
        b, x = rng.standard_normal((A.N, n)), rng.standard_normal((A.N, n))
        if mixed:                      # the kernels take FP32 inputs
            b, x = b.astype(np.float32).astype(np.float64), x.astype(np.float32).astype(np.float64)
        scale = np.abs(A.vals).max() * np.abs(x).max() * 64 + np.abs(b).max()
        r = _np(sysm.level_apply(1, P.LEVEL_RESIDUAL, b, x)).astype(np.float64)
        assert np.abs(r - (b - O.spmv(A, x))).max() <= (1e-6 if mixed else 1e-14) * scale
        Dinv = O.blockinv(O.diag_blocks(A))
        y = _np(sysm.level_apply(1, P.LEVEL_SWEEP, b, x)).astype(np.float64)
        ref = (x + 0.9 * (b - (Dinv @ O.spmv(A, x)[:, :, None])[:, :, 0]) if mixed and scaled
               else O.bjacobi_sweep(A, Dinv, b, x, 0.9))
        assert np.abs(y - ref).max() <= (1e-5 if mixed else 1e-13) * (np.abs(ref).max() + 1.0)

        lv0 = sysm.get_level(0)
        order = _np(lv0["order"])
        A0 = O.BCSR(lv0["N"], n, _np(lv0["row_ptr"]), _np(lv0["col"]), _np(lv0["vals"]))
        aggs = [_np(sysm.get_level(l)["agg"]) for l in range(nlev - 1)]
        f, g = rng.standard_normal((A0.N, n)), rng.standard_normal((A0.N, n))
        z, zt = _np(sysm.apply_precond(f)), _np(sysm.apply_precond(g, transpose=True))
    assert abs((z * g).sum() - (f * zt).sum()) <= (1e-5 if mixed else 1e-11) * np.linalg.norm(z) * np.linalg.norm(g)
    if n == 1:        # (negative couplings end the coarsening early; the oracle would invert thousands of rows)
        return
    zi = O.AMG(A0, nu1=1, nu2=1, omega=0.9, aggs=aggs).apply(f[order])
    zr = np.empty_like(zi)
    zr[order] = zi
    assert np.abs(z - zr).max() <= (1e-5 if mixed else 1e-11) * np.abs(zr).max()
