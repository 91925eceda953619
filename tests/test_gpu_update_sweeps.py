"""BiCGStab iterations whose vector updates also make the preconditioner's first
sweep: work items of several tiles and ragged ones, every block size and
precision, both directions, batches with systems of one row and systems that
finish early, and the size from which the sweep is a launch of its own."""
import numpy as np
import pytest

import oracle as O
from workloads import concat_systems, jacobian_box

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


def _np(t):
    return t.detach().cpu().numpy()


def _iterate(sysm, s, transposed, its):
    """its BiCGStab iterations with the handle's own products and preconditioner."""
    mul = lambda v: _np(sysm.spmv(v, transpose=transposed))        # noqa: E731
    prec = lambda v: _np(sysm.apply_precond(v, transpose=transposed))        # noqa: E731
    b = s["b"]
    x, r = np.zeros_like(b), b.copy()
    rh, p, v = r.copy(), np.zeros_like(b), np.zeros_like(b)
    rho0 = alpha = omega = 1.0
    rho = (rh * r).sum()
    for _ in range(its):
        p = r + (rho / rho0) * (alpha / omega) * (p - omega * v)
        ph = prec(p)
        v = mul(ph)
        alpha = rho / (rh * v).sum()
        sv = r - alpha * v
        sh = prec(sv)
        t = mul(sh)
        omega = (t * sv).sum() / (t * t).sum()
        x = x + alpha * ph + omega * sh
        r = sv - omega * t
        rho0, rho = rho, (rh * r).sum()
    return x


# (scalar systems with negative couplings stop coarsening early, and their dense
# coarsest inverse takes minutes on the largest shape)
@pytest.mark.parametrize("shape,n", [((5, 4, 3), n) for n in (1, 2, 3, 4, 5)] +
                         [((23, 11, 9), n) for n in (1, 2, 3, 4, 5)] + [((61, 53, 47), n) for n in (2, 3, 4, 5)])
@pytest.mark.parametrize("precision", [P.PRECISION_FP64, P.PRECISION_MIXED])
def test_iterate_is_that_of_separate_steps(shape, precision, n):
    """Two iterations against the same recurrence made from cbs_spmv and
    cbs_apply_precond.  FP64: sums of 760,000 terms and the order of a product's
    blocks, bar 1e-10.  Mixed: a rounding of p can move its FP32 copy by an FP32
    unit, which the second iteration carries on: bar 1e-5."""
    print("update sweeps", shape, precision, n, flush=True)
    s = jacobian_box(*shape, n=n, seed=140 + n)
    with P.System.from_dict(s) as sysm:
        sysm.setup(precond=P.PREC_AMG, precision=precision, tol=1e-14, max_iter=2, match_passes=2, coarse_max=40)
        for tr in (False, True):
            x, _ = sysm.solve_transpose(s["b"]) if tr else sysm.solve(s["b"])
            ref = _iterate(sysm, s, tr, 2)
            err = np.linalg.norm(_np(x) - ref) / np.linalg.norm(ref)
            assert err <= (1e-10 if precision == P.PRECISION_FP64 else 1e-5), (tr, err)


@pytest.mark.parametrize("precision", [P.PRECISION_FP64, P.PRECISION_MIXED])
def test_batch_of_uneven_systems_converges(precision):
    """Systems that are through while others go on, down to two rows."""
    systems = [jacobian_box(*sh, n=3, seed=150 + k) for k, sh in
               enumerate([(2, 1, 1), (3, 3, 2), (16, 15, 14), (9, 2, 1), (21, 20, 19)])]
    cat = concat_systems(systems)
    with P.System.from_dict(cat) as bs:
        bs.setup(precond=P.PREC_AMG, precision=precision, tol=1e-10, max_iter=100)
        x, st = bs.solve_batch(cat["b"])
    x = _np(x)
    for k, sk in enumerate(systems):
        xk = x[cat["cell_off"][k]:cat["cell_off"][k + 1]]
        r = sk["b"] - O.spmv(O.from_system(sk), xk)
        assert np.linalg.norm(r) <= 1.01e-10 * np.linalg.norm(sk["b"]), k


@pytest.mark.parametrize("shape", [(128, 64, 64), (127, 64, 64)])
def test_size_from_which_the_sweep_is_its_own_launch(shape):
    """2,097,152 values and just under."""
    print("update sweep limit", shape, flush=True)
    s = jacobian_box(*shape, n=4, seed=160)
    with P.System.from_dict(s) as sysm:
        sysm.setup(precond=P.PREC_AMG, precision=P.PRECISION_FP64, tol=1e-14, max_iter=1)
        x, _ = sysm.solve(s["b"])
        ref = _iterate(sysm, s, False, 1)
    assert np.linalg.norm(_np(x) - ref) <= 1e-10 * np.linalg.norm(ref)
