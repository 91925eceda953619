"""The coarsest level's dense inverse on its own: with one level the
preconditioner is that inverse.  Full random matrices (every pair of cells
shares a face), so rows are exchanged; sizes around the register kernel's
column groups, its largest order and the general kernel beyond it, and a batch
of uneven systems.  Gauss-Jordan with partial pivoting is accurate to a small
multiple of m eps cond(A): bar 20 m eps cond(A)."""
import itertools

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


def _full(cells, n, seed):
    rng = np.random.default_rng(seed)
    la, ua = np.array(list(itertools.combinations(range(cells), 2)), dtype=np.int32).reshape(-1, 2).T
    d, u, lo = (rng.standard_normal((k, n, n)) for k in (cells, la.size, la.size))
    A = np.zeros((cells, n, cells, n))
    for i in range(cells):
        A[i, :, i] = d[i]
    for f, (i, j) in enumerate(zip(la, ua)):
        A[i, :, j], A[j, :, i] = u[f], lo[f]
    return la, ua, d, u, lo, A.reshape(cells * n, cells * n)


def _bar(A):
    return 20 * A.shape[0] * 2.3e-16 * np.linalg.cond(A)


@pytest.mark.parametrize("cells,n", [(1, 1), (1, 5), (3, 4), (13, 5), (16, 4), (17, 4), (16, 5), (63, 2), (42, 3),
                                     (32, 4), (33, 4)])
def test_one_level_is_the_dense_inverse(cells, n):
    print("coarsest", cells, n, flush=True)
    la, ua, d, u, lo, A = _full(cells, n, 90 + cells)
    r = np.random.default_rng(91).standard_normal((cells, n))
    with P.System(cells, n, la, ua, d, u, lo) as s:
        s.setup(precond=P.PREC_AMG, coarse_max=64)
        assert s.info()["levels"] == 1
        z = s.apply_precond(r).cpu().numpy().ravel()
        zt = s.apply_precond(r, transpose=True).cpu().numpy().ravel()
    for got, M in ((z, A), (zt, A.T)):
        ref = np.linalg.solve(M, r.ravel())
        assert np.linalg.norm(got - ref) <= _bar(A) * np.linalg.norm(ref)


def test_batch_of_dense_inverses_and_a_singular_one():
    parts = [_full(c, 3, 95 + c) for c in (1, 9, 22, 40)]
    cat = [np.concatenate([p[k] for p in parts]) for k in range(5)]
    co = np.cumsum([0] + [p[2].shape[0] for p in parts])
    fo = np.cumsum([0] + [p[0].size for p in parts])
    r = np.random.default_rng(96).standard_normal((co[-1], 3))
    with P.System(int(co[-1]), 3, *cat, cell_off=co, face_off=fo) as s:
        s.setup(precond=P.PREC_AMG, coarse_max=64)
        z = s.apply_precond(r).cpu().numpy()
        for k, p in enumerate(parts):
            ref = np.linalg.solve(p[5], r[co[k]:co[k + 1]].ravel())
            assert np.linalg.norm(z[co[k]:co[k + 1]].ravel() - ref) <= _bar(p[5]) * np.linalg.norm(ref)
        # two equal block rows of the third system
        d, u, lo = cat[2].copy(), cat[3].copy(), cat[4].copy()
        d[co[2]:co[3]] = 1.0
        u[fo[2]:fo[3]] = 1.0
        lo[fo[2]:fo[3]] = 1.0
        s.update_values(d, u, lo)
        with pytest.raises(P.CbsError) as e:
            s.setup(precond=P.PREC_AMG, coarse_max=64)
        assert e.value.code == P.ERR_SINGULAR


@pytest.mark.parametrize("precision,bar", [(P.PRECISION_FP64, 1e-11), (P.PRECISION_MIXED, 1e-5)])
@pytest.mark.parametrize("renumber", [0, 1])
@pytest.mark.parametrize("n", [1, 4, 5])
def test_tail_operator_is_the_cycle(n, renumber, precision, bar):
    """The dense operators of the coarse levels against the same levels run
    step by step, forward and transposed: one system and an uneven batch whose
    systems are frozen at different levels; in the caller's numbering (the
    members of an aggregate are then scattered) and the internal one.  Bars:
    rounding of a cycle in the hierarchy's precision, as for the oracle."""
    from workloads import concat_systems, jacobian_box, pressure_velocity
    make = (lambda *sh, seed: pressure_velocity(*sh, seed=seed)) if n == 4 else (
        lambda *sh, seed: jacobian_box(*sh, n=n, seed=seed))
    one = make(13, 11, 9, seed=97)
    cat = concat_systems([make(*sh, seed=98 + k) for k, sh in enumerate([(9, 8, 7), (2, 1, 1), (3, 3, 3), (11, 9, 8)])])
    for s in (one, cat):
        r = np.random.default_rng(99).standard_normal((s["N"], n))
        z = {}
        with P.System.from_dict(s) as sysm:
            for tail in (-1, 0):
                sysm.setup(precond=P.PREC_AMG, precision=precision, renumber=renumber, tail_rows=tail, coarse_max=8)
                z[tail] = [sysm.apply_precond(r, transpose=t).cpu().numpy() for t in (False, True)]
        for a, b in zip(z[-1], z[0]):
            assert np.linalg.norm(a - b) <= bar * np.linalg.norm(a)
