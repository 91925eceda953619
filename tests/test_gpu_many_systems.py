"""Batches of hundreds of small systems, on both sides of the counts from which
their kernels change."""
import itertools

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


def _full(cells, n, rng):
    """A matrix in which every pair of cells shares a face."""
    la, ua = np.array(list(itertools.combinations(range(cells), 2)), dtype=np.int32).reshape(-1, 2).T
    d, u, lo = (rng.standard_normal((k, n, n)) for k in (cells, la.size, la.size))
    A = np.zeros((cells, n, cells, n))
    A[np.arange(cells), :, np.arange(cells)] = d
    A[la, :, ua], A[ua, :, la] = u, lo
    return la, ua, d, u, lo, A.reshape(cells * n, cells * n)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("most", [48, 49])
@pytest.mark.parametrize("count", [768, 769])
def test_dense_inverses_of_many_systems(count, most, n):
    """Full random matrices of up to 48 unknowns and of up to 49 (or the block
    size's next).  Gauss-Jordan with partial pivoting: 20 m eps cond(A)."""
    print("many inverses", count, most, n, flush=True)
    rng = np.random.default_rng(260 + n)
    big = most // n if most == 48 else 48 // n + 1
    kinds = [_full(c, n, rng) for c in (1, 2, 3, max(1, big // 2), big)]
    pick = [kinds[(i * i + i // 5) % 5] for i in range(count - 1)] + [kinds[4]]
    cat = [np.concatenate([p[k] for p in pick]) for k in range(5)]
    co = np.cumsum([0] + [p[2].shape[0] for p in pick])
    fo = np.cumsum([0] + [p[0].size for p in pick])
    r = rng.standard_normal((co[-1], n))
    with P.System(int(co[-1]), n, *cat, cell_off=co, face_off=fo) as s:
        s.setup(precond=P.PREC_AMG, coarse_max=64)
        assert s.info()["levels"] == 1
        z = [s.apply_precond(r, transpose=t).cpu().numpy() for t in (False, True)]
        cat[2][co[-2]:] = 1.0                          # the last system is singular
        cat[3][fo[-2]:] = 1.0
        cat[4][fo[-2]:] = 1.0
        if pick[-1][5].shape[0] > 1:
            s.update_values(*cat[2:])
            with pytest.raises(P.CbsError) as e:
                s.setup(precond=P.PREC_AMG, coarse_max=64)
            assert e.value.code == P.ERR_SINGULAR
    for k, p in enumerate(pick):
        for got, M in ((z[0], p[5]), (z[1], p[5].T)):
            ref = np.linalg.solve(M, r[co[k]:co[k + 1]].ravel())
            bar = 20 * M.shape[0] * 2.3e-16 * np.linalg.cond(M)
            assert np.linalg.norm(got[co[k]:co[k + 1]].ravel() - ref) <= bar * np.linalg.norm(ref), k


@pytest.mark.parametrize("precision", [P.PRECISION_FP64, P.PRECISION_MIXED])
@pytest.mark.parametrize("count", [128, 129])
def test_tail_of_the_coarsest_level_alone(count, precision):
    """Chains of 20 cells, 5x5, whose level 1 is the coarsest: two workgroups to a
    system of the tail's product, up to 256 of them, else the level's own launches.
    Against the cycle without a tail: 1e-11, FP32 1e-5."""
    rng = np.random.default_rng(270)
    N, n = 20, 5
    la = np.arange(N - 1, dtype=np.int32)
    off = rng.uniform(0.2, 1.0, (count, N - 1))[:, :, None, None] * (np.eye(n) + 0.2 * rng.standard_normal((count, N - 1, n, n)))
    diag = np.tile(0.2 * np.eye(n), (count, N, 1, 1))
    diag[:, :-1] += off
    diag[:, 1:] += off
    flat = lambda a: a.reshape(-1, n, n)        # noqa: E731
    f = rng.standard_normal((count * N, n))
    z = {}
    with P.System(count * N, n, np.tile(la, count), np.tile(la + 1, count), flat(diag), flat(-off), flat(-off),
                  cell_off=N * np.arange(count + 1), face_off=(N - 1) * np.arange(count + 1)) as s:
        for tail in (-1, 0):
            s.setup(precond=P.PREC_AMG, precision=precision, tail_rows=tail)
            assert s.info()["levels"] == 2
            z[tail] = [s.apply_precond(f, transpose=t).cpu().numpy() for t in (False, True)]
            assert all(st["status"] == P.OK for st in s.solve_batch(f)[1])
    for a, b in zip(z[0], z[-1]):
        assert np.abs(a - b).max() <= (1e-5 if precision == P.PRECISION_MIXED else 1e-11) * np.abs(b).max()


@pytest.mark.parametrize("solver", [P.SOLVER_BICGSTAB, P.SOLVER_GMRES, P.SOLVER_FGMRES])
@pytest.mark.parametrize("count", [1023, 1024])
def test_state_of_many_systems_reaches_the_host(count, solver):
    """Systems that are solved, have a zero right side, start converged or (with
    BiCGStab) break down, each with its own statistics, as on their own."""
    print("many states", count, solver, flush=True)
    kinds = {"solved": (np.array([[2.0, 1.0], [0.0, 3.0]]), [3.0, 3.0]), "zero": (np.eye(2), [0.0, 0.0]),
             "broken": (np.array([[0.0, 1.0], [-1.0, 0.0]]), [1.0, 0.0]), "started": (4.0 * np.eye(2), [4.0, 4.0])}
    bicg = solver == P.SOLVER_BICGSTAB
    pick = [list(kinds)[(i * 7 + i // 4) % 4] for i in range(count)]
    if not bicg:
        pick = [k if k != "broken" else "solved" for k in pick]
    D, b = np.array([kinds[k][0] for k in pick]), np.array([kinds[k][1] for k in pick])
    x0 = np.array([[1.0, 1.0] if k == "started" else [0.0, 0.0] for k in pick])
    none, no = np.zeros((0, 2, 2)), np.zeros(0, np.int32)
    kw = dict(precond=P.PREC_NONE, solver=solver, tol=1e-12, restart=5)

    def solve(sel):
        m = len(sel)
        with P.System(m, 2, no, no, D[sel], none, none, cell_off=np.arange(m + 1), face_off=np.zeros(m + 1)) as s:
            s.setup(**kw)
            bd, x = (torch.tensor(a[sel], device="cuda") for a in (b, x0))
            st = (P.Stats * m)()
            rc = P.lib().cbs_solve_batch(s.h, bd.data_ptr(), x.data_ptr(), st)
        assert rc == min(q.status for q in st)
        return x.cpu().numpy(), [(q.status, q.iterations, q.rel_res_true, q.rel_res_recursive, q.rel_res_initial) for q in st]

    x, st = solve(list(range(count)))
    own = {k: solve([pick.index(k)]) for k in set(pick)}
    for i, k in enumerate(pick):
        assert st[i] == own[k][1][0], (i, k)
        assert np.array_equal(x[i], own[k][0][0]), (i, k)
    assert {own[k][1][0][0] for k in own} == ({P.OK, P.ERR_BREAKDOWN} if bicg else {P.OK})
