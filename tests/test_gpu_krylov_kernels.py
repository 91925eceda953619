"""The Krylov loops' own kernels against the oracle's iterates, at the sizes
where their splits change: groups of eight basis vectors and their remainders,
a triangular solve beyond the staged size, and every length of a work item."""
import numpy as np
import pytest

import oracle as O
from workloads import concat_systems, jacobian_box, pressure_velocity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


@pytest.mark.parametrize("solver", ["gmres", "fgmres"])
@pytest.mark.parametrize("restart", [1, 7, 8, 9, 16, 64, 66])
def test_gmres_iterate_matches_oracle(restart, solver):
    """x after one whole cycle and three iterations of the next, block-Jacobi
    preconditioned (far from converged).  Both orthogonalise to rounding, so
    the iterates differ by the rounding of at most 69 steps on a system of
    condition below 1e5: 69 * 1.1e-16 * 1e5 = 8e-10, bar 1e-9."""
    print("gmres iterate", solver, restart, flush=True)
    s = pressure_velocity(9, 8, 7, seed=71)
    A = O.from_system(s)
    its = restart + 3
    xo, so = getattr(O, solver)(A, s["b"], prec=O.PREC_BJACOBI, tol=1e-14, maxit=its, restart=restart)
    with P.System.from_dict(s) as sysm:
        sysm.setup(precond=P.PREC_BJACOBI, restart=restart, tol=1e-14, max_iter=its,
                   solver=P.SOLVER_GMRES if solver == "gmres" else P.SOLVER_FGMRES)
        x, st = sysm.solve(s["b"])
    assert st["iterations"] == so["iterations"] == its
    x = x.cpu().numpy()
    assert np.linalg.norm(x - xo) <= 1e-9 * np.linalg.norm(xo), np.linalg.norm(x - xo) / np.linalg.norm(xo)


@pytest.mark.parametrize("shape", [(9, 7, 5), (81, 83, 85), (107, 105, 109), (130, 131, 129)])
def test_bicgstab_iterate_over_item_lengths(shape):
    """x after three iterations on scalar systems of 315 to 2.2M unknowns (work
    items of 512, 1024, 2048 and 4096 elements, the last ones ragged).  Sums of
    m terms differ by at most m * 1.1e-16 relative to the sum of magnitudes,
    2.4e-10 for the largest; the usual sqrt(m) growth is 1.7e-13.  Bar 1e-10."""
    print("item lengths", shape, flush=True)
    s = jacobian_box(*shape, n=1, seed=72)
    A = O.from_system(s)
    xo, so = O.bicgstab(A, s["b"], prec=O.PREC_BJACOBI, tol=1e-14, maxit=3)
    with P.System.from_dict(s) as sysm:
        sysm.setup(precond=P.PREC_BJACOBI, tol=1e-14, max_iter=3)
        x, st = sysm.solve(s["b"])
    assert st["iterations"] == so["iterations"] == 3
    x = x.cpu().numpy()
    assert np.linalg.norm(x - xo) <= 1e-10 * np.linalg.norm(xo), np.linalg.norm(x - xo) / np.linalg.norm(xo)


def test_batched_gmres_systems_match_solo_iterates():
    """A batch shares every launch: systems of one item and of several."""
    systems = [pressure_velocity(3, 2, 2, seed=73), pressure_velocity(9, 8, 7, seed=74),
               pressure_velocity(5, 5, 5, seed=75)]
    cat = concat_systems(systems)
    kw = dict(precond=P.PREC_BJACOBI, solver=P.SOLVER_GMRES, restart=9, tol=1e-14, max_iter=12)
    with P.System.from_dict(cat) as bs:
        bs.setup(**kw)
        x, _ = bs.solve(cat["b"])
    x = x.cpu().numpy()
    for k, sk in enumerate(systems):
        xo, _ = O.gmres(O.from_system(sk), sk["b"], prec=O.PREC_BJACOBI, tol=1e-14, maxit=12, restart=9)
        xk = x[cat["cell_off"][k]:cat["cell_off"][k + 1]]
        assert np.linalg.norm(xk - xo) <= 1e-9 * np.linalg.norm(xo), k


def test_breakdown_reaches_the_host():
    """A block [[0, 1], [-1, 0]] makes (r, A r) vanish: BiCGStab without a
    preconditioner breaks down, restarts once and gives up, alone and beside a
    system that converges (its solution is still written)."""
    D = np.array([[[0.0, 1.0], [-1.0, 0.0]], [[2.0, 1.0], [0.0, 3.0]]])
    none = np.zeros((0, 2, 2))
    no = np.zeros(0, np.int32)
    with P.System(1, 2, no, no, D[:1], none, none) as s:
        s.setup(precond=P.PREC_NONE)
        with pytest.raises(P.CbsError) as e:
            s.solve(np.array([[1.0, 0.0]]))
        assert e.value.code == P.ERR_BREAKDOWN
    with P.System(2, 2, no, no, D, none, none, cell_off=[0, 1, 2], face_off=[0, 0, 0]) as s:
        s.setup(precond=P.PREC_NONE, tol=1e-12)
        with pytest.raises(P.CbsError) as e:
            s.solve_batch(np.array([[1.0, 0.0], [3.0, 3.0]]))
        assert e.value.code == P.ERR_BREAKDOWN
        # the handle still works
        s.update_values(D[[1, 1]], none, none)
        s.setup(precond=P.PREC_NONE, tol=1e-12)
        x, st = s.solve_batch(np.array([[3.0, 3.0], [3.0, 3.0]]))
        assert all(q["status"] == P.OK for q in st)
        assert np.allclose(x.cpu().numpy(), 1.0, atol=1e-10)


@pytest.mark.parametrize("solver", [P.SOLVER_BICGSTAB, P.SOLVER_FGMRES, P.SOLVER_GMRES])
@pytest.mark.parametrize("max_iter,tol", [(0, 1e-8), (3, 1e-14), (500, 1e-10)])
def test_reported_residuals_are_those_of_x(solver, max_iter, tol):
    """The statistics' true residual against the oracle's on the returned x,
    where the solve stops at once, at the cap and converged (relative error of
    a residual formed in another order: eps |A||x| / |r|, under 1e-3 at 1e-10)."""
    s = pressure_velocity(8, 7, 6, seed=76)
    A = O.from_system(s)
    x0 = np.random.default_rng(77).standard_normal((s["N"], 4))
    with P.System.from_dict(s) as sysm:
        sysm.setup(precond=P.PREC_AMG, solver=solver, restart=10, tol=tol, max_iter=max_iter)
        x, st = sysm.solve(s["b"], x0)
    assert abs(O.relres(A, s["b"], x.cpu().numpy()) - st["rel_res_true"]) <= 1e-3 * st["rel_res_true"]
    assert abs(O.relres(A, s["b"], x0) - st["rel_res_initial"]) <= 1e-9 * st["rel_res_initial"]
    assert abs(st["rel_res_recursive"] - st["rel_res_true"]) <= 0.1 * st["rel_res_true"] + 1e-13
    assert st["status"] == (P.OK if max_iter == 500 else P.NOT_CONVERGED)
