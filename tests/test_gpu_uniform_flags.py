"""Systems that break down or finish in a launch whose other workgroups read the
same flag: systems of many work items, alone and beside others."""
import numpy as np
import pytest

import oracle as O
from workloads import concat_systems, jacobian_box

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


@pytest.mark.parametrize("cells", [1, 300, 20000])
def test_breakdown_of_many_workgroups(cells):
    """Blocks [[0, 1], [-1, 0]] make (r, A r) vanish in every system's sum; the
    diagonal system beside them is solved as if alone (its two eigenvalues take
    one or two iterations), to the rounding of its sums."""
    print("breakdown", cells, flush=True)
    skew = np.tile([[0.0, 1.0], [-1.0, 0.0]], (cells, 1, 1))
    fine = np.tile([[2.0, 0.0], [0.0, 3.0]], (cells, 1, 1))
    none, no = np.zeros((0, 2, 2)), np.zeros(0, np.int32)
    b = np.concatenate([np.tile([1.0, 0.0], (cells, 1)), np.tile([2.0, 3.0], (cells, 1)), np.tile([1.0, 0.0], (cells, 1))])
    with P.System(3 * cells, 2, no, no, np.concatenate([skew, fine, skew]), none, none,
                  cell_off=[0, cells, 2 * cells, 3 * cells], face_off=[0] * 4) as s:
        s.setup(precond=P.PREC_NONE, tol=1e-12)
        bd = torch.tensor(b, device="cuda").reshape(-1)
        x = torch.zeros_like(bd)
        st = (P.Stats * 3)()
        rc = P.lib().cbs_solve_batch(s.h, bd.data_ptr(), x.data_ptr(), st)
    x = x.reshape(-1, 2).cpu().numpy()
    assert rc == P.ERR_BREAKDOWN and [q.status for q in st] == [P.ERR_BREAKDOWN, P.OK, P.ERR_BREAKDOWN]
    # two attempts each, both broken in their first iteration; x is the guess
    assert st[0].iterations == st[2].iterations == 2
    assert (x[:cells] == 0.0).all() and (x[2 * cells:] == 0.0).all()
    assert np.abs(x[cells:2 * cells] - 1.0).max() <= 1e-11


@pytest.mark.parametrize("solver", [P.SOLVER_GMRES, P.SOLVER_FGMRES])
def test_gmres_systems_that_finish_in_different_steps(solver):
    """A system of one step, others of many, several work items each."""
    systems = [jacobian_box(*sh, n=5, seed=170 + k, vdt=v) for k, (sh, v) in
               enumerate([((12, 11, 10), 1e9), ((13, 12, 11), 0.1), ((9, 9, 9), 10.0), ((14, 13, 12), 1e3)])]
    cat = concat_systems(systems)
    with P.System.from_dict(cat) as s:
        s.setup(precond=P.PREC_BJACOBI, solver=solver, restart=12, tol=1e-10)
        x, st = s.solve_batch(cat["b"])
    x = x.cpu().numpy()
    its = [q["iterations"] for q in st]
    assert len(set(its)) > 2, its
    for k, sk in enumerate(systems):
        assert st[k]["status"] == P.OK
        assert O.relres(O.from_system(sk), sk["b"], x[cat["cell_off"][k]:cat["cell_off"][k + 1]]) <= 1.01e-10
