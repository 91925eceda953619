"""Krylov loops on a system with so many work items that their partial sums get a
launch of their own, on both sides of the 2,048 items from which they do.  The
system is many copies of a small one, so its iterates are the small one's: every
inner product is that many times as large."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402

N, n = 2053, 5                                     # a chain of cells; items of 4,095 values


@pytest.mark.parametrize("copies", [816, 819])
@pytest.mark.parametrize("solver", ["bicgstab", "gmres", "fgmres"])
@pytest.mark.parametrize("weak", [False, True])
def test_copies_take_the_small_systems_iterates(copies, solver, weak):
    """Weak couplings: w loses nearly all of its norm to the basis, so GMRES takes
    its second pass.  Sums of 8.4M terms: 8.4e6 eps = 1.9e-9 of their magnitudes
    at most, eps sqrt(8.4e6) = 6e-13 usually; five steps far from converged on
    matrices of condition below 100: bar 1e-9."""
    print("folded sums", copies, solver, weak, flush=True)
    assert (2053 * copies * 5 + 4094) // 4095 == {816: 2046, 819: 2053}[copies]
    g = torch.Generator(device="cuda").manual_seed(240)
    rnd = lambda *a: torch.randn(*a, generator=g, dtype=torch.float64, device="cuda")        # noqa: E731
    c = 1e-3 if weak else 0.3
    up, lo = c * rnd(N - 1, n, n), c * rnd(N - 1, n, n)
    diag = 3.0 * torch.eye(n, dtype=torch.float64, device="cuda") + 0.2 * rnd(N, n, n)
    b = rnd(N, n)
    la = torch.arange(N - 1, dtype=torch.int32, device="cuda")
    kw = dict(precond=P.PREC_BJACOBI, restart=4, tol=1e-15, max_iter=3 if weak else 5,
              solver={"bicgstab": P.SOLVER_BICGSTAB, "gmres": P.SOLVER_GMRES, "fgmres": P.SOLVER_FGMRES}[solver])
    with P.System(N, n, la, la + 1, diag, up, lo) as s:
        s.setup(**kw)
        ref, st0 = s.solve(b)
    shift = (N * torch.arange(copies, dtype=torch.int32, device="cuda"))[:, None]
    many = lambda t: t.repeat(copies, 1, 1)        # noqa: E731
    with P.System(N * copies, n, (la + shift).reshape(-1), (la + 1 + shift).reshape(-1), many(diag), many(up),
                  many(lo)) as s:
        s.setup(**kw)
        x, st = s.solve(b.repeat(copies, 1))
    assert st["iterations"] == st0["iterations"]
    err = (x.reshape(copies, N, n) - ref).abs().max() / ref.abs().max()
    assert err <= 1e-9, float(err)
