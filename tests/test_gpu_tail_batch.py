"""The V-cycle tail of batches whose small systems have 32,768 rows or more
together on the level that their own sizes would let it start at.  Such a level
keeps its rows in window order and is left to the kernels that read it so; the
tail starts below it."""
import numpy as np
import pytest

from workloads import box_faces, concat_systems

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


def _box(shape, n, seed):
    """Blocks w_f (I + 0.2 G_f) off the diagonal, their row sums and I on it."""
    rng = np.random.default_rng(seed)
    la, ua, _ = box_faces(*shape)
    N, F = int(np.prod(shape)), la.size
    off = rng.uniform(0.2, 1.0, F)[:, None, None] * (np.eye(n) + 0.2 * rng.standard_normal((F, n, n)))
    diag = np.tile(np.eye(n), (N, 1, 1))
    np.add.at(diag, la, off)
    np.add.at(diag, ua, off)
    return {"N": N, "F": F, "n": n, "lower_addr": la, "upper_addr": ua, "diag": diag, "upper": -off, "lower": -off,
            "b": rng.standard_normal((N, n)), "meta": {}}


# shapes of about 300 and 100 cells: 60 to 80 and 17 to 27 rows on level 1
SHAPES = {1: [(7, 7, 6), (6, 9, 5), (5, 11, 6), (8, 6, 6), (7, 7, 5)], 2: [(4, 5, 5), (3, 6, 5), (4, 4, 6), (9, 3, 3), (5, 5, 4)]}


@pytest.mark.parametrize("n,count", [(1, 561), (2, 1801)])
@pytest.mark.parametrize("precision", [P.PRECISION_FP64, P.PRECISION_MIXED])
def test_large_first_level_of_small_systems(n, count, precision):
    """Against the same cycle step by step: bars of the cycles elsewhere, 1e-11
    (FP32 levels: 1e-5); the solves take the same iterations give or take one."""
    print("tail batch", n, count, precision, flush=True)
    kinds = [_box(sh, n, 200 + k) for k, sh in enumerate(SHAPES[n])]
    s = concat_systems([kinds[i % len(kinds)] for i in range(count)])
    f = np.random.default_rng(201).standard_normal((s["N"], n))
    z, its = {}, {}
    with P.System.from_dict(s) as sysm:
        for tail in (-1, 0):
            sysm.setup(precond=P.PREC_AMG, precision=precision, tail_rows=tail)
            rows = sysm.get_level(1)["N"]
            per = rows / count
            # the case: window-ordered by its total, small by its systems, operators within their limit
            assert rows >= 32768 and rows % 64 and per < 100 and count * per * n * (np.ceil(per * n / 16) * 16) * 8 < 32 << 20
            z[tail] = [sysm.apply_precond(f, transpose=t).cpu().numpy() for t in (False, True)]
            sols = sysm.solve_batch(s["b"])
            its[tail] = np.array([st["iterations"] for st in sols[1]])
            assert all(st["status"] == P.OK for st in sols[1])
    for a, b in zip(z[0], z[-1]):
        assert np.abs(a - b).max() <= (1e-5 if precision == P.PRECISION_MIXED else 1e-11) * np.abs(b).max()
    assert np.abs(its[0] - its[-1]).max() <= 1
