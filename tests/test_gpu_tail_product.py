"""The tail operator's product on both sides of the 512 unknowns up to which its
values are loaded ahead, against the same levels run step by step."""
import numpy as np
import pytest

from workloads import jacobian_box

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


@pytest.mark.parametrize("n,rows", [(4, 127), (4, 128), (4, 129), (2, 255), (2, 256), (5, 102), (5, 103), (3, 170), (3, 171)])
@pytest.mark.parametrize("precision", [P.PRECISION_FP64, P.PRECISION_MIXED])
def test_product_is_the_steps(n, rows, precision):
    """Level 1 of a chain of cells, of a length that leaves it that many rows.
    Bars of the cycles elsewhere: 1e-11, with FP32 levels 1e-5."""
    print("tail product", n, rows, precision, flush=True)
    kw = dict(precond=P.PREC_AMG, precision=precision, match_passes=1, coarse_max=8)
    for N in range(2 * rows, 3 * rows + 4):
        s = jacobian_box(N, 1, 1, n=n, seed=190 + n)
        with P.System.from_dict(s) as sysm:
            sysm.setup(**kw)
            if sysm.get_level(1)["N"] != rows:
                continue
            f = np.random.default_rng(191).standard_normal((N, n))
            z = {}
            for tail in (0, -1):
                sysm.setup(tail_rows=tail, **kw)
                z[tail] = [sysm.apply_precond(f, transpose=t).cpu().numpy() for t in (False, True)]
        for a, b in zip(z[0], z[-1]):
            assert np.abs(a - b).max() <= (1e-5 if precision == P.PRECISION_MIXED else 1e-11) * np.abs(b).max()
        return
    pytest.fail("no chain with that many rows on level 1")
