"""cbs_spmv after its first product only launches: nothing is allocated by the
later ones, and products can be captured into a graph after it, whatever number
of them came before."""
import ctypes as C

import numpy as np
import pytest

import oracle as O
from workloads import jacobian_box

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402
from paper_2403_07882_amd import binding as B  # noqa: E402

SHAPES = {"split rows": (9, 8, 7), "whole rows": (37, 31, 29)}


def _mul(sysm, x, y, tr):
    assert P.lib().cbs_spmv(sysm.h, x.data_ptr(), y.data_ptr(), 1 if tr else 0) == P.OK, P.lib().cbs_last_error()


@pytest.mark.parametrize("n", [4, 5])
@pytest.mark.parametrize("shape", SHAPES)
def test_only_the_first_product_allocates(n, shape):
    s = jacobian_box(*SHAPES[shape], n=n, seed=230)
    x = torch.tensor(s["b"], device="cuda")
    y = torch.empty_like(x)
    count = [0]

    def alloc(ctx, nbytes, stream):
        count[0] += 1
        return torch.cuda.caching_allocator_alloc(int(nbytes), None, int(stream or 0))

    hook = P.Allocator(B._ALLOC_FN(alloc), B._FREE_FN(lambda ctx, p, st: torch.cuda.caching_allocator_delete(int(p))), None)
    with P.System.from_dict(s) as sysm:
        assert P.lib().cbs_set_allocator(sysm.h, C.byref(hook)) == P.OK
        for fresh in range(2):
            for tr in (False, True):
                _mul(sysm, x, y, tr)
                was = count[0]
                for _ in range(20):
                    _mul(sysm, x, y, tr)
                assert count[0] == was, (fresh, tr)
            sysm.update_values(s["diag"], s["upper"], s["lower"])


@pytest.mark.parametrize("n", [4, 5])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("before", [0, 1, 12, 20])
def test_products_captured_after_any_number(n, shape, before):
    """Twenty captured products with eager ones between the replays, and eager
    ones after the capture: all have the bits of the first."""
    print("capture", n, shape, before, flush=True)
    s = jacobian_box(*SHAPES[shape], n=n, seed=231)
    A = O.from_system(s)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        x = torch.tensor(s["b"], device="cuda")
        sysm = P.System.from_dict(s)
    with sysm:
        for tr in (False, True):
            ys = torch.zeros((20,) + tuple(x.shape), dtype=x.dtype, device="cuda")
            y = torch.zeros_like(x)
            torch.cuda.synchronize()
            for _ in range(before):
                _mul(sysm, x, y, tr)
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=st):
                for k in range(20):
                    _mul(sysm, x, ys[k], tr)
            for k in range(3):
                _mul(sysm, x, y, tr)                # eager, before the first replay too
                torch.cuda.synchronize()
                ys.zero_()
                torch.cuda.synchronize()
                with torch.cuda.stream(st):
                    g.replay()
                torch.cuda.synchronize()
                assert all(torch.equal(q, y) for q in ys), (tr, k)
            ref = O.spmv_t(A, s["b"]) if tr else O.spmv(A, s["b"])
            assert np.abs(y.cpu().numpy() - ref).max() <= 1e-14 * np.abs(A.vals).max() * np.abs(s["b"]).max() * 8 * n
            for _ in range(20):
                _mul(sysm, x, y, tr)
            torch.cuda.synchronize()
            assert torch.equal(ys[0], y), tr
            del g
