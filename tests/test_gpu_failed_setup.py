"""A setup that runs out of memory leaves nothing behind that a later call of the
same host thread, on another handle and stream, could take for its own error."""
import ctypes as C
import time

import pytest

from workloads import jacobian_box

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402
from paper_2403_07882_amd import binding as B  # noqa: E402


@pytest.mark.parametrize("shape", [(12, 11, 10), (20, 19, 18)])
def test_calls_after_a_setup_without_memory(shape):
    """Every allocation of the setup is refused in turn, while its stream is busy
    with earlier work, so that the kernels it has enqueued run after it returned."""
    s = jacobian_box(*shape, n=5, seed=250)
    o = jacobian_box(4, 4, 4, n=5, seed=251)
    st, other = torch.cuda.Stream(), torch.cuda.Stream()
    big = torch.zeros(1 << 28, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(other):
        vals = [torch.tensor(o[k], device="cuda") for k in ("diag", "upper", "lower")]
        good = P.System.from_dict(o)
    refused = 1
    while True:
        calls = [0]

        def alloc(ctx, nbytes, stream):
            calls[0] += 1
            if calls[0] == refused:
                return None
            if calls[0] == refused - 1:
                with torch.cuda.stream(st):
                    for _ in range(30):
                        big.mul_(1.0)
            return torch.cuda.caching_allocator_alloc(int(nbytes), None, int(stream or 0))

        hook = P.Allocator(B._ALLOC_FN(alloc), B._FREE_FN(lambda ctx, p, q: torch.cuda.caching_allocator_delete(int(p))),
                           None)
        with torch.cuda.stream(st):
            sysm = P.System.from_dict(s)
        with sysm:
            assert P.lib().cbs_set_allocator(sysm.h, C.byref(hook)) == P.OK
            try:
                sysm.setup(precond=P.PREC_AMG)
                break                                  # as many allocations as it wants
            except P.CbsError as e:
                assert e.code == P.ERR_OOM, refused
            end = time.perf_counter() + 0.03
            with torch.cuda.stream(other):
                while time.perf_counter() < end:
                    good.update_values(*vals)          # raises if it reads another call's word
        if refused % 10 == 0:
            print("refused", refused, flush=True)
        refused += 1
    assert refused > 40
    good.close()


def test_solve_whose_fallback_runs_out_of_memory():
    """The FP64 hierarchy of a mixed solve that did not converge finds no memory:
    the handle has no preconditioner until the next setup, and works after it."""
    s = jacobian_box(12, 11, 10, n=5, seed=252)
    refuse = [False]

    def alloc(ctx, nbytes, stream):
        return None if refuse[0] else torch.cuda.caching_allocator_alloc(int(nbytes), None, int(stream or 0))

    hook = P.Allocator(B._ALLOC_FN(alloc), B._FREE_FN(lambda ctx, p, q: torch.cuda.caching_allocator_delete(int(p))), None)
    with P.System.from_dict(s) as sysm:
        assert P.lib().cbs_set_allocator(sysm.h, C.byref(hook)) == P.OK
        kw = dict(precond=P.PREC_AMG, precision=P.PRECISION_MIXED)
        sysm.setup(**kw)
        sysm.solve(s["b"])
        sysm.setup(max_iter=1, tol=1e-14, reuse_aggregates=1, **kw)
        refuse[0] = True
        with pytest.raises(P.CbsError) as e:
            sysm.solve(s["b"])
        assert e.value.code == P.ERR_OOM
        refuse[0] = False
        for call in (sysm.solve, sysm.apply_precond):
            with pytest.raises(P.CbsError) as e:
                call(s["b"])
            assert e.value.code == P.ERR_STATE
        sysm.setup(**kw)
        assert sysm.solve(s["b"])[1]["status"] == P.OK
