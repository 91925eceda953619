"""Row offsets of a chain of cells on both sides of the lengths at which the
prefix sum takes another workgroup size, a second launch, and a scan of its
totals; and its coefficients where they belong."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402


@pytest.mark.parametrize("N", [2, 2047, 2048, 2049, 8191, 8192, 8193, 10240, 10241, 524289, 4096 * 2048, 4096 * 2048 + 1])
def test_row_offsets_of_a_chain(N):
    print("scan", N, flush=True)
    la = torch.arange(N - 1, dtype=torch.int32)
    one = torch.ones(N, dtype=torch.float64)
    up = 2.0 + torch.arange(N - 1, dtype=torch.float64) / N
    with P.System(N, 1, la, la + 1, one, up, -up) as sysm:
        m = sysm.get_bcsr()
        x = sysm.spmv(one)[:, 0].cpu()
    rp, col, v = (m[k].cpu() for k in ("row_ptr", "col", "vals"))
    deg = torch.full((N,), 3, dtype=torch.int64)
    deg[0] = deg[-1] = 2
    ref = torch.zeros(N + 1, dtype=torch.int64)
    ref[1:] = torch.cumsum(deg, 0)
    assert torch.equal(rp.long(), ref)
    rows = torch.repeat_interleave(torch.arange(N), deg)
    first = torch.arange(int(ref[-1])) - ref[:-1][rows]
    assert torch.equal(col.long(), rows + first - (rows > 0).long())
    y = one.clone()
    y[:-1] += up
    y[1:] -= up
    assert np.abs((x - y).numpy()).max() <= 1e-14
    assert torch.equal(v.reshape(-1)[col == rows], one)
