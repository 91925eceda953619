"""The aggregates of every level against a plain handshake matching on that
level's matrix, on both sides of the size up to which one workgroup runs a
whole step of the setup: rows, cached and uncached graphs, systems frozen at
different levels, one to three passes."""
import numpy as np
import pytest

import oracle as O
from workloads import concat_systems, jacobian_box, jacobian_graph, pressure_velocity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2403_07882_amd as P  # noqa: E402

ROUNDS = 4


def _best(i, rp, col, w, ok):
    best, bw = -1, 0.0
    for k in range(rp[i], rp[i + 1]):
        j = col[k]
        if j == i or not ok(j) or not w[k] > 0.0:
            continue
        if w[k] > bw or (w[k] == bw and j < best):
            best, bw = j, w[k]
    return best


def _handshake(N, rp, col, w, frozen):
    partner = np.where(frozen, -2, -1)
    for _ in range(ROUNDS):
        cand = [_best(i, rp, col, w, lambda j: partner[j] == -1) if partner[i] == -1 else -1 for i in range(N)]
        for i in range(N):
            if cand[i] >= 0 and cand[cand[i]] == i:
                partner[i] = cand[i]
    rep = np.arange(N)
    for i in range(N):
        if partner[i] >= 0:
            rep[i] = min(i, partner[i])
        elif partner[i] == -1:
            b = _best(i, rp, col, w, lambda j: partner[j] >= 0)
            if b >= 0:
                rep[i] = min(b, partner[b])
    root = rep == np.arange(N)
    return (np.cumsum(root) - root)[rep], int(root.sum())


def _aggregate(A, frozen, passes):
    rp, col, w, N = A.row_ptr, A.col, O.strength(A), A.N
    agg = np.arange(N)
    for p in range(passes):
        a, nc = _handshake(N, rp, col, w, frozen)
        agg = a[agg]
        if p + 1 == passes or nc <= 1:
            break
        fr = np.zeros(nc, bool)
        fr[a] = frozen
        B = O.rap(O.BCSR(N, 1, rp, col, w), a, nc)
        rp, col, w, N, frozen = B.row_ptr, B.col, B.vals.reshape(-1), nc, fr
    return agg, nc


@pytest.mark.parametrize("passes", [1, 2, 3])
@pytest.mark.parametrize("case", ["2047", "2048", "2049", "box", "graph", "batch", "tiny"])
def test_aggregates_are_the_handshake_matching(case, passes):
    print("aggregates", case, passes, flush=True)
    s = {"2047": lambda: jacobian_box(23, 89, 1, n=2, seed=110), "2048": lambda: jacobian_box(16, 128, 1, n=2, seed=111),
         "2049": lambda: jacobian_box(683, 3, 1, n=2, seed=112), "box": lambda: pressure_velocity(14, 13, 12, seed=113),
         "graph": lambda: jacobian_graph(N=1900, n=1, hubs=5, hub_degree=300, seed=114),
         "batch": lambda: concat_systems([jacobian_box(*sh, n=3, seed=115 + k) for k, sh in
                                          enumerate([(2, 2, 2), (9, 8, 7), (3, 1, 1), (12, 12, 12)])]),
         "tiny": lambda: jacobian_box(3, 3, 2, n=5, seed=119)}[case]()
    n, off = s["n"], s.get("cell_off", [0, s["N"]])
    with P.System.from_dict(s) as sysm:
        sysm.setup(precond=P.PREC_AMG, match_passes=passes, renumber=0, coarse_max=16)
        nlev = sysm.info()["levels"]
        assert nlev >= 2
        off = np.asarray(off)
        for l in range(nlev - 1):
            lv = sysm.get_level(l)
            A = O.BCSR(lv["N"], n, *(lv[k].cpu().numpy() for k in ("row_ptr", "col", "vals")))
            size = np.diff(off)
            frozen = np.repeat(size <= 16, size)
            agg, nc = _aggregate(A, frozen, passes)
            got = lv["agg"].cpu().numpy()
            assert np.array_equal(got, agg), (l, int((got != agg).sum()))
            # each system's rows stay together on the next level
            off = np.concatenate([[0], [int(agg[off[k]:off[k + 1]].max()) + 1 for k in range(size.size)]])
