"""The persistent batch with problems of few columns beside wide ones: streaming items and tile
items from one queue, both forms of the small solve, problems whose partials are one chunk
(which have no sum) and several, in every order.  Results equal the single calls' bit for bit,
eagerly and from a captured graph, three replays with other work between."""
import pytest
import torch

from workloads import quadratic as wq
from tests.helpers import gpu_input, make_pairs

pytestmark = pytest.mark.gpu
# nx, nz (n = 3 nx nz), k
SHAPES = [(7, 5, 3), (41, 35, 24), (31, 67, 130), (5, 5, 8), (53, 39, 128), (43, 29, 65), (21, 41, 129), (13, 25, 16)]


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("cols", [[1] * 8, [4, 1, 2, 3, 4, 2, 1, 4], [1, 37, 2, 60, 3, 5, 4, 130], [5, 6, 1, 16, 17, 90, 9, 33],
                                  [37, 1, 37, 1, 37, 1, 37, 1]])
def test_few_beside_wide(storage, cols):
    import paper_2009_12663_amd as P
    probs = [make_pairs("secant", nx, nz, k, seed=nx + k) for nx, nz, k in SHAPES]
    ns = [p[0].n for p in probs]
    cols = [min(c, n) for c, n in zip(cols, ns)]
    print(f"\n[batch few {storage}] n={ns} cols={cols}", flush=True)
    B = P.BfgsBatch(ns, [s[2] for s in SHAPES], storage=storage)
    assert B.push_pairs([gpu_input(p[1], storage) for p in probs], [gpu_input(p[2], storage) for p in probs]) == 0
    V = [gpu_input(wq.normal_block(n, c, seed=i), storage) for i, (n, c) in enumerate(zip(ns, cols))]
    want = [H.apply_Hinv(v) for H, v in zip(B.problems, V)]
    got = B.apply_Hinv(V)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    out = [torch.empty_like(v) for v in V]
    U, Sig = B._rsvd_bufs([2] * len(ns))
    B.graph_build(V, out, [2] * len(ns), 1, 9, U, Sig)
    for _ in range(3):
        for o in out:
            o.fill_(float("nan"))
        B.graph_launch()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, want))
        again = B.apply_Hinv(V)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(again, want))
    B.autotune(V)
    assert all(torch.equal(a, b) for a, b in zip(B.apply_Hinv(V), want))
    assert all(H.get_status() == 0 for H in B.problems)
    B.close()
