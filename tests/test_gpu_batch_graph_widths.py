"""A captured batch whose rSVD has more columns than its apply, fewer, and as many: the
workspace of the partial sums then grows while the graph is built, and the graph has to use
the one that is there when it is replayed.

Replays are compared bit for bit with the eager calls, three of them, with a poisoned output
and other allocations between, so that memory given back would not hold what it held."""
import pytest
import torch

from workloads import quadratic as wq
from tests.helpers import gpu_input, make_pairs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("cols,rank,oversample", [(5, 24, 40), (64, 24, 4), (28, 24, 4)])
def test_graph_after_wider_rsvd(storage, cols, rank, oversample):
    import paper_2009_12663_amd as P
    shapes = [(41, 35, 24), (31, 67, 33), (21, 41, 40)]
    probs = [make_pairs("secant", nx, nz, k, seed=nx) for nx, nz, k in shapes]
    ns = [p[0].n for p in probs]
    print(f"\n[graph widths {storage}] n={ns} cols={cols} rsvd={rank}+{oversample}", flush=True)
    B = P.BfgsBatch(ns, [s[2] for s in shapes], storage=storage)
    assert B.push_pairs([gpu_input(p[1], storage) for p in probs], [gpu_input(p[2], storage) for p in probs]) == 0
    V = [gpu_input(wq.normal_block(n, cols, seed=i), storage) for i, n in enumerate(ns)]
    out = [torch.empty_like(v) for v in V]
    U, Sig = B._rsvd_bufs([rank] * len(ns))
    B.graph_build(V, out, [rank] * len(ns), oversample, 9, U, Sig)
    want = [o.clone() for o in B.apply_Hinv(V)]
    wantU, wantS = B.rsvd([rank] * len(ns), oversample, 9)
    torch.cuda.synchronize()
    for _ in range(3):
        for x in out + U + Sig:
            x.fill_(float("nan"))
        B.graph_launch()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out + U + Sig, want + list(wantU) + list(wantS)))
        junk = [torch.randn(1 << 22, device="cuda") for _ in range(4)]
        del junk
    B.close()
