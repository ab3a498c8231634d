"""The inner solve's chains at the edges of their batches of 16 pairs, waves of 64 rows and
four segments, after pairs have been dropped and others refused (the stored inverse is read
as a full matrix, so what lies outside its triangle has to stay zero), against the float64
oracle on the pairs that are held.

Tolerance: as for the tiles' edges, 1e-12 of a column's largest entry in float64."""
import pytest
import torch

from oracle import recursion
from workloads import quadratic as wq
from tests.helpers import col_max_rel, make_pairs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 120, 127, 128, 129, 193, 255, 256])
def test_chain_edges(k):
    import paper_2009_12663_amd as P
    drop, extra = 3, 2
    prob, S, Y, h0 = make_pairs("secant", 41, 35, k + drop + extra, seed=k, precond=True)
    H = P.Bfgs(prob.n, k + drop, h0.cuda(), "f64")
    for i in range(k + drop):
        H.push_pair(S[i].cuda(), Y[i].cuda())
    for _ in range(drop):
        H.pop_oldest()
    bad = S[k + drop].cuda()
    for y in (-bad, torch.full_like(bad, float("nan"))):     # no curvature; not finite
        with pytest.raises(P._lib.BfgsError):
            H.push_pair(bad, y)
    assert H.k == k
    print(f"\n[solve chains] k={k}", flush=True)
    for c in (1, 4, 5, 37):
        V = wq.normal_block(prob.n, c, seed=c)
        want = recursion.apply_hk(h0.numpy(), S[drop:drop + k].numpy(), Y[drop:drop + k].numpy(), V.numpy())
        err = col_max_rel(H.apply_Hinv(V.cuda()).cpu().numpy(), want)
        print(f"  c={c} {err:.2e}", flush=True)
        assert err <= 1e-12
    assert H.get_status() == 0
    H.close()
