"""Tuning with a few bfloat16 columns, which stream the pairs and read no row slots, leaves the
choice of slots as it was; tuning with more takes one of the candidates."""
import pytest
import torch

from workloads import quadratic as wq
from tests.helpers import make_pairs
from tests.test_gpu_mfma import build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cols", [1, 2, 4, 5])
def test_few_columns_leave_the_slots(cols):
    prob, S, Y, h0 = make_pairs("secant", 21, 15, 12, seed=4, precond=True)
    H = build(S, Y, h0)
    H.set_tuning(g1_rows=72)     # no candidate
    print(f"\n[autotune few] {cols} columns", flush=True)
    V = wq.normal_block(prob.n, cols, seed=1).to("cuda", torch.bfloat16)
    got = H.autotune(V)["g1_rows"]
    assert got == 72 if cols <= 4 else got in (64, 128, 256, 512)
    assert H.get_status() == 0
    H.close()


@pytest.mark.parametrize("storage", ["f32", "f64"])
def test_other_storage_leaves_the_slots(storage):
    import paper_2009_12663_amd as P
    prob, S, Y, h0 = make_pairs("secant", 21, 15, 12, seed=4, precond=True)
    H = P.Bfgs(prob.n, 12, h0.cuda(), storage)
    for s, y in zip(S, Y):
        H.push_pair(s.cuda(), y.cuda())
    H.set_tuning(g1_rows=72)
    assert H.autotune(wq.normal_block(prob.n, 40, seed=1).cuda())["g1_rows"] == 72
    H.close()
