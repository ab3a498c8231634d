"""The bfloat16 pass 2 where a workgroup walks several row blocks: every form of its loop
(columns held by one wave or shared by two; pairs that leave the last group of chunks
whole or cut short), n no multiple of a block, odd or a multiple of 4 (the vector stores).

Tolerance: that of the path's other shapes, float32 accumulation with the small operand
split into two bfloat16 halves (2^-17 of it); 2e-5 of a column's largest entry, 3e-4 on
the difference form, which is a tenth of it or less."""
import pytest
import torch

from workloads import quadratic as wq
from tests.helpers import col_max_rel, gpu_input, make_pairs
from tests.test_gpu_mfma import DIFF_ELEM, ELEM, build, oracle

pytestmark = pytest.mark.gpu

# nx, nz (n = 3 nx nz), k, c, diagonal B_0: blocks of 256 rows, 8 x 64 of them at once up to
# 128 columns and 8 x 32 beyond
SHAPES = [(271, 259, 5, 20, True), (269, 260, 17, 64, False), (271, 259, 40, 96, True), (271, 260, 63, 128, False),
          (269, 259, 33, 150, True), (149, 151, 47, 190, False), (148, 152, 100, 220, True), (149, 153, 9, 256, True)]


@pytest.mark.parametrize("nx,nz,k,c,diag", SHAPES)
def test_row_blocks_in_turn(nx, nz, k, c, diag):
    prob, S, Y, h0 = make_pairs("secant", nx, nz, k, seed=k + c, precond=diag)
    print(f"\n[mfma blocks] n={prob.n} k={k} c={c} diagonal={diag}", flush=True)
    H = build(S, Y, h0)
    V = wq.normal_block(prob.n, c, seed=c + 1)
    Vg = gpu_input(V, "bf16")
    got = {d: (H.apply_Hdiff(Vg) if d else H.apply_Hinv(Vg)) for d in (False, True)}
    torch.cuda.synchronize()
    for diff, tol in ((False, ELEM), (True, DIFF_ELEM)):
        want, _, _ = oracle(S, Y, V, h0, diff)
        err = col_max_rel(got[diff].double().cpu().numpy(), want)
        print(f"  diff={diff} elementwise {err:.2e}", flush=True)
        assert err <= tol
    assert H.get_status() == 0
    H.close()
