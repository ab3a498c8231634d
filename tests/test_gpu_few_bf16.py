"""B_k V of one to five columns from bfloat16 pairs, on both sides of the rule that sends a
few columns through the streaming passes: up to 128 pairs, or two columns of at least
65,536 rows; and the allocation-free form against the ordinary one.

Tolerance: the streaming passes round float64 sums once to float32 (1.2e-7 of a column's
largest entry, one rounding and a half); the matrix-core path as in its own tests (2e-5)."""
import ctypes

import pytest
import torch

from workloads import quadratic as wq
from tests.helpers import col_max_rel, gpu_input, make_pairs
from tests.test_gpu_mfma import ELEM, build, oracle

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (5, 5, 2), (17, 5, 7), (43, 16, 33), (61, 28, 128), (61, 29, 129), (151, 145, 129), (149, 147, 150)]


@pytest.mark.parametrize("nx,nz,k", SHAPES)
def test_few_columns_bf16(nx, nz, k):
    prob, S, Y, h0 = make_pairs("secant", nx, nz, k, seed=nz + 3 * k, precond=(nx + nz) % 2 == 0)
    n = prob.n
    H = build(S, Y, h0)
    print(f"\n[few bf16] n={n} k={k}", flush=True)
    for c in range(1, min(5, n) + 1):
        V = wq.normal_block(n, c, seed=c)
        Vg = gpu_input(V, "bf16")
        stored = Vg.to(torch.bfloat16)   # what the C entry is handed
        out = H.apply_Hinv(Vg)
        fixed = torch.empty_like(out)
        args = (ctypes.c_void_p(stored.data_ptr()), c, ctypes.c_void_p(fixed.data_ptr()))
        assert H.L.bfgs_apply_Hinv_noalloc(H.h, *args) == 0
        torch.cuda.synchronize()
        want, _, _ = oracle(S, Y, V, h0)
        streamed = c <= 4 and (k <= 128 or (c <= 2 and n >= 65536))
        for name, x in (("apply", out), ("noalloc", fixed)):
            err = col_max_rel(x.double().cpu().numpy(), want)
            print(f"  c={c} {name} elementwise {err:.2e}", flush=True)
            assert err <= (1.2e-7 if streamed else ELEM)
    assert H.get_status() == 0
    H.close()
