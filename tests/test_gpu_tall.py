"""The float64 matrix-core apply at the edges of its tiles: 16-row steps and 128-row blocks,
16-column blocks in tiles of up to seven, pairs that are no multiple of 4 or 16, odd n
(columns at any 4- or 8-byte alignment), and the persistent batch's fixed tiles against
the per-problem ones, bit for bit.

Tolerance: float64 sums of n + 4k terms, whose rounding is within a few hundred units of
2^-53 of the largest term of each column (1e-12 elementwise leaves a factor of ten);
float32 results are those sums rounded once, 2^-24, to which the inputs' exactness adds
nothing (1.2e-7 elementwise: one rounding and a half)."""
import numpy as np
import pytest
import torch

from oracle import recursion
from workloads import quadratic as wq
from tests.helpers import col_max_rel, gamma_of, gpu_input, h0_storage, make_pairs, oracle_input

pytestmark = pytest.mark.gpu
TOL = {"f64": 1e-12, "f32": 1.2e-7}

# nx, nz (n = 3 nx nz), k, c: n around the row steps and blocks, c around every tile width
SHAPES = [(3, 5, 1, 1), (5, 5, 2, 2), (11, 5, 3, 5), (7, 13, 4, 16), (9, 19, 7, 17), (43, 3, 8, 33), (21, 41, 9, 48),
          (13, 25, 16, 65), (33, 31, 17, 81), (43, 29, 33, 97), (35, 37, 40, 112), (41, 35, 63, 113), (31, 67, 64, 129),
          (53, 39, 65, 225), (45, 51, 100, 256)]


def oracle_h0(storage, S, Y, h0):
    if h0 is not None:
        return h0_storage(h0, storage)
    g = gamma_of(oracle_input(S, storage), oracle_input(Y, storage))
    return np.full(S.shape[1], g if storage == "f64" else float(np.float32(g)))


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("nx,nz,k,c", SHAPES)
def test_tile_edges(storage, nx, nz, k, c):
    import paper_2009_12663_amd as P
    precond = (nx + k) % 2 == 0
    prob, S, Y, h0 = make_pairs("secant", nx, nz, k, seed=nx + 7 * k, precond=precond)
    n = prob.n
    c = min(c, n)
    print(f"\n[tall {storage}] n={n} k={k} c={c} diagonal={precond}", flush=True)
    Sg, Yg = gpu_input(S, storage), gpu_input(Y, storage)
    V = gpu_input(wq.normal_block(n, c, seed=c), storage)
    B = P.BfgsBatch([n], [k], [None if h0 is None else gpu_input(h0, storage)], storage)
    assert B.push_pairs([Sg], [Yg]) == 0
    H = B.problems[0]
    got = {d: (H.apply_Hdiff(V) if d else H.apply_Hinv(V)) for d in (False, True)}
    batch = B.apply_Hinv([V])[0]
    torch.cuda.synchronize()
    assert torch.equal(batch, got[False])
    h = oracle_h0(storage, S, Y, h0)
    for diff, out in got.items():
        want = recursion.apply_hk(h, oracle_input(S, storage), oracle_input(Y, storage),
                                  oracle_input(V.double().cpu(), storage), subtract_b0=diff)
        err = col_max_rel(out.double().cpu().numpy(), want)
        print(f"  diff={diff} elementwise {err:.2e}", flush=True)
        assert err <= TOL[storage]
    assert H.get_status() == 0
    B.close()
