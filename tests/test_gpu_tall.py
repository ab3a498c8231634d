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


# n around the 128- and 256-row runs, pairs around the groups of 8 and the four segments of
# the solve, k past the stored inverse's 256, every column count of the few-column path
FEW = [(1, 1, 1), (5, 5, 2), (17, 5, 7), (11, 31, 8), (29, 3, 9), (43, 16, 33), (61, 28, 64), (37, 37, 65), (53, 41, 129),
       (43, 61, 257)]


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("nx,nz,k", FEW)
def test_few_columns(storage, nx, nz, k):
    """One to five columns: the streaming passes (up to four) and the tiles beside them, the
    allocation-free form, and a batch of them against the per-problem results."""
    import ctypes

    import paper_2009_12663_amd as P
    precond = (nx + nz) % 2 == 0
    prob, S, Y, h0 = make_pairs("secant", nx, nz, k, seed=nz + 3 * k, precond=precond)
    n = prob.n
    h0g = None if h0 is None else gpu_input(h0, storage)
    B = P.BfgsBatch([n, n], [k, k], [h0g, h0g], storage)
    Sg, Yg = gpu_input(S, storage), gpu_input(Y, storage)
    assert B.push_pairs([Sg, Sg], [Yg, Yg]) == 0
    H = B.problems[0]
    h = oracle_h0(storage, S, Y, h0)
    print(f"\n[few {storage}] n={n} k={k} diagonal={precond}", flush=True)
    for c in range(1, min(5, n) + 1):
        V = gpu_input(wq.normal_block(n, c, seed=c), storage)
        for diff in (False, True):
            out = H.apply_Hdiff(V) if diff else H.apply_Hinv(V)
            want = recursion.apply_hk(h, oracle_input(S, storage), oracle_input(Y, storage),
                                      oracle_input(V.double().cpu(), storage), subtract_b0=diff)
            err = col_max_rel(out.double().cpu().numpy(), want)
            print(f"  c={c} diff={diff} elementwise {err:.2e}", flush=True)
            assert err <= TOL[storage]
        ref = H.apply_Hinv(V)
        fixed = torch.empty_like(ref)
        assert H.L.bfgs_apply_Hinv_noalloc(H.h, ctypes.c_void_p(V.data_ptr()), c, ctypes.c_void_p(fixed.data_ptr())) == 0
        both = B.apply_Hinv([V, V])
        torch.cuda.synchronize()
        assert torch.equal(fixed, ref) and torch.equal(both[0], ref) and torch.equal(both[1], ref)
    assert H.get_status() == 0
    B.close()
