"""The float64 and float32 rSVD at block widths around its tiles: 16-column blocks in tiles
of up to seven for the products with Q, quads of roots in the merges of the small
eigenproblem, panels of 32 in the LU, odd n.

What is compared does not depend on the condition of the c x c block Q^T X: the posterior
diagonal (the variance terms of a converged sketch are those of B_k - B_0) and the
orthonormality of U = Q M.  Sigma itself does depend on it: rounding the inputs of the
float64 oracle once moves it by up to 3e-9 at these shapes (condition 1e4 at c = 33,
n = 2583).  Tolerance: the storage's rounding (2^-53, 2^-24) times 1e4; of the
orthonormality, the rounding over 200 terms."""
import pytest

from tests.helpers import make_pairs
from tests.test_gpu_rsvd import run_case

pytestmark = pytest.mark.gpu
TOL = {"f64": 1e-11, "f32": 6e-4}
ORTH = {"f64": 1e-12, "f32": 1e-5}

# nx, nz (n = 3 nx nz), c = rank + p
WIDTHS = [(3, 5, 1), (5, 5, 3), (5, 13, 4), (13, 5, 15), (7, 13, 16), (9, 19, 17), (43, 3, 31), (21, 41, 33), (13, 25, 48),
          (33, 31, 49), (43, 29, 65), (35, 37, 81), (41, 35, 97), (31, 67, 113), (53, 39, 129), (45, 51, 161)]


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("nx,nz,c", WIDTHS)
def test_block_widths(storage, nx, nz, c):
    k = max(1, (c - 1) // 2)
    rank = min(c, 2 * k)
    print(f"\n[rsvd width {storage}] n={3 * nx * nz} k={k} rank={rank} c={c}", flush=True)
    prob, S, Y, h0 = make_pairs("secant", nx, nz, k, seed=c, precond=c % 4 == 1)
    r = run_case(storage, S, Y, h0, rank, c - rank, seed=5)
    print(f"  sigma {r['sig']:.2e} rec {r['rec']:.2e} diag_max {r['diag_max']:.2e} orth {r['orth']:.2e}", flush=True)
    assert r["diag_max"] <= TOL[storage] and r["orth"] <= ORTH[storage]
