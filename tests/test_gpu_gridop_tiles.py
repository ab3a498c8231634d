"""The grid operator's smoother at the edges of its 32 x 32 tiles and on both sides of the
half-width its LDS holds (20), against banded matrices in float64.

Tolerance: sums of at most 2 x 43 positive-weight terms in float64 and a coupling of three:
a few dozen roundings of 2^-53 relative to the largest entry, 2e-14."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def band(m, sigma, half):
    t = torch.arange(-half, half + 1, dtype=torch.float64)
    w = torch.exp(-0.5 * (t / sigma) ** 2)
    w = w / w.sum()
    off = torch.arange(m).view(-1, 1) - torch.arange(m).view(1, -1)
    G = torch.zeros(m, m, dtype=torch.float64)
    inside = off.abs() <= half
    G[inside] = w[off[inside] + half]
    return G


@pytest.mark.parametrize("nx,nz,nparam,half", [(1, 1, 1, 0), (31, 33, 3, 1), (32, 32, 2, 20), (33, 31, 3, 20),
                                               (65, 64, 1, 19), (97, 3, 3, 20), (3, 97, 4, 20), (40, 40, 3, 21)])
def test_smoother_tiles(nx, nz, nparam, half):
    import paper_2009_12663_amd as P
    g = torch.Generator().manual_seed(nx * 100 + nz)
    n = nx * nz * nparam
    D = torch.rand(n, generator=g, dtype=torch.float64) + 0.5
    x = torch.randn(2, n, generator=g, dtype=torch.float64)
    sigma, c = 4.0, 0.3
    op = P.GridOp(nx, nz, nparam, D.cuda(), sigma, half, c)
    got = op.apply(x.cuda()).cpu()
    f = band(nz, sigma, half) @ x.view(2, nparam, nz, nx) @ band(nx, sigma, half)
    want = ((1 - c) * f + c * f.sum(1, keepdim=True)).reshape(2, n) + D * x
    err = float((got - want).abs().max() / want.abs().max())
    print(f"\n[smoother] {nx} x {nz} x {nparam} half {half}: {err:.2e}", flush=True)
    assert err <= 2e-14
    op.close()
