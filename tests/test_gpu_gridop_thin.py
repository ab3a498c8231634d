"""The grid operator's smoother on both sides of the rule that chooses between its 32 x 32
tiles and the two stencils (how many tiles, how full they are, how many taps), on thin grids, and on a row of 2^27 points, whose tiles would not fit a launch.

Tolerance: as for the tiles' own edges, sums of at most 2 x 41 positive-weight terms in
float64 and a coupling of up to three: a few dozen roundings of 2^-53 relative to the largest
entry, 2e-14."""
import pytest
import torch

pytestmark = pytest.mark.gpu
SIGMA, C = 4.0, 0.3


def weights(half):
    t = torch.arange(-half, half + 1, dtype=torch.float64)
    w = torch.exp(-0.5 * (t / SIGMA) ** 2)
    return w / w.sum()


def along(f, half, dim):
    """The truncated smoother along one dimension, zero outside, taps added one by one."""
    out, m = torch.zeros_like(f), f.shape[dim]
    for t, w in zip(range(-half, half + 1), weights(half).tolist()):
        k = m - abs(t)
        if k > 0:
            out.narrow(dim, max(0, -t), k).add_(f.narrow(dim, max(0, t), k), alpha=w)
    return out


@pytest.mark.parametrize("nx,nz,nparam,half", [(8192, 1, 1, 20), (8193, 1, 1, 20), (1, 8225, 1, 6), (16384, 3, 1, 5),
                                               (16385, 3, 1, 5), (16416, 16, 1, 2), (16416, 15, 1, 2), (16416, 14, 1, 4),
                                               (16416, 12, 1, 5), (16416, 11, 1, 20), (12288, 2, 1, 10),
                                               (12289, 2, 1, 10), (16416, 28, 1, 1), (16416, 27, 1, 0), (5, 7, 600, 20), (50000, 1, 3, 20)])
def test_rule_edges(nx, nz, nparam, half):
    import paper_2009_12663_amd as P
    g = torch.Generator().manual_seed(nx + 100 * nz)
    n = nx * nz * nparam
    D = torch.rand(n, generator=g, dtype=torch.float64) + 0.5
    x = torch.randn(n, generator=g, dtype=torch.float64)
    op = P.GridOp(nx, nz, nparam, D.cuda(), SIGMA, half, C)
    got = op.apply(x.cuda()).cpu()
    f = along(along(x.view(nparam, nz, nx), half, 2), half, 1)
    want = ((1 - C) * f + C * f.sum(0, keepdim=True)).reshape(n) + D * x
    err = float((got - want).abs().max() / want.abs().max())
    print(f"\n[smoother rule] {nx} x {nz} x {nparam} half {half}: {err:.2e}", flush=True)
    assert err <= 2e-14
    op.close()


def test_longest_row():
    import paper_2009_12663_amd as P
    nx, half = (1 << 27) + 5, 3
    print(f"\n[smoother rule] {nx} x 1 x 1 half {half}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    D = torch.rand(nx, generator=g, dtype=torch.float64, device="cuda") + 0.5
    x = torch.randn(nx, generator=g, dtype=torch.float64, device="cuda")
    op = P.GridOp(nx, 1, 1, D, SIGMA, half, C)
    got = op.apply(x)
    want = along(x, half, 0).mul_(weights(half)[half].item()).addcmul_(D, x)
    assert float((got - want).abs().max() / want.abs().max()) <= 2e-14
    op.close()
