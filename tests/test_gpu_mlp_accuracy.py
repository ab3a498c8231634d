"""Rounding of the network's gradient: what is common to all samples is not averaged away, and
a small batch averages nothing.

Copies of one sample: up to 128 samples a wave takes one each, its partial is that sample's
gradient, and the sum of N = 2^p equal partials in float64 and the factor 2 / N are exact, so
the gradient equals the single sample's bit for bit.

A common factor: with none that is rounded to float32, an entry of the gradient is a sum of
8,000 terms whose float32 roundings are independent, rounded once to float32 (2^-24 at most,
1.7e-8 rms), beside the two constants of the GELU's slope (7e-9): 4.5e-8 in the Frobenius
norm leaves a factor of two over their root sum of squares with the sums of 32 (1.2e-8).  The
factor 2 / 8,000 alone would be off by 4.75e-8."""
import numpy as np
import pytest
import torch

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


def params(seed):
    rng = np.random.default_rng(seed)
    return (omlp.init_params(seed) + 0.05 * rng.standard_normal(omlp.NPARAM)).astype(np.float32)


@pytest.mark.parametrize("N", [2, 16, 64, 128])
def test_copies_of_one_sample(N):
    import paper_2009_12663_amd as P
    rng = np.random.default_rng(N)
    net = P.Mlp(torch.from_numpy(params(N)))
    x = torch.from_numpy(rng.standard_normal((1, 8)).astype(np.float32))
    t = torch.tensor([0.3])
    one, loss1 = net.grad(x, t)
    many, loss = net.grad(x.repeat(N, 1), t.repeat(N))
    assert torch.equal(one, many) and torch.equal(loss1, loss)
    net.close()


def test_no_common_error():
    import paper_2009_12663_amd as P
    N, errs = 8000, []
    for seed in range(8):
        rng = np.random.default_rng(seed)
        p = params(seed)
        X = rng.standard_normal((N, 8)).astype(np.float32)
        t = (0.3 * X[:, 0] - 0.1 * X[:, 3] + 0.1 * rng.standard_normal(N)).astype(np.float32)
        net = P.Mlp(torch.from_numpy(p))
        g, _ = net.grad(torch.from_numpy(X), torch.from_numpy(t))
        _, want = omlp.loss_and_grad(omlp.round_bf16(p), X.astype(np.float64), t.astype(np.float64))
        errs.append(np.linalg.norm(g.double().cpu().numpy() - want) / np.linalg.norm(want))
        net.close()
    print(f"\n[mlp common error] {np.median(errs):.2e}", flush=True)
    assert np.median(errs) <= 4.5e-8
