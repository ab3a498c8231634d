"""The network's forward pass on infinite features and on finite ones near float32's largest:
the three-term split of an infinity must not make a NaN of it, nor x + |x| overflow.

With all weights positive an infinite feature gives an infinite output (a negative last layer
the other sign, and 0 and infinity through the exponential); samples beside it in the wave
keep every bit.  At 3e38 the sums stay finite by the choice of weights, within the forward
pass's 1e-6 of the float64 oracle."""
import math

import numpy as np
import pytest
import torch

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


def network(sign):
    rng = np.random.default_rng(5)
    p = np.abs(omlp.init_params(5) + 0.01 * rng.standard_normal(omlp.NPARAM)).astype(np.float32) + np.float32(1e-3)
    p[4736:] *= sign
    return p


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_infinite_feature(sign):
    import paper_2009_12663_amd as P
    net = P.Mlp(torch.from_numpy(network(sign)))
    X = torch.from_numpy(np.random.default_rng(6).standard_normal((70, 8)).astype(np.float32))
    clean, bad = X.clone(), [3, 33, 69]
    for s in bad:
        X[s, s % 8] = math.inf
    out, h0 = net.forward(X).cpu(), net.forward(X, exp_out=True).cpu()
    want, keep = net.forward(clean).cpu(), [s for s in range(70) if s not in bad]
    assert torch.equal(out[keep], want[keep])
    assert (out[bad] == sign * math.inf).all() and (h0[bad] == (math.inf if sign > 0 else 0.0)).all()
    net.close()


@pytest.mark.parametrize("x", [1e30, 1.5e38, 2.5e38, 3.3e38])
def test_near_overflow(x):
    import paper_2009_12663_amd as P
    p = network(1.0)
    p[:512].reshape(64, 8)[:] = [1, 0, 0, 0, 0, 0, 0, 0]     # z1 = x, where 2 x may overflow
    p[576:4672] /= 64 * p[576:4672].max()
    p[4736:4800] /= 64 * p[4736:4800].max()
    net = P.Mlp(torch.from_numpy(p))
    X = np.full((5, 8), x, dtype=np.float32)
    X[1::2, ::2] = 0.0
    got = net.forward(torch.from_numpy(X)).double().cpu().numpy()
    want = omlp.forward(omlp.round_bf16(p), X.astype(np.float64))
    assert np.isfinite(got).all() and np.abs(got - want).max() <= 1e-6 * np.abs(want).max()
    net.close()


@pytest.mark.parametrize("N", [64, 1000, 65536])
def test_large_residuals(N):
    """Residuals of 1e37 whose mean float32 holds and whose sum it does not: with X = 0 every
    sample is the same, so db3 = 2 r and dw3 = 2 r h2 up to rounding."""
    import paper_2009_12663_amd as P
    p = network(1.0)
    net = P.Mlp(torch.from_numpy(p))
    r = 1e37
    grad, _ = net.grad(torch.zeros(N, 8), torch.full((N,), -r))
    grad = grad.double().cpu().numpy()
    w = omlp.round_bf16(p).astype(np.float64)
    gelu = np.vectorize(lambda z: 0.5 * z * math.erfc(-z / math.sqrt(2.0)))
    h2 = gelu(w[576:4672].reshape(64, 64) @ gelu(w[512:576]) + w[4672:4736])
    want = 2 * r * np.append(h2, 1.0)
    assert np.isfinite(grad).all()
    assert np.abs(grad[4736:] - want).max() <= 1e-6 * np.abs(want).max()
    net.close()
