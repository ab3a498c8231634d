"""The learned-B_0 network at the edges of its tiles: a wave takes 32 samples, a workgroup
128, the grid 32,768 (gradient) or 98,304 (forward) before a wave loops; features at a
float's alignment only; pre-activations far into both tails of the GELU.

Tolerances.  Forward: the output is a sum of 64 GELUs of sums of 64, all in float32, each
rounding within 2^-24 of a term: 1e-6 of the largest output leaves a factor of about ten
over the root-mean-square sum of those roundings.  Gradient: the same chain twice and a
float32 sum over the samples of a wave, 1e-6 in the Frobenius norm for N > 32; a single
wave's samples average nothing: 4e-6."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


def problem(N, scale=1.0):
    rng = np.random.default_rng(N)
    p = (omlp.init_params(3) + 0.05 * rng.standard_normal(omlp.NPARAM)).astype(np.float32)
    X = (scale * rng.standard_normal((N, 8))).astype(np.float32)
    t = (0.3 * X[:, 0] - 0.1 * X[:, 3]).astype(np.float32)
    return p, X, t


@pytest.mark.parametrize("N", [1, 31, 32, 33, 127, 128, 129, 98303, 98305])
def test_forward_tiles(N):
    import paper_2009_12663_amd._lib as L
    p, X, _ = problem(N)
    net = L.Mlp(torch.from_numpy(p))
    got = net.forward(torch.from_numpy(X)).double().cpu().numpy()
    want = omlp.forward(omlp.round_bf16(p), X.astype(np.float64))
    err = np.abs(got - want).max() / np.abs(want).max()
    print(f"\n[mlp forward tiles] N={N} {err:.2e}", flush=True)
    assert err <= 1e-6
    # the same features one float past a 16-byte boundary
    buf = torch.empty(N * 8 + 1, dtype=torch.float32, device="cuda")
    buf[1:] = torch.from_numpy(X).cuda().reshape(-1)
    out = torch.full((N + 1,), 7.0, dtype=torch.float32, device="cuda")
    assert net.L.bfgs_mlp_forward(net.m, ctypes.c_void_p(buf.data_ptr() + 4), N, ctypes.c_void_p(out.data_ptr()), 0) == 0
    torch.cuda.synchronize()
    assert np.array_equal(out[:N].double().cpu().numpy(), got) and float(out[N]) == 7.0
    net.close()


@pytest.mark.parametrize("N", [1, 31, 32, 33, 127, 129, 32767, 32801])
def test_gradient_tiles(N):
    import paper_2009_12663_amd as P
    p, X, t = problem(N)
    net = P.Mlp(torch.from_numpy(p))
    g, loss = net.grad(torch.from_numpy(X), torch.from_numpy(t))
    lw, gw = omlp.loss_and_grad(omlp.round_bf16(p), X.astype(np.float64), t.astype(np.float64))
    err = np.linalg.norm(g.double().cpu().numpy() - gw) / np.linalg.norm(gw)
    print(f"\n[mlp gradient tiles] N={N} {err:.2e}", flush=True)
    assert err <= (1e-6 if N > 32 else 4e-6) and abs(float(loss) - lw) <= 4e-6 * lw
    net.close()


@pytest.mark.parametrize("scale", [10.0, 1e4])
def test_gelu_tails(scale):
    """Pre-activations of +-100 and +-1e5: GELU is x or 0 to float32 rounding, its slope 1 or 0."""
    import paper_2009_12663_amd as P
    p, X, t = problem(500, scale)
    net = P.Mlp(torch.from_numpy(p))
    got = net.forward(torch.from_numpy(X)).double().cpu().numpy()
    want = omlp.forward(omlp.round_bf16(p), X.astype(np.float64))
    g, _ = net.grad(torch.from_numpy(X), torch.from_numpy(t))
    _, gw = omlp.loss_and_grad(omlp.round_bf16(p), X.astype(np.float64), t.astype(np.float64))
    err = np.abs(got - want).max() / np.abs(want).max()
    gerr = np.linalg.norm(g.double().cpu().numpy() - gw) / np.linalg.norm(gw)
    print(f"\n[mlp tails] scale {scale} forward {err:.2e} gradient {gerr:.2e}", flush=True)
    assert err <= 1e-6 and gerr <= 1e-6
    X[7, 2] = np.nan
    bad = net.forward(torch.from_numpy(X)).cpu().numpy()
    assert np.isnan(bad[7]) and np.isfinite(np.delete(bad, 7)).all()
    net.close()
