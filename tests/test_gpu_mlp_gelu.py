"""The network's GELU by itself: W1 = 0 and b1 = 0 leave h1 = 0, so the second layer's
pre-activations are its biases and the output is the sum of 64 GELUs of one bfloat16 value.

Tolerances.  From -8 down the GELU is below 1e-13 in magnitude, 64 of them below
1e-11.  In between, 64 equal terms are summed exactly but for the float32 rounding of each
sum (2^-24 of it, six roundings), and a GELU is within 2.5e-7 on |x| <= 6 and within a
float32 rounding of x beyond."""
import numpy as np
import pytest
import torch
from math import erfc, sqrt

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


def output(x):
    import paper_2009_12663_amd as P
    p = np.zeros(omlp.NPARAM, dtype=np.float32)
    p[4672:4736] = x      # b2
    p[4736:4800] = 1.0    # w3
    net = P.Mlp(torch.from_numpy(p))
    out = float(net.forward(torch.zeros(1, 8))[0])
    net.close()
    return out


@pytest.mark.parametrize("x", [-8.0, -9.0, -40.0, -1e4])
def test_lower_tail_vanishes(x):
    assert abs(output(x)) <= 1e-11


@pytest.mark.parametrize("x", [-6.5, -6.0, -5.0, -2.0, -0.53125, -1e-3, 0.0, 1e-3, 0.53125, 2.0, 5.0, 6.5, 8.5, 100.0])
def test_value(x):
    x = float(omlp.round_bf16(np.array([x], dtype=np.float32))[0])
    want = 64 * 0.5 * x * erfc(-x / sqrt(2.0))
    assert abs(output(x) - want) <= 64 * 2.5e-7 * max(1.0, abs(x) / 6.0) + 6 * 2.0 ** -24 * abs(want)
