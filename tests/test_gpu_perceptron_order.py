"""The order in which the perceptron's sums are taken is part of its results: q is
compared with 24-bit uniforms for the initial draws, and seeded runs are to
reproduce.  A row's logit is summed by unit position over the chunks of 32 hidden
units, then over the positions as a balanced tree, in FP32; the gradient over
1024 workgroups' rows."""
import hashlib

import numpy as np
import pytest

from oracle import learned as M
from tests.parity import say

pytestmark = pytest.mark.gpu


def _upload(net, params):
    import torch
    net.params.copy_(torch.from_numpy(params))
    net.sync()


def _bits(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).bfloat16().view(torch.int16).cuda()


# Inputs and weights are small integers, so the hidden layer is exact in any
# order; hidden units come in pairs of opposite output weights, so a logit is b2
# plus the rounding of its FP32 sums, a multiple of at least 1/8 that another
# order changes.  Tolerance: q of a logit that is equal, by two exponentials.
@pytest.mark.parametrize("rows,seed", [(1, 1), (33, 2), (257, 3), (4100, 4)])
def test_logits_are_summed_in_the_stated_order(hip, rows, seed):
    import torch
    from paper_2311_02101_amd import learned as Lr
    rng = np.random.default_rng(seed)
    half = M.HIDDEN // 2
    unit = rng.permutation(M.HIDDEN)
    W1, b1, w2 = np.zeros((M.F_IN, M.HIDDEN)), np.zeros(M.HIDDEN), np.zeros(M.HIDDEN)
    w = rng.integers(-100, 101, (M.F_IN, half))
    b = rng.integers(-500, 501, half)
    o = rng.integers(129, 256, half) / 8.0
    for side, sign in ((unit[:half], 1.0), (unit[half:], -1.0)):
        W1[:, side], b1[side], w2[side] = w, b, sign * o
    b2 = 0.25
    x = rng.integers(-100, 101, (rows, M.F_IN)).astype(np.float64)
    net = Lr.MLP(seed=1)
    _upload(net, np.concatenate([W1.ravel(), b1, w2, [b2]]).astype(np.float32))
    h = np.maximum(x @ W1 + b1, 0.0)
    s = np.zeros((rows, 32), dtype=np.float32)
    for j in range(M.HIDDEN // 32):                 # a fused multiply-add each: one rounding
        k = slice(32 * j, 32 * j + 32)
        s = (s.astype(np.float64) + h[:, k] * w2[k]).astype(np.float32)
    while s.shape[1] > 1:
        s = s[:, 0::2] + s[:, 1::2]
    logit = s[:, 0] + np.float32(b2)
    want = M.sigmoid(logit.astype(np.float64))
    if rows > 100:
        exact = np.float64(b2)
        assert np.mean(np.abs(logit - exact) >= 0.125) > 0.5      # the order shows
    say(f"[mlp order] rows={rows}")
    q = net.forward(_bits(x))
    torch.cuda.synchronize()
    assert np.max(np.abs(q.cpu().numpy() - want)) < 1e-6


# q, gradient and loss of fixed inputs: the bits that a seeded run has always had
# (recorded on an MI355X from the kernels that summed rows in the lanes)
GOLDEN = {
    33: ("5a1ee8e6b583e78d", "4a71dfcda3835b63", "aa3c4073cad929fd"),
    3000: ("9c14d6133f34e897", "f8e23dc69250b5cd", "6870f184cebed384"),
    65537: ("39036de6e0f68382", "a4dc44e6e9a24a38", "d1b8e2e1ceba1c1f"),
    140001: ("58b4409c158311c9", "e102fc137499d52e", "b382035be03f7496"),
}


def _digests(rows):
    import torch
    from paper_2311_02101_amd import learned as Lr
    rng = np.random.default_rng(rows)
    x = _bits(rng.integers(0, 40, (rows, M.F_IN)) / 8.0)
    y = torch.from_numpy(rng.integers(0, 33, rows).astype(np.float32) / 32.0).cuda()
    net, _ = Lr.MLP.load()
    q = net.forward(x)
    loss = net.backward(x, y)
    torch.cuda.synchronize()
    return tuple(hashlib.sha256(a.cpu().numpy().tobytes()).hexdigest()[:16] for a in (q, net.grad, loss))


@pytest.mark.parametrize("rows", sorted(GOLDEN))
def test_recorded_bits(hip, rows):
    say(f"[mlp bits] rows={rows}")
    assert _digests(rows) == GOLDEN[rows]
