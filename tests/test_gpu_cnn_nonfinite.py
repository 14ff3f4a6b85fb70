"""An activation that overflows bfloat16: one channel of one point is infinite,
and the weight gradients of the other channels stay what they are.

Layer 2's channel 5 is 1e37 times the sum of its input: infinite at the spike
of the field only.  Layer 3 does not use the channel (zero weights), so its
outputs are NaN, stored as 0 by the ReLU, next to the spike (0 times infinity)
and finite elsewhere.  Tolerance on layer 3's gradient as in
test_gpu_cnn_tiles.py: 2e-2 relative L2.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import rel_l2, to_dev
from oracle import cnn
from paper_1707_09177_amd import gdecon, synth

pytestmark = pytest.mark.gpu

CH = 5


def relu(z):
    return cnn.bf16(np.fmax(z, 0.0))  # the number where one argument is NaN


@pytest.mark.parametrize("shape", [(64, 70), (12, 20, 33)], ids=["64x70", "12x20x33"])
def test_gradients_of_finite_channels(shape):
    nd = len(shape)
    r = np.random.default_rng(1)
    p = synth.cnn_init_params(3, ndim=nd)
    W = cnn.unpack(p, ndim=nd)
    mid = len(cnn.taps(nd)) // 2
    W[1][0][CH] = 0.0
    W[1][0][CH, mid] = 1e37
    W[1][1][CH] = 0.0
    W[2][0][:, :, CH] = 0.0
    ub = r.uniform(0.5, 1.0, (1,) + shape)
    spike = tuple(n // 2 for n in shape)
    ub[(0,) + spike] = 300.0
    ub = ub.astype(np.float32).astype(np.float64)
    u = (ub + 0.1 * r.standard_normal(ub.shape)).astype(np.float32).astype(np.float64)

    with np.errstate(all="ignore"):
        P = [(cnn.bf16(w), b.astype(np.float64)) for w, b in W]
        s = float(cnn.rms(ub)[0])
        acts, a = [], (ub / s)[..., None]
        for w, b in P[:-1]:
            a = relu(cnn.conv(a, w, b))
            acts.append(a)
        inf = np.isinf(acts[1])
        assert inf.sum() >= 1 and inf.sum() == inf[..., CH].sum() <= 3 ** nd and not any(np.isinf(x).any() for x in acts[2:])
        y = cnn.g_power(cnn.conv(a, *P[-1])[..., 0], nd, 1)
        g = cnn.g_power(2.0 / ub.size * (y - (u - ub) / s), nd, 1)[..., None]
        for li in range(5, 2, -1):
            g = cnn.bf16(cnn.conv_grad_input(g, P[li][0]) * (acts[li - 1] > 0))
        x = acts[1].copy()
        x[..., CH] = 0.0
        dW, db = cnn.conv_grad_weight(x, g)

    ws = gdecon.WarmStart(p, ndim=nd, band=None)
    ws.train_step(to_dev(ub, torch.float32), to_dev(u, torch.float32))
    grad = cnn.unpack(ws.grad.double().cpu().numpy(), ndim=nd)
    got = np.delete(grad[2][0], CH, axis=2)
    assert np.isfinite(got).all() and np.isfinite(grad[2][1]).all()
    assert rel_l2(got, np.delete(dW, CH, axis=2)) <= 2e-2
    assert rel_l2(grad[2][1], db) <= 2e-2
    for li in (3, 4):
        assert np.isfinite(grad[li][0]).all() and np.isfinite(grad[li][1]).all()
