"""The layer kernels of the warm-start network at the edges of their tiles:
fields smaller than a tile, one point or one row past it, partial strips and
runs along z, in 2D and 3D, forward and backward, against the FP64 reference.

Tolerances as in test_gpu_cnn.py: rounding at the same places, so FP32
accumulation order flips an occasional bfloat16 rounding: 3e-3 relative L2 on
the output and the loss, 2e-2 on a layer's weight gradient.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import rel_l2, to_dev
from oracle import cnn
from paper_1707_09177_amd import gdecon, synth

pytestmark = pytest.mark.gpu

# conv tiles are 16 x 32, end-layer strips 64 wide and 16 high, weight-gradient
# units 32 or 16 wide and 8 rows high at this size, runs along z 16 planes
SHAPES = [(1, 1), (2, 3), (7, 31), (16, 32), (17, 33), (15, 65), (33, 16), (70, 50),
          (1, 1, 1), (2, 3, 5), (17, 4, 33), (18, 17, 16), (33, 5, 7), (3, 33, 65)]


def inputs(shape, B):
    nd = len(shape)
    r = np.random.default_rng(sum(shape))
    u = np.stack([oracle.filter(r.standard_normal(shape), nd) for _ in range(B)])
    ub = np.stack([oracle.filter(x, nd) for x in u])
    p = synth.cnn_init_params(3, ndim=nd)
    for _, b in cnn.unpack(p, ndim=nd):
        b[:] = 0.05 * r.standard_normal(b.shape)
    return p, ub.astype(np.float32).astype(np.float64), u.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("shape", SHAPES)
def test_gradients_and_forward(shape):
    nd = len(shape)
    p, ub, u = inputs(shape, 2)
    ws = gdecon.WarmStart(p, ndim=nd, band=None)
    u0 = ws.forward(to_dev(ub, torch.float32)).double().cpu().numpy()
    ref = cnn.forward(p, ub, emulate_bf16=True, ndim=nd)
    s = ref["s"].reshape((-1,) + (1,) * nd)
    # u0 is stored in FP32: its rounding, relative to the correction, is part of the bound
    floor = 1e-7 * np.linalg.norm(u0) / max(np.linalg.norm(s * ref["y"]), 1e-300)
    assert rel_l2((u0 - ub) / s, ref["y"]) <= 3e-3 + 2 * floor
    loss = ws.train_step(to_dev(ub, torch.float32), to_dev(u, torch.float32)).item()
    l_ref, g_ref = cnn.loss_and_grad(p, ub, u, emulate_bf16=True, ndim=nd)
    assert abs(loss - l_ref) <= 3e-3 * l_ref
    g = ws.grad.double().cpu().numpy()
    off = 0
    for li, (W, b) in enumerate(cnn.unpack(p, ndim=nd)):
        n = W.size + b.size
        assert rel_l2(g[off:off + n], g_ref[off:off + n]) <= 2e-2, li
        off += n


# the fused 2D forward marches two rows per step down strips of 54 columns and 256 rows
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("shape", [(1, 54), (2, 55), (3, 1), (6, 108), (255, 53), (256, 20), (257, 54), (258, 109), (515, 7)])
def test_fused_forward_pairs_of_rows(shape, dtype):
    p, ub, _ = inputs(shape, 2)
    got = gdecon.WarmStart(p, band=None).forward(to_dev(ub, dtype)).double().cpu().numpy()
    ref = cnn.forward(p, ub, emulate_bf16=True)
    y = (got - ub) / ref["s"][:, None, None]
    assert rel_l2(y, ref["y"]) <= 3e-3, rel_l2(y, ref["y"])
