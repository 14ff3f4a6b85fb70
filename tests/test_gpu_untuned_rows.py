"""The untuned launch of streamed 2D batches of several fields with one value
per lane (odd rows): two tiles per wave where one would give each wave one tile
of fields larger than the caches, else one; the same u either way.

Tolerance: only the order in which inner products are summed differs: FP32 1e-5,
FP64 1e-10 relative L2 after two passes.
"""
import pytest
import torch

from paper_1707_09177_amd import gdecon

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape, solver, dtype, tpw", [
    ((8, 3176, 1073), "sd", torch.float32, 2), ((10, 1851, 3179), "bicgstab", torch.float32, 2),
    ((10, 2730, 1793), "sd", torch.float64, 2),
    ((1, 7139, 4523), "vc", torch.float32, 1),        # one field
    ((2, 4219, 2099), "bicgstab", torch.float32, 1),  # 18 M points
    ((4, 4032, 3308), "cg", torch.float32, 1),        # whole 16-byte lanes
], ids=str)
def test_tiles_per_wave(shape, solver, dtype, tpw):
    ub = gdecon.filter_apply(torch.randn(shape, device="cuda", dtype=dtype))
    d = gdecon.Deconvolver(ub.shape, 2, dtype, solver)
    got = d.solve(ub, 2).u
    launch = gdecon.last_launch()
    out = torch.empty_like(ub)
    tiles = {}
    try:
        for k in (1, 2):
            gdecon.tune_set(solver, ub, out, tiles_per_wave=k)
            d.solve(ub, 2, out=out)
            tiles[k] = gdecon.last_launch()["tiles"]
            assert float((got - out).norm() / got.norm()) <= (1e-5 if dtype == torch.float32 else 1e-10)
    finally:
        gdecon.tune_reset()
    assert launch["tiles"] == tiles[tpw]
    if tpw == 2:
        assert tiles[1] < tiles[2]
