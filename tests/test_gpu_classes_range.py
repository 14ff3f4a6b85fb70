"""The differential-filter solve on wavenumber classes at the ends of the FP64
range and on fields that are not finite: what the general solver gives there."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import to_dev
from paper_1707_09177_amd import gdecon

pytestmark = pytest.mark.gpu

SHAPES = [(32, 32), (32, 64), (16, 16, 16)]   # square, signs only, cube


def base(shape):
    u = np.random.default_rng(2).standard_normal((1,) + shape)
    return to_dev(oracle.germano_filter(u, len(shape), 0.5), torch.float64)


def solve(solver, ub, N, **kw):
    u, info, _ = gdecon.deconvolve_germano(solver, ub, N, 0.5, ndim=ub.dim() - 1, **kw)
    return u, info[0]


@pytest.mark.parametrize("solver", ["vc", "sd", "cg", "bicgstab"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_not_finite(solver, shape):
    """Nothing is iterated: u is the start."""
    for bad in (float("nan"), float("inf")):
        ub = base(shape)
        ub.view(-1)[77] = bad
        u, info = solve(solver, ub, 4, init="zero")
        assert info["status_name"] == "NONFINITE" and info["iters"] == 0 and float(u.abs().max()) == 0.0
    big = base(shape) * 2.0 ** 532            # finite, its inner products are not
    u, info = solve(solver, big, 4)
    assert info["status_name"] == "NONFINITE" and info["iters"] == 0 and info["r_ref"] == float("inf")
    assert float((u / big.abs().max() - big / big.abs().max()).abs().max()) <= 1e-13
    u, info = solve(solver, big, 4, init="zero")
    assert info["status_name"] == "NONFINITE" and float(u.abs().max()) == 0.0


@pytest.mark.parametrize("solver", ["vc", "sd", "cg", "bicgstab"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_mean_beyond_the_root_of_the_range(solver, shape):
    """The square of the mean overflows, but the mean has no residual.  The FFT
    rounds the rest at 2^-52 2^40 times a few: 1e-2."""
    _, want = solve(solver, base(shape), 3)
    _, info = solve(solver, base(shape) * 2.0 ** 482 + 2.0 ** 522, 3)
    assert info["status_name"] == "MAXITER" and info["iters"] == 3
    for k in ("r_ref", "r_final", "r_true"):
        assert abs(info[k] / 2.0 ** 482 - want[k]) <= 1e-2 * want["r_ref"], k


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_squares_that_underflow(shape):
    """Van Cittert takes no scalars from the sums: its iterate scales with the
    field, also in the classes whose |coefficient|^2 is below the range."""
    want, _ = solve("vc", base(shape), 2)
    u, info = solve("vc", base(shape) * 2.0 ** -533, 2)
    assert info["iters"] == 2
    assert float((u * 2.0 ** 533 - want).norm() / want.norm()) <= 1e-10
