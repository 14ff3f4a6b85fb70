"""The differential-filter solve from ubar and zero on a grid whose wavenumber
classes do not fit the class solve (4096 x 2048: 2.1 M of them), and the class
solve's rounds.

Tolerances as in test_gpu_classes.py: FP32 2e-4 after three passes.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import rel_l2, to_dev
from paper_1707_09177_amd import gdecon

pytestmark = pytest.mark.gpu

SHAPE = (1, 2048, 4096)
SPECTRAL = 5000   # variant codes of the general spectral sweeps start here


@pytest.fixture(scope="module")
def ub():
    u = np.random.default_rng(8).standard_normal(SHAPE)
    return oracle.germano_filter(u, 2, 0.02).astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("solver, init", [("vc", "ubar"), ("sd", "zero"), ("cg", "ubar"), ("bicgstab", "ubar"),
                                          ("bicgstab", "zero")])
def test_grid_without_class_solve_matches_oracle(ub, solver, init):
    want, winf, whist = oracle.solve(solver, ub, 2, 3, init=init, gamma=0.02)
    got, ginf, ghist = gdecon.deconvolve_germano(solver, to_dev(ub, torch.float32), 3, 0.02, init=init, history=True)
    assert gdecon.last_launch()["variant"] >= SPECTRAL
    assert rel_l2(got.double().cpu().numpy(), want) <= 2e-4
    np.testing.assert_allclose(ghist.cpu().numpy(), whist, rtol=2e-4)
    assert ginf[0]["iters"] == winf[0]["iters"] == 3 and ginf[0]["status_name"] == winf[0]["status_name"]
    assert abs(ginf[0]["r_true"] - winf[0]["r_true"]) <= 2e-4 * winf[0]["r_ref"]


@pytest.mark.parametrize("solver", ["cg", "bicgstab"])
def test_grid_without_class_solve_stops_on_the_true_residual(ub, solver):
    x = to_dev(ub, torch.float32)
    seen = set()
    for tol in (1e-1, 1e-2, 1e-7):
        _, inf, _ = gdecon.deconvolve_germano(solver, x, 400, 0.02, tol=tol)
        assert gdecon.last_launch()["variant"] >= SPECTRAL
        i = inf[0]
        seen.add(i["status_name"])
        if i["status_name"] == "CONVERGED":
            assert i["r_true"] <= tol * i["r_ref"]
        elif i["status_name"] == "STAGNATED":
            assert i["replaced"] == 2 and i["r_true"] > tol * i["r_ref"]
        else:
            assert i["status_name"] == "MAXITER" and i["iters"] == 400
    assert "CONVERGED" in seen and len(seen) == 2


def test_class_solve_in_rounds():
    """13 fields of 1024^2 at 22 workgroups each: more than fit at once, every field as if alone."""
    g = torch.Generator("cuda").manual_seed(2)
    x = gdecon.germano_filter(torch.randn(13, 1024, 1024, device="cuda", generator=g), 0.2)
    d = gdecon.GermanoDeconvolver(x.shape, 2, x.dtype, "bicgstab", 0.2)
    res = d.solve(x, 20)
    launch = gdecon.last_launch()
    assert launch["variant"] < SPECTRAL and launch["tiles"] > launch["blocks"]
    infos = res.info()
    one = gdecon.GermanoDeconvolver(x[:1].shape, 2, x.dtype, "bicgstab", 0.2)
    for b in (0, 11, 12):
        r1 = one.solve(x[b:b + 1].contiguous(), 20)
        assert torch.equal(r1.u[0], res.u[b]) and r1.info()[0] == infos[b]
