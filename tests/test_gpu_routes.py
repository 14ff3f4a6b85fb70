"""The control paths of a uniform solve on both of its routes: starts, guards,
the tolerance stop, residual replacement, the wait bound and capture, streamed
and in registers, whatever the dispatch chooses for their small fields.

The imported tests run here with the route pinned, and every solve is checked to
have taken it.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import gpu_solve, rel_l2
from paper_1707_09177_amd import gdecon
from test_gpu_control import (test_converged_means_true_residual_within_tol,  # noqa: F401
                              test_replacement_near_the_fp32_floor, test_replacement_restarts_from_the_current_iterate,
                              test_warm_start_choice_and_parity, test_warm_start_reference_norms)
from test_gpu_parity import (test_batch_equals_single, test_bicgstab_single_mode_half_step,  # noqa: F401
                             test_bitwise_deterministic, test_fp32_mode_2d_against_fp64_oracle,
                             test_fp32_mode_3d_against_fp64_oracle, test_given_exact_start_converges_at_once,
                             test_guards, test_init_modes_and_reference_norm, test_mean_preserved,
                             test_solver_fp64_fixed_passes, test_tolerance_stop_matches_oracle)

pytestmark = pytest.mark.gpu

RESIDENT = 10000
plain_solve = gdecon.Deconvolver.solve


@pytest.fixture(params=["streamed", "resident"], autouse=True)
def route(request, monkeypatch):
    """Every uniform solve of the test takes this route."""
    def solve(self, ubar, *args, **kw):
        if type(self) is not gdecon.Deconvolver:
            return plain_solve(self, ubar, *args, **kw)
        out = kw.get("out")
        gdecon.tune_set(self.solver, ubar, ubar if out is None else out, ndim=self.ndim, tiles_per_wave=1,
                        rows=4 if self.ndim == 3 else 0, resident=int(request.param == "resident"))
        res = plain_solve(self, ubar, *args, **kw)
        assert (gdecon.last_launch()["variant"] >= RESIDENT) == (request.param == "resident")
        return res
    monkeypatch.setattr(gdecon.Deconvolver, "solve", solve)
    yield request.param
    gdecon.tune_reset()


@pytest.mark.parametrize("solver", ["sd", "cg", "bicgstab"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("shape", [(16, 24), (4, 6, 8), (300, 200)], ids=lambda s: "x".join(map(str, s)))
def test_breakdown_where_g_vanishes(solver, dtype, shape):
    """ubar alternating along x: G ubar = 0, so the first step has no length."""
    ub = np.broadcast_to(np.where(np.arange(shape[-1]) % 2, -1.0, 1.0), (1,) + shape).copy()
    u, info, _ = gpu_solve(solver, ub, len(shape), 5, dtype=dtype)
    _, winf, _ = oracle.solve(solver, ub, len(shape), 5)
    assert info[0]["status_name"] == winf[0]["status_name"] == "BREAKDOWN_RHO"
    assert info[0]["iters"] == winf[0]["iters"] == 0 and np.array_equal(u, ub)


@pytest.mark.parametrize("solver", ["vc", "sd", "cg", "bicgstab"])
@pytest.mark.parametrize("init", ["zero", "given", "warm"])
def test_history_of_every_start(solver, init):
    shape = (2, 60, 90)
    r = np.random.default_rng(4)
    ub = oracle.filter(r.standard_normal(shape), 2)
    u0 = None if init == "zero" else np.stack([ub[0] + 0.9 * (ub[0] - oracle.filter(ub[0], 2)), ub[1] + r.standard_normal(shape[1:])])
    want, winf, whist = oracle.solve(solver, ub, 2, 5, init=init, u0=u0)
    got, ginf, ghist = gpu_solve(solver, ub, 2, 5, init=init, u0=u0)
    assert rel_l2(got, want) <= 1e-10
    np.testing.assert_allclose(ghist, whist, rtol=1e-9)
    assert [i["status"] for i in ginf] == [i["status"] for i in winf]


def test_wait_bound(route):
    """A solve that ran over the bound says so in every record."""
    ub = gdecon.filter_apply(torch.randn(4, 512, 512, device="cuda", dtype=torch.float64))
    d = gdecon.Deconvolver(ub.shape, 2, ub.dtype, "bicgstab")
    full = d.solve(ub, 6).info()
    seen = set()
    for limit in (1, 1, 1, 2, 2):
        names = {i["status_name"] for i in d.solve(ub, 6, wait_limit_us=limit).info()}
        assert len(names) == 1 and names <= {"TIMEOUT", "MAXITER"}
        seen |= names
    assert "TIMEOUT" in seen
    assert d.solve(ub, 6).info() == full


@pytest.mark.parametrize("solver, tol", [("bicgstab", 1e-5), ("vc", 0.0)])
def test_capture_and_replay(solver, tol):
    ub = gdecon.filter_apply(gdecon.filter_apply(torch.randn(3, 200, 300, device="cuda")))
    d = gdecon.Deconvolver(ub.shape, 2, ub.dtype, solver)
    out = torch.empty_like(ub)
    res = d.solve(ub, 30, tol, out=out)
    eager, info = out.clone(), res.info()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        d.solve(ub, 30, tol, out=out)
    for _ in range(3):
        out.fill_(float("nan"))
        (torch.randn(1 << 20, device="cuda") * 2).sum().item()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager) and res.info() == info
