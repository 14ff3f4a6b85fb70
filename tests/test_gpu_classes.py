"""The differential-filter solve on wavenumber classes (starts from ubar or
zero) against the oracle, at the edges of its dispatch: every kind of fold
(signs only, square, cube), one and several classes per thread, fields that
span several workgroups and more fields than fit at once, exits before the
first pass, and the hand-over to the general solver at the FP32 floor.

Tolerances: FP64 as for the general path, 1e-10 relative L2 for a few passes on
mildly conditioned filters, or 20 times the oracle's spread between its
summation orders; FP32 2e-4.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import rel_l2_per_field, to_dev
from paper_1707_09177_amd import gdecon, synth

pytestmark = pytest.mark.gpu

# (shape, fields): square of one, two, four and more classes per thread and of
# five workgroups (512^2: 33153 classes); cube; signs only, with sizes of 2
FOLDS = [((32, 32), 3), ((64, 64), 2), ((128, 128), 1), ((512, 512), 2), ((2, 64), 2), ((256, 64), 1),
         ((16, 16, 16), 2), ((32, 32, 32), 1), ((64, 64, 64), 1), ((4, 16, 16), 2), ((64, 32, 128), 1)]


@pytest.mark.parametrize("solver", ["vc", "sd", "cg", "bicgstab"])
@pytest.mark.parametrize("shape,count", FOLDS)
def test_folds_match_oracle(solver, shape, count):
    nd = len(shape)
    u = np.random.default_rng(11 + len(shape)).standard_normal((count,) + shape)
    ub = oracle.germano_filter(u, nd, 0.5)
    want, winf, whist = oracle.solve(solver, ub, nd, 4, gamma=0.5)
    spread = max(max(rel_l2_per_field(oracle.solve(solver, ub, nd, 4, gamma=0.5, sum_mode=m)[0], want, nd))
                 for m in (1, 2))
    for dtype, tol in ((torch.float64, max(1e-10, 20 * spread)), (torch.float32, 2e-4)):
        got, ginf, ghist = gdecon.deconvolve_germano(solver, to_dev(ub, dtype), 4, 0.5, ndim=nd, history=True)
        for e in rel_l2_per_field(got.double().cpu().numpy(), want, nd):
            assert e <= tol, e
        np.testing.assert_allclose(ghist.cpu().numpy(), whist, rtol=max(tol, 1e-8))
        for gi, wi in zip(ginf, winf):
            assert gi["iters"] == wi["iters"] == 4 and gi["status_name"] == wi["status_name"]
            assert abs(gi["r_true"] - wi["r_true"]) <= max(tol, 1e-8) * wi["r_ref"]


def test_more_fields_than_fit_at_once():
    """9 fields of 1024^2 need 22 workgroups each: several rounds over the fields; every field as if alone."""
    u = np.stack([synth.field_2d(256, synth.spectrum_kraichnan, 4.0, 64.0, synth.rng_for(2, i)) for i in range(13)])
    ub = to_dev(np.tile(oracle.germano_filter(u, 2, 0.2), (1, 4, 4)), torch.float32)
    d = gdecon.GermanoDeconvolver(ub.shape, 2, ub.dtype, "bicgstab", 0.2)
    res = d.solve(ub, 100, 1e-3)
    infos = res.info()
    one = gdecon.GermanoDeconvolver(ub[:1].shape, 2, ub.dtype, "bicgstab", 0.2)
    for b in (0, 5, 12):
        r1 = one.solve(ub[b:b + 1].contiguous(), 100, 1e-3)
        assert torch.equal(r1.u[0], res.u[b]) and r1.info()[0] == infos[b]
        assert infos[b]["status_name"] == "CONVERGED"


def test_exits_before_the_first_pass():
    ub = np.random.default_rng(3).standard_normal((4, 32, 32))
    ub[1] = 0.0                      # zero reference norm: u = ubar
    ub[2] = 1.0                      # G ubar = ubar: the same
    ub[3, 5, 5] = np.nan
    got, inf, _ = gdecon.deconvolve_germano("bicgstab", to_dev(ub, torch.float64), 0, 0.5)
    assert [i["status_name"] for i in inf][0::3] == ["MAXITER", "NONFINITE"]
    assert inf[1]["status_name"] == "ZERO_REF" and inf[2]["r_ref"] <= 1e-12
    g = got.cpu().numpy()
    np.testing.assert_allclose(g[:3], ub[:3], atol=1e-13)
    got, inf, _ = gdecon.deconvolve_germano("cg", to_dev(ub, torch.float64), 5, 0.5, init="zero")
    want, winf, _ = oracle.solve("cg", ub[:1], 2, 5, init="zero", gamma=0.5)
    assert rel_l2_per_field(got[:1].cpu().numpy(), want, 2)[0] <= 1e-10
    assert inf[1]["status_name"] == "ZERO_REF" and inf[3]["status_name"] == "NONFINITE"
    assert float(got[1].abs().max()) == 0.0


@pytest.mark.parametrize("solver", ["cg", "bicgstab", "vc"])
def test_fp32_floor_is_handed_to_the_general_solver(solver):
    """At tolerances around the FP32 rounding of u_hat the recursive residual
    (FP64) meets tol where the true one does not: CONVERGED keeps meaning
    r_true <= tol r_ref, and below the floor the solve ends STAGNATED after the
    replacements allowed."""
    u = np.stack([synth.field_2d(64, synth.spectrum_kraichnan, 4.0, 16.0, synth.rng_for(2, i)) for i in range(2)])
    ub = to_dev(oracle.germano_filter(u, 2, 1.0), torch.float32)
    seen = set()
    for tol in (1e-5, 1e-6, 6e-7, 3e-7, 2e-7, 1e-7, 3e-8):
        _, inf, _ = gdecon.deconvolve_germano(solver, ub, 2000, 1.0, tol=tol)
        for i in inf:
            seen.add(i["status_name"])
            if i["status_name"] == "CONVERGED":
                assert i["r_true"] <= tol * i["r_ref"]
            else:
                assert i["status_name"] == "STAGNATED" and i["replaced"] == 2 and i["r_true"] > tol * i["r_ref"]
    assert seen == {"CONVERGED", "STAGNATED"}
