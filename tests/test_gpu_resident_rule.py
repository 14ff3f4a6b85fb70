"""Which batches are solved in registers, and in which boxes: fields that fit
stream where a batch would take too many rounds, small fields are cut into few
boxes where many boxes would take more rounds, and a pinned choice holds.

Tolerances as in test_gpu_resident.py: FP64 1e-10 relative L2 (or 20 times the
oracle's spread between its summation orders), FP32 1e-5.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import filtered_input, rel_l2_per_field, to_dev
from paper_1707_09177_amd import gdecon

pytestmark = pytest.mark.gpu

RESIDENT = 10000


def run(solver, ub, N, **kw):
    nd = ub.dim() - 1
    out = torch.empty_like(ub)
    res = gdecon.Deconvolver(ub.shape, nd, ub.dtype, solver).solve(ub, N, 0.0, out=out, **kw)
    return out, res.info(), gdecon.last_launch()


# (fields, shape, solver, dtype, in registers): one field at a time on 189 and 156
# boxes; the same fields alone; batches that fill their rounds
@pytest.mark.parametrize("shape, solver, dtype, resident", [
    ((8, 160, 160, 160), "vc", torch.float32, False), ((1, 160, 160, 160), "vc", torch.float32, True),
    ((20, 150, 150, 150), "vc", torch.float64, False), ((16, 1024, 1024), "bicgstab", torch.float32, True),
    ((16, 2048, 2048), "bicgstab", torch.float32, True), ((3, 90, 100, 97), "cg", torch.float64, True),
    ((24528, 19, 12, 9), "vc", torch.float32, False), ((5, 19, 12, 9), "vc", torch.float32, True),
], ids=str)
def test_route(shape, solver, dtype, resident):
    nd = len(shape) - 1
    ub = gdecon.filter_apply(torch.randn(shape, device="cuda", dtype=dtype), ndim=nd)
    got, info, launch = run(solver, ub, 3)
    assert (launch["variant"] >= RESIDENT) == resident
    out = torch.empty_like(ub)
    gdecon.tune_set(solver, ub, out, ndim=nd, resident=0 if resident else 1)
    try:
        res = gdecon.Deconvolver(ub.shape, nd, dtype, solver).solve(ub, 3, 0.0, out=out)
        other = gdecon.last_launch()
    finally:
        gdecon.tune_reset()
    # a pinned choice is used where the field fits (150^3 FP64 does not)
    assert (other["variant"] >= RESIDENT) == (not resident and shape != (20, 150, 150, 150))
    tol = 1e-10 if dtype == torch.float64 else 1e-5
    assert float((got - out).norm() / got.norm()) <= tol
    assert [(i["iters"], i["status"]) for i in res.info()] == [(i["iters"], i["status"]) for i in info]


# batches past one round of short columns: full columns, of one box and of two
@pytest.mark.parametrize("solver", ["vc", "sd", "cg", "bicgstab"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("shape", [(70, 14, 9, 20), (300, 5, 6, 7), (90, 17, 12, 30), (100, 80, 136), (150, 97, 50)],
                         ids=lambda s: "x".join(map(str, s)))
def test_full_columns_match_oracle(solver, dtype, shape):
    nd = len(shape) - 1
    few = torch.empty((2,) + shape[1:], device="cuda", dtype=dtype).normal_(generator=torch.Generator("cuda").manual_seed(3))
    small = run(solver, gdecon.filter_apply(few, ndim=nd), 3)[2]
    u = np.random.default_rng(sum(shape)).standard_normal(shape)
    ub = filtered_input(oracle.filter(u, nd), nd, dtype)
    got, info, launch = run(solver, to_dev(ub, dtype), 3)
    assert launch["variant"] >= RESIDENT and launch["tiles"] // shape[0] <= small["tiles"] // 2
    want, winf, _ = oracle.solve(solver, ub, nd, 3)
    spread = max(max(rel_l2_per_field(oracle.solve(solver, ub, nd, 3, sum_mode=m)[0], want, nd)) for m in (1, 2))
    tol = max(1e-10, 20 * spread) if dtype == torch.float64 else 1e-5
    assert max(rel_l2_per_field(got.double().cpu().numpy(), want, nd)) <= tol
    assert [(i["iters"], i["status_name"]) for i in info] == [(i["iters"], i["status_name"]) for i in winf]


def test_tuner_times_both():
    """Where the rule streams a field that fits, the tuner has the solve in registers among its candidates."""
    ub = gdecon.filter_apply(torch.randn(8, 160, 160, 160, device="cuda"), ndim=3)
    assert run("vc", ub, 2)[2]["variant"] < RESIDENT
    try:
        t = gdecon.autotune("vc", ub, ndim=3)
        assert t["resident"] in (0, 1) and t["best_ms"] <= t["default_ms"] * 1.05
        _, _, launch = run("vc", ub, 2)
        assert (launch["variant"] >= RESIDENT) == (t["resident"] == 1)
    finally:
        gdecon.tune_reset()
