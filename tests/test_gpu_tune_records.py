"""What the tuner reports and saves: a choice of either route, in uniform solves
and in uneven batches, that a later process reads back and uses."""
import os
import subprocess
import sys

import pytest
import torch

from paper_1707_09177_amd import gdecon

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHAPES = [(300, 200), (40, 50, 60), (512, 512)]
CHILD = """
import sys, torch
sys.path.insert(0, sys.argv[1])
from paper_1707_09177_amd import gdecon
shapes = eval(sys.argv[2])
ubs = [torch.zeros(s, device="cuda") for s in shapes]
gdecon.BatchDeconvolver(shapes, torch.float32, "cg").solve(ubs, 1)
a = gdecon.last_launch()
x = torch.zeros(1, 300, 200, device="cuda")
gdecon.Deconvolver(x.shape, 2, x.dtype, "cg").solve(x, 1)
print([a["tiles"], a["blocks"], gdecon.last_launch()["variant"], gdecon.last_launch()["tiles"]])
"""


def test_saved_choices_are_read_back(tmp_path, monkeypatch):
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("GD_TUNE_CACHE", str(cache))
    try:
        ubs = [gdecon.filter_apply(torch.randn(s, device="cuda"), ndim=len(s)) for s in SHAPES]
        bd = gdecon.BatchDeconvolver(SHAPES, torch.float32, "cg")
        assert bd.autotune(ubs)["resident"] == 0          # uneven batches stream
        # a choice that no default makes, so that its loss would show
        bd.tune_set(ubs, [torch.empty_like(u) for u in ubs], tiles_per_wave=6, tail_pct=25, blocks_per_cu=1)
        bd.solve(ubs, 1)
        want = gdecon.last_launch()
        x = torch.zeros(1, 300, 200, device="cuda")
        gdecon.tune_set("cg", x, torch.empty_like(x), tiles_per_wave=4, resident=0)
        gdecon.Deconvolver(x.shape, 2, x.dtype, "cg").solve(x, 1)
        one = gdecon.last_launch()
        assert one["variant"] < 10000
        for line in cache.read_text().splitlines():
            assert len(line.split()) == 9 and line.split()[-1] in ("0", "1"), line
        r = subprocess.run([sys.executable, "-c", CHILD, ROOT, repr(SHAPES)], capture_output=True, text=True, timeout=100)
        assert r.returncode == 0, r.stderr[-2000:]
        assert eval(r.stdout.strip().splitlines()[-1]) == [want["tiles"], want["blocks"], one["variant"], one["tiles"]]
    finally:
        gdecon.tune_reset()
