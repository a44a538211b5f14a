"""GPU: the vector sweep with long blocks split over the wavefronts of a work-group.

Small grids against the float64 oracle; larger ones, with several long blocks per launch beside short
ones, against the unsplit sweep (SBIM_SWEEP_DEPTH=4, which is never split), forward and gradient.
Bars: relative L2 1e-12 in float64 and 1e-5 in the float32 forms, as for the other sweeps.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2102_08756_amd import SBIM, Config, SBIMRun

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ONE = [dict(side=1)]
TWO = [dict(side=1), dict(side=-1)]
BIMATERIAL = [dict(side=1), dict(side=-1, cs=1.2, cp=2.5)]
BAR = {"fp64": 1e-12, "fp32": 1e-5, "fp32_comp": 1e-5}

SMALL = {
    "w20": (dict(n1=16, n3=16, window_cap=20, planes=ONE), 50),                # 6 steps a pass
    "w25_two": (dict(n1=32, n3=16, window_cap=25, planes=TWO), 60),
    "w70": (dict(n1=16, n3=16, window_cap=70, planes=ONE), 160),               # 8 or 12 steps a pass
    "w97_bimaterial": (dict(n1=8, n3=16, window_cap=97, planes=BIMATERIAL), 130),
    "per_mode": (dict(n1=32, n3=16, window_cap=60, window_mode="per_mode", planes=TWO), 90),
}
LARGE = {
    "per_mode_128x64": dict(n1=128, n3=64, window_cap=200, window_mode="per_mode", planes=TWO),
    "per_mode_256": dict(n1=256, n3=256, window_cap=90, window_mode="per_mode", planes=ONE),
    "w25_256": dict(n1=256, n3=256, window_cap=25, planes=ONE),
    "w60_bimaterial": dict(n1=64, n3=64, window_cap=60, planes=BIMATERIAL),
}


def rel_l2(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(np.asarray(b)))


def inputs(cfg, steps):
    return np.random.default_rng(9).standard_normal((steps, len(cfg["planes"]), 3, cfg["n1"], cfg["n3"]))


def run(cfg, u, precision):
    sb = SBIM(Config.from_dict(cfg, precision=precision), device=DEV)
    assert sb.info()["sweep_matrix_cores"] == 0
    ut = torch.tensor(u, dtype=sb.dtype, device=DEV).requires_grad_(True)
    tau = SBIMRun.apply(sb, ut)
    (grad,) = torch.autograd.grad(tau.square().sum(), ut)
    depth = sb.info()["sweep_depth"]
    sb.close()
    return tau.detach().double().cpu().numpy(), grad.double().cpu().numpy(), depth


@pytest.fixture(autouse=True)
def vector_sweep(monkeypatch):
    monkeypatch.setenv("SBIM_SWEEP_KIND", "valu")
    monkeypatch.delenv("SBIM_SWEEP_DEPTH", raising=False)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_comp"])
@pytest.mark.parametrize("case", sorted(SMALL))
def test_small_grids_match_oracle(case, precision):
    cfg = dict(SMALL[case][0], input_kind="increment")
    u = inputs(cfg, SMALL[case][1])
    got, _, depth = run(cfg, u, precision)
    err = rel_l2(got, oracle.forward(cfg, u))
    print(f"[split] {case} {precision} depth {depth}: {err:.1e}", flush=True)
    assert err < BAR[precision]


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_comp"])
@pytest.mark.parametrize("case", sorted(LARGE))
def test_larger_grids_match_the_unsplit_sweep(case, precision, monkeypatch):
    cfg = dict(LARGE[case], input_kind="increment")
    u = inputs(cfg, min(cfg["window_cap"], 100) + 20)
    tau, grad, depth = run(cfg, u, precision)
    monkeypatch.setenv("SBIM_SWEEP_DEPTH", "4")
    tau4, grad4, depth4 = run(cfg, u, precision)
    assert depth != 4 and depth4 == 4
    assert rel_l2(tau, tau4) < BAR[precision] and rel_l2(grad, grad4) < BAR[precision]
