"""GPU: the in-order float32 sweep with its history staged through LDS, against the float64 oracle.

It serves float32 handles that drive a fault, at 12 steps a pass with windows of 64 lags or more; a
handle keeps that form after its fault is closed, so its tractions for random inputs are compared
directly.  Windows on both sides of a whole number of 12-lag stages per chunk; runs long enough for the
ring to wrap.  Bar: relative L2 1e-5, as for the other float32 sweeps.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2102_08756_amd import SBIM, Config, Fault

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ONE = [dict(side=1)]
BIMATERIAL = [dict(side=1), dict(side=-1, cs=1.2, cp=2.5)]


@pytest.mark.parametrize("n1,n3,window,planes,precision", [
    (4, 4, 64, ONE, "fp32_comp"), (16, 16, 65, ONE, "fp32_comp"), (16, 8, 72, BIMATERIAL, "fp32_comp"),
    (32, 16, 73, ONE, "fp32_comp"), (16, 16, 97, BIMATERIAL, "fp32_comp"), (8, 8, 1500, ONE, "fp32")])
def test_staged_sweep_matches_oracle(n1, n3, window, planes, precision, monkeypatch):
    for k in ("SBIM_SWEEP_KIND", "SBIM_SWEEP_DEPTH"):
        monkeypatch.delenv(k, raising=False)
    cfg = dict(n1=n1, n3=n3, window_cap=window, planes=planes, input_kind="increment")
    sb = SBIM(Config.from_dict(cfg, precision=precision), device=DEV)
    cell = torch.ones((n1, n3), dtype=torch.float64, device=DEV)
    Fault(sb, torch.stack([cell, -cell, 0 * cell]), cell, 0.5 * cell, cell).close()
    info = sb.info()
    assert info["sweep_depth"] == 12 and info["sweep_matrix_cores"] == 0
    u = np.random.default_rng(window).standard_normal((window + 90, len(planes), 3, n1, n3))
    got = np.empty(u.shape)
    for n in range(len(u)):
        sb.push(torch.tensor(u[n], dtype=sb.dtype, device=DEV))
        got[n] = sb.tractions().double().cpu().numpy()
    sb.close()
    ref = oracle.forward(cfg, u)
    err = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    print(f"[staged] {n1} x {n3} W = {window} {precision}: {err:.1e}", flush=True)
    assert err < 1e-5
