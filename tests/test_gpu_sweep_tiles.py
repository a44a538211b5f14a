"""GPU: the time-tiled matrix-core history sweep in the forms it serves beside two-plane float32.

float64, one plane per material group, groups of two modes per kernel row and the 64-step depth,
against the float64 oracle on small grids (switched on with SBIM_SWEEP_KIND=mfma), and by the
library's own rule against the vector-unit sweep on a grid where the rule picks it.  Bars: relative
L2 1e-12 in float64 and 1e-5 in the float32 forms, as for the other sweeps.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_2102_08756_amd import SBIM, Config, Fault, SBIMError, SBIMRun

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ONE = [dict(side=1)]
TWO = [dict(side=1), dict(side=-1, mu=2.5)]
BIMATERIAL = [dict(side=1), dict(side=-1, cs=1.2, cp=2.5)]
BAR = {"fp64": 1e-12, "fp32": 1e-5, "fp32_comp": 1e-5}

CASES = {
    # the shortest window it takes, one of a whole number of 32-lag rounds and one more; ragged last block
    "one16_w4": (dict(n1=16, n3=16, window_cap=4, planes=ONE), 40),
    "one16_w32": (dict(n1=16, n3=16, window_cap=32, planes=ONE), 100),
    "one32x16_w33": (dict(n1=32, n3=16, window_cap=33, planes=ONE), 110),
    # anisotropic: only +-m1 share a row, two modes a group and 64 steps a pass
    "one_aniso16x32_w37": (dict(n1=16, n3=32, dx1=0.7, dx3=1.3, window_cap=37, planes=ONE), 170),
    "two_aniso16x32_w37": (dict(n1=16, n3=32, dx1=0.7, dx3=1.3, window_cap=37, planes=TWO), 100),
    "two32_w40": (dict(n1=32, n3=32, window_cap=40, planes=TWO), 110),
    "bimaterial4x8_w21": (dict(n1=4, n3=8, window_cap=21, planes=BIMATERIAL), 90),
}
_REF = {}


def rel_l2(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(np.asarray(b)))


def inputs(cfg, steps, seed=3):
    rng = np.random.default_rng(seed)
    return rng.standard_normal((steps, len(cfg["planes"]), 3, cfg["n1"], cfg["n3"]))


def run(cfg, u, precision):
    sb = SBIM(Config.from_dict(cfg, precision=precision), device=DEV)
    ut = torch.tensor(u, dtype=sb.dtype, device=DEV).requires_grad_(True)
    tau = SBIMRun.apply(sb, ut)
    (grad,) = torch.autograd.grad(tau.square().sum(), ut)
    info = sb.info()
    sb.close()
    return tau.detach().double().cpu().numpy(), grad.double().cpu().numpy(), info


@pytest.mark.parametrize("chunks", [1, 4])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_comp"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_tiled_sweep_matches_oracle(case, precision, chunks, monkeypatch):
    monkeypatch.setenv("SBIM_SWEEP_KIND", "mfma")
    monkeypatch.setenv("SBIM_SWEEP_CHUNKS", str(chunks))
    cfg = dict(CASES[case][0], input_kind="increment" if chunks == 1 else "absolute")
    u = inputs(cfg, CASES[case][1])
    key = (case, chunks)
    if key not in _REF:
        _REF[key] = oracle.forward(cfg, u)
    got, _, info = run(cfg, u, precision)
    assert info["sweep_matrix_cores"] == 1 and info["sweep_lag_chunks"] == chunks
    err = rel_l2(got, _REF[key])
    print(f"[tiles] {case} {precision} chunks {chunks} depth {info['sweep_depth']}: {err:.1e}",
          flush=True)
    assert err < BAR[precision]


@pytest.mark.parametrize("planes", ["one", "two", "bimaterial"])
@pytest.mark.parametrize("dx3", [1.0, 1.3])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_comp"])
def test_rule_and_agreement_with_the_vector_sweep(precision, dx3, planes, monkeypatch):
    """128 x 65 modes x 64 lags is past the rule's bound (2^18), 63 lags are under its window."""
    for k in ("SBIM_SWEEP_KIND", "SBIM_SWEEP_DEPTH", "SBIM_SWEEP_CHUNKS", "SBIM_SWEEP_QUADS"):
        monkeypatch.delenv(k, raising=False)
    cfg = dict(n1=128, n3=128, dx1=1.0, dx3=dx3, window_cap=64, input_kind="increment",
               planes=dict(one=ONE, two=TWO, bimaterial=BIMATERIAL)[planes])
    u = inputs(cfg, 140)
    tau, grad, info = run(cfg, u, precision)
    assert info["sweep_matrix_cores"] == 1
    monkeypatch.setenv("SBIM_SWEEP_KIND", "valu")
    tau_v, grad_v, info_v = run(cfg, u, precision)
    assert info_v["sweep_matrix_cores"] == 0
    assert rel_l2(tau, tau_v) < BAR[precision] and rel_l2(grad, grad_v) < BAR[precision]
    monkeypatch.delenv("SBIM_SWEEP_KIND")
    sb = SBIM(Config.from_dict(dict(cfg, window_cap=63), precision="fp64"), device=DEV)
    assert sb.info()["sweep_matrix_cores"] == 0
    sb.close()


def test_fault_on_a_float32_handle_sums_in_order(monkeypatch):
    """The handle is planned again for the fault: same steps as with the vector sweep, bit for bit."""
    wl = workloads.FaultWorkload("tpv3_128", 128, 128, 250.0, 90)
    out = []
    for kind in (None, "valu"):
        monkeypatch.delenv("SBIM_SWEEP_KIND", raising=False)
        if kind:
            monkeypatch.setenv("SBIM_SWEEP_KIND", kind)
        sb = SBIM(Config.from_dict(wl.config_dict(), precision="fp32_comp"), device=DEV)
        assert sb.info()["sweep_matrix_cores"] == (0 if kind else 1)
        f = Fault(sb, *[torch.tensor(a, dtype=torch.float64, device=DEV) for a in wl.params()])
        assert sb.info()["sweep_matrix_cores"] == 0
        out.append(f.run(wl.steps))
        f.close()
        sb.close()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert out[0][1].abs().max() > 0


@pytest.mark.parametrize("running", [False, True])
def test_snapshot_names_its_mode_order(running, monkeypatch):
    """A snapshot without the mark (lag order) is refused by a tiled handle, taken by another."""
    cfg = dict(n1=16, n3=16, window_cap=8, planes=ONE)
    for kind, fits in (("mfma", False), ("valu", True)):
        monkeypatch.setenv("SBIM_SWEEP_KIND", kind)
        sb = SBIM(Config.from_dict(cfg, precision="fp64"), device=DEV)
        sb.push(sb.new_field().normal_())
        snap = sb.save_running_state() if running else sb.save_state()
        load = sb.load_running_state if running else sb.load_state
        load(snap)
        snap[8:256] = 0
        if fits:
            load(snap)
        else:
            with pytest.raises(SBIMError, match="orders the modes"):
                load(snap)
        assert sb.info()["step"] == 1
        sb.close()
