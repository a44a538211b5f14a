"""GPU: handles without the device memory for the time-tiled form (SBIM_MEMORY_LIMIT stands in for
a full device) are planned in the forms that hold less, and keep their history when that is found
out by the first adjoint."""
import pytest
import torch

from paper_2102_08756_amd import SBIM, Config, Fault, SBIMError

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MIB = 1 << 20


def handle(monkeypatch, precision, kind=None, limit=None, planes=(dict(side=1),), input_kind="absolute"):
    for k in ("KIND", "DEPTH", "CHUNKS", "QUADS"):
        monkeypatch.delenv("SBIM_SWEEP_" + k, raising=False)
    monkeypatch.delenv("SBIM_MEMORY_LIMIT", raising=False)
    if kind:
        monkeypatch.setenv("SBIM_SWEEP_KIND", kind)
    if limit:
        monkeypatch.setenv("SBIM_MEMORY_LIMIT", str(limit))
    cfg = dict(n1=128, n3=128, window_cap=64, planes=list(planes), input_kind=input_kind)
    return SBIM(Config.from_dict(cfg, precision=precision), device=DEV)


def fields(sb, n):
    gen = torch.Generator(device=DEV).manual_seed(5)
    return [torch.randn(sb.new_field().shape, dtype=sb.dtype, device=DEV, generator=gen) for _ in range(n)]


def step(sb, u):
    sb.push(u)
    return sb.tractions().clone()


@pytest.mark.parametrize("precision", ["fp64", "fp32_comp"])
def test_init_without_room_for_the_tiled_form(precision, monkeypatch):
    tiled, vector = handle(monkeypatch, precision), handle(monkeypatch, precision, "valu")
    assert tiled.info()["sweep_matrix_cores"] == 1 and vector.info()["sweep_matrix_cores"] == 0
    limit = vector.state_bytes() + vector.info()["table_bytes"] + 6 * MIB
    assert tiled.state_bytes() + tiled.info()["table_bytes"] > limit
    sb = handle(monkeypatch, precision, limit=limit)
    assert sb.info() == vector.info()
    u = fields(sb, 90)
    for x in u[:75]:
        assert torch.equal(step(sb, x), step(vector, x))
        tiled.push(x)
    # the snapshots of either fit the other
    snap = sb.save_state()
    sb.load_state(tiled.save_state())
    for x in u[75:]:
        assert torch.equal(step(sb, x), step(vector, x))
    tiled.load_state(snap)
    monkeypatch.delenv("SBIM_MEMORY_LIMIT")
    assert tiled.info()["step"] == 75
    for h in (tiled, vector, sb):
        h.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_adjoint_without_room_beside_the_tiled_form(precision, monkeypatch):
    bimaterial = (dict(side=1), dict(side=-1, cs=1.2, cp=2.5))
    own = handle(monkeypatch, precision, "valu", planes=bimaterial)
    sb = handle(monkeypatch, precision, planes=bimaterial)
    assert sb.info()["sweep_matrix_cores"] == 1
    u = fields(sb, 60)
    for x in u[:40]:
        sb.push(x)
        own.push(x)
    state = 2 * 128 * 65 * 3 * 16
    limit = own.state_bytes() + state + 4 * MIB
    assert sb.state_bytes() > limit
    monkeypatch.setenv("SBIM_MEMORY_LIMIT", str(limit))
    for x in u[:30]:
        assert torch.equal(sb.backward(x), own.backward(x))
    assert sb.info() == own.info() and sb.info()["sweep_matrix_cores"] == 0
    for x in u[40:]:
        assert torch.equal(step(sb, x), step(own, x))
    sb.close()
    own.close()


def test_without_room_for_any_form(monkeypatch):
    with pytest.raises(SBIMError, match="SBIM_E_OOM"):
        handle(monkeypatch, "fp64", limit=MIB)
    # an adjoint that finds none: the handle and its history stay as they are
    sb, own = handle(monkeypatch, "fp64"), handle(monkeypatch, "fp64")
    u = fields(sb, 20)
    for x in u[:10]:
        assert torch.equal(step(sb, x), step(own, x))
    info = sb.info()
    monkeypatch.setenv("SBIM_MEMORY_LIMIT", str(MIB))
    with pytest.raises(SBIMError, match="SBIM_E_OOM"):
        sb.backward(u[0])
    monkeypatch.delenv("SBIM_MEMORY_LIMIT")
    assert sb.info() == info
    for x in u[10:]:
        assert torch.equal(step(sb, x), step(own, x))
    assert torch.equal(sb.backward(u[0]), own.backward(u[0]))
    sb.close()
    own.close()


def test_handle_without_buffers_refuses_every_call(monkeypatch):
    """Planned again for a fault without memory for any form: the calls say so."""
    sb = handle(monkeypatch, "fp32")
    u, snap, light = sb.new_field(), sb.save_state(), sb.save_running_state()
    prm = [torch.full((3, 128, 128), -1.0, dtype=torch.float64, device=DEV)]
    prm += [torch.full((128, 128), v, dtype=torch.float64, device=DEV) for v in (0.6, 0.5, 0.4)]
    monkeypatch.setenv("SBIM_MEMORY_LIMIT", "1")
    with pytest.raises(SBIMError, match="SBIM_E_OOM"):
        Fault(sb, *prm)
    monkeypatch.delenv("SBIM_MEMORY_LIMIT")
    for call in (lambda: sb.push(u), lambda: sb.backward(u), lambda: sb.save_state(snap),
                 lambda: sb.load_state(snap), lambda: sb.save_running_state(light),
                 lambda: sb.load_running_state(light), sb.reset, sb.backward_reset,
                 lambda: sb.mode_kernel(0, 1, 1, 4)):
        with pytest.raises(SBIMError, match="SBIM_E_STATE.*no history buffers"):
            call()
    sb.info(), sb.state_bytes(), sb.step_work(3)
    sb.close()
