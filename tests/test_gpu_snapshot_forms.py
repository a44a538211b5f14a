"""GPU: snapshots say how they lie in memory.

A handle holds its modes, history and pending sums in an order that depends on its sweep form and
depth; a snapshot is that memory with a header.  Continuing from one must give what the same handle
gives without it, bit for bit, or the snapshot must be refused.
"""
import pytest
import torch

from paper_2102_08756_amd import SBIM, Config, SBIMError

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ONE = [dict(side=1)]
TWO = [dict(side=1), dict(side=-1, mu=2.5)]
BIMATERIAL = [dict(side=1), dict(side=-1, cs=1.2, cp=2.5)]


def handle(monkeypatch, cfg, precision, kind=None, depth=None):
    for k, v in (("SBIM_SWEEP_KIND", kind), ("SBIM_SWEEP_DEPTH", depth)):
        monkeypatch.delenv(k, raising=False)
        if v is not None:
            monkeypatch.setenv(k, str(v))
    return SBIM(Config.from_dict(cfg, precision=precision), device=DEV)


def pushes(sb, n, seed=4):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    return [torch.randn(sb.new_field().shape, dtype=sb.dtype, device=DEV, generator=gen) for _ in range(n)]


def steps(sb, fields):
    out = []
    for u in fields:
        sb.push(u)
        out.append(sb.tractions().clone())
    return out


@pytest.mark.parametrize("planes", [ONE, TWO, BIMATERIAL], ids=["one", "two", "bimaterial"])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_comp"])
def test_snapshot_without_a_mark(precision, planes, monkeypatch):
    """Snapshots without a mark hold the pending sums as ten real arrays per slot and plane."""
    cfg = dict(n1=16, n3=16, window_cap=20, planes=planes)
    sb = handle(monkeypatch, cfg, precision)
    assert sb.info()["sweep_matrix_cores"] == 0
    fields = pushes(sb, 45)
    steps(sb, fields[:33])
    snap = sb.save_state()
    want = steps(sb, fields[33:])
    real = 8 if precision == "fp64" else 4
    groups = sb.info()["material_groups"]
    np_, m = len(planes) // groups, 16 * 9
    slots = sb.info()["sweep_depth"] + 1
    snap[8:256] = 0
    end = snap.numel()
    for _ in range(groups):  # the last group lies last; its pending sums end it
        size = slots * np_ * 5 * m * 2 * real
        part = snap[end - size:end].view(sb.dtype).reshape(slots, np_, 5, m, 2)
        part.copy_(part.permute(0, 1, 2, 4, 3).reshape(slots, np_, 10, m).contiguous().reshape(part.shape))
        end -= (snap.numel() - 256 - len(planes) * 3 * m * 2 * real) // groups
    assert end == 256 + len(planes) * 3 * m * 2 * real
    sb.reset()
    sb.load_state(snap)
    got = steps(sb, fields[33:])
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    sb.close()


# (configuration, precision, form that writes, form that reads); a form is (kind, depth)
FORMS = {
    "depths_fp64": (dict(n1=16, n3=16, window_cap=20, planes=ONE), "fp64", ("valu", 6), ("valu", 8)),
    "depths_quads": (dict(n1=16, n3=16, window_cap=40, planes=TWO), "fp32", ("mfma", 16), ("mfma", None)),
    "tiled_to_vector": (dict(n1=16, n3=16, window_cap=24, planes=TWO), "fp32_comp", ("mfma", None), ("valu", None)),
    "vector_to_tiled": (dict(n1=16, n3=32, dx3=1.3, window_cap=24, planes=ONE), "fp64", ("valu", None), ("mfma", None)),
    "bimaterial": (dict(n1=8, n3=16, window_cap=21, planes=BIMATERIAL), "fp32", ("mfma", None), ("valu", 12)),
    "per_mode": (dict(n1=16, n3=16, window_cap=50, window_mode="per_mode", eta_w=1.0, planes=TWO), "fp64",
                 ("valu", 6), ("valu", 12)),
    # a step before the first tile is whole, windows past the tiles' end, two steps a tile
    "tiled_fp64_to_vector": (dict(n1=16, n3=16, window_cap=21, planes=TWO), "fp64", ("mfma", None), ("valu", None)),
    "vector_to_quads": (dict(n1=16, n3=16, window_cap=5, planes=ONE), "fp32", ("valu", 8), ("mfma", None)),
}


@pytest.mark.parametrize("cut", [2, 61])
@pytest.mark.parametrize("running", [False, True])
@pytest.mark.parametrize("case", sorted(FORMS))
def test_snapshot_of_another_form(case, running, cut, monkeypatch):
    """The steps after it are those of a handle of the reading form that made the whole run
    (after the running state: the steps once the history is rebuilt)."""
    cfg, precision, (kind_a, depth_a), (kind_b, depth_b) = FORMS[case]
    a = handle(monkeypatch, cfg, precision, kind_a, depth_a)
    own = handle(monkeypatch, cfg, precision, kind_b, depth_b)
    b = handle(monkeypatch, cfg, precision, kind_b, depth_b)
    replay = b.replay_steps() if running else 0
    fields = pushes(a, cut + replay + 45)
    for sb in (a, own):
        for u in fields[:cut]:
            sb.push(u)
    snap = a.save_running_state() if running else a.save_state()
    (b.load_running_state if running else b.load_state)(snap)
    for u in fields[cut:cut + replay]:
        own.push(u)
        b.push(u)
    for x, y in zip(steps(b, fields[cut + replay:]), steps(own, fields[cut + replay:])):
        assert torch.equal(x, y)


def test_snapshot_without_a_mark_where_one_lag_is_all(monkeypatch):
    """Quasi-dynamic handles kept their modes by wavenumber, then by bin."""
    n1, n3 = 16, 8
    cfg = dict(n1=n1, n3=n3, dx1=0.7, window_cap=1, window_mode="static", planes=TWO, input_kind="increment")
    sb = handle(monkeypatch, cfg, "fp64")
    fields = pushes(sb, 9)
    steps(sb, fields[:6])
    snap = sb.save_state()
    want = steps(sb, fields[6:])
    m1 = torch.arange(n1)
    k1 = (6.283185307179586 * torch.where(m1 < n1 // 2, m1, m1 - n1).double()) / (n1 * 0.7)
    k3 = (6.283185307179586 * torch.arange(n3 // 2 + 1).double()) / n3
    q = (k1[None, :] ** 2 + k3[:, None] ** 2).sqrt().reshape(-1).tolist()
    by_bin = sorted(range(len(q)), key=lambda b: (q[b] == 0, b))      # now
    by_q = sorted(range(len(q)), key=lambda b: (q[b] == 0, q[b], b))  # then
    old = torch.tensor([by_bin.index(b) for b in by_q], device=DEV)
    m, p, out = len(q), 2, 256 + 2 * 3 * len(q) * 16
    slots = sb.info()["sweep_depth"] + 1
    snap[8:256] = 0
    end = snap.numel() - slots * p * 5 * m * 16
    state = snap[end - p * 3 * m * 16:end].view(torch.float64).reshape(p * 3, m, 2)
    state.copy_(state[:, old].contiguous())
    # (the ring: one slot a block; blocks of a phase lie together, 80 modes make two)
    ring = snap[out:end - p * 3 * m * 16].view(torch.float64).reshape(-1, p, 3, 64, 2)
    flat = ring.permute(1, 2, 0, 3, 4).reshape(p, 3, -1, 2)[:, :, :m]
    pad = torch.zeros(p, 3, ring.shape[0] * 64, 2, dtype=torch.float64, device=DEV)
    pad[:, :, :m] = flat[:, :, old]
    ring.copy_(pad.reshape(p, 3, ring.shape[0], 64, 2).permute(2, 0, 1, 3, 4))
    sb.reset()
    sb.load_state(snap)
    got = steps(sb, fields[6:])
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    sb.close()


@pytest.mark.parametrize("change", [dict(n1=32), dict(window_cap=21), dict(planes=ONE)])
def test_snapshot_of_another_configuration_is_refused(change, monkeypatch):
    cfg = dict(n1=16, n3=16, window_cap=24, planes=TWO)
    a = handle(monkeypatch, cfg, "fp64")
    b = handle(monkeypatch, dict(cfg, **change), "fp64", "mfma")
    a.push(a.new_field().normal_())
    snap = torch.cat([a.save_state(), torch.zeros(1 << 22, dtype=torch.uint8, device=DEV)])
    with pytest.raises(SBIMError, match="another configuration"):
        b.load_state(snap)
    with pytest.raises(ValueError, match="too small"):
        a.load_state(snap[:a.state_bytes() - 256])
    assert b.info()["step"] == 0
