"""GPU: the strip's corrector over its ways of splitting the node layers among threads.

A periodic field that repeats a small tile has the same solution on the tile alone, so a strip on
the large grid (several layers a thread, wavefronts inside one run of layers) is compared with the
oracle-checked strip on its tile (one layer a thread; 4 x 4 and 4 x 8 cells: wavefronts over several
layers).  The two differ by transforms of different length: the bar is that of the
comparison with the oracle, 1e-12 of each field's largest value in float64, identical sliding sets.
"""
import numpy as np
import pytest
import torch

import workloads
from paper_2102_08756_amd import SBIM, Config, Strip

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
T = workloads.TPV3
A = (T["rho"], T["cp"], T["cs"])
B = (T["rho"], 0.7 * T["cp"], 0.7 * T["cs"])
STEPS = 12


def run(tile, grid, above, below):
    m1, m3 = tile
    rng = np.random.default_rng(5)
    tau0 = np.stack([65e6 + 20e6 * rng.random(tile), -120e6 + 5e6 * rng.random(tile),
                     10e6 * rng.random(tile)])
    prm = [tau0, np.full(tile, 0.677), np.full(tile, 0.525), np.full(tile, 0.4)]
    rep = (grid[0] // m1, grid[1] // m3)
    prm = [torch.tensor(np.tile(p, rep if p.ndim == 2 else (1,) + rep), device=DEV) for p in prm]
    dx = 100.0
    up = dict(side=1, mu=T["rho"] * T["cs"] ** 2, cs=T["cs"], cp=T["cp"])
    cfg = Config.from_dict(dict(n1=grid[0], n3=grid[1], dx1=dx, dx3=dx, dt=0.3 * dx / T["cp"],
                                planes=[up, dict(up, side=-1)] if below else [up],
                                window_cap=STEPS, window_mode="fixed", input_kind="absolute"),
                           precision="fp64")
    sb = SBIM(cfg, device=DEV)
    s = Strip(sb, above, *prm, layers_below=below)
    tau, rate = s.run(STEPS)
    out = dict(tau=tau, rate=rate, u=s.read("displacement"), slip=s.read("slip"),
               sliding=s.read("sliding"))
    out = {k: v.cpu() for k, v in out.items()}
    s.close()
    sb.close()
    return out


@pytest.mark.parametrize("tile,grid,above,below", [
    ((4, 4), (16, 16), [A], []),                       # 2 node layers: one run of any depth
    ((4, 8), (8, 64), [A, B, A], [A, B]),              # 7 node layers, rows over a wavefront's end
    ((16, 16), (256, 256), [A, B], [B]),               # 5 node layers in runs of 1
    ((16, 16), (256, 512), [B, A, A, A], []),          # 5 node layers in runs of 4
    ((8, 8), (256, 256), [B, A, A], [A, A, B]),        # 8 node layers in runs of 2
])
def test_large_grid_repeats_its_tile(tile, grid, above, below):
    ref = run(tile, tile, above, below)
    got = run(tile, grid, above, below)
    rep = (grid[0] // tile[0], grid[1] // tile[1])
    assert ref["sliding"].any() and not ref["sliding"].all()
    for k, r in ref.items():
        want = r.repeat(*([1] * (r.ndim - 2)), *rep)
        err = float((got[k] - want).abs().max() / want.abs().max())
        print(f"[strip] {tile} on {grid}: {k} {err:.1e}", flush=True)
        assert err < (1e-12 if k != "sliding" else 1e-300), k
