"""GPU: transforms of fields that one work-group holds in LDS, at the edges of that range.

The same field repeated on a grid past the range has the transform of the tile at the tile's bins,
so the pushed displacement's tractions on the small grid are compared with the oracle and, repeated,
with the larger grid's two-kernel transforms.  Bars: 1e-12 relative L2 in float64 and 1e-5 in the
float32 forms, as for the library's other comparisons with the oracle.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2102_08756_amd import SBIM, Config

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BAR = {"fp64": 1e-12, "fp32": 1e-5, "fp32_comp": 1e-5}


def run(cfg, u, precision):
    sb = SBIM(Config.from_dict(cfg, precision=precision), device=DEV)
    far = torch.linspace(-1.0, 1.0, u[0].size, dtype=torch.float64).reshape(u[0].shape)
    far = far.to(sb.dtype).to(DEV)
    out = []
    for n in range(len(u)):
        sb.push(torch.tensor(u[n], dtype=sb.dtype, device=DEV))
        out.append((sb.tractions(far) - far).double().cpu().numpy())
    sb.close()
    return np.stack(out)


def rel_l2(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


# the smallest, the longest rows and columns, the largest in float64 (64 x 33 points) and in float32
# (64 x 65 and 128 x 33), and grids just past the range
@pytest.mark.parametrize("n1,n3", [(4, 4), (4, 256), (512, 4), (8, 64), (64, 64), (32, 128),
                                   (128, 32), (64, 128), (128, 64), (4, 2048), (1024, 4)])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_comp"])
def test_small_fields(n1, n3, precision):
    cfg = dict(n1=n1, n3=n3, window_cap=3, planes=[dict(side=1), dict(side=-1, cs=1.2, cp=2.5)])
    u = np.random.default_rng(n1 + 7 * n3).standard_normal((3, 2, 3, n1, n3))
    err = rel_l2(run(cfg, u, precision), oracle.forward(cfg, u))
    print(f"[fft] {n1} x {n3} {precision}: {err:.1e}", flush=True)
    assert err < BAR[precision]


@pytest.mark.parametrize("n1,n3,rep", [(4, 4, (64, 64)), (64, 64, (4, 2)), (16, 128, (16, 2))])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_repeated_field_has_the_tile_s_tractions(n1, n3, rep, precision):
    cfg = dict(n1=n1, n3=n3, window_cap=3, planes=[dict(side=1)])
    u = np.random.default_rng(3).standard_normal((3, 1, 3, n1, n3))
    small = run(cfg, u, precision)
    big = run(dict(cfg, n1=n1 * rep[0], n3=n3 * rep[1]), np.tile(u, (1, 1, 1) + rep), precision)
    assert rel_l2(big, np.tile(small, (1, 1, 1) + rep)) < BAR[precision]
