"""GPU: the strip's corrector with more than four node layers a thread, and layers that share a
stencil: a strip on a large grid repeats the one on its tile (bars of test_gpu_strip_columns)."""
import pytest

from test_gpu_strip_columns import A, B, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,above,below", [
    ((512, 512), [A] * 6, []),                           # 7 node layers in one run
    ((512, 512), [A] * 4, [A] * 4),                      # 10 in runs of 5, three stencils a side
    ((512, 512), [A, A, B, A, A, A], [B, B, A, A, A]),   # 13 in runs of 7 and 6
    ((256, 512), [A, B] * 8, []),                        # 17 in runs of 6, 6 and 5
])
def test_long_runs_and_shared_stencils(grid, above, below):
    ref = run((16, 16), (16, 16), above, below)
    got = run((16, 16), grid, above, below)
    assert ref["sliding"].any() and not ref["sliding"].all()
    for k, r in ref.items():
        want = r.repeat(*([1] * (r.ndim - 2)), grid[0] // 16, grid[1] // 16)
        err = float((got[k] - want).abs().max() / want.abs().max())
        print(f"[strip] {grid}: {k} {err:.1e}", flush=True)
        assert err < (1e-12 if k != "sliding" else 1e-300), k
