"""GPU: which sweep a configuration is planned with (its window against its grid).

One window for every mode: the matrix-core form from the windows where it is the faster one.  The
sizes are either side of each bound of the rule.
"""
import pytest

from paper_2102_08756_amd import SBIM, Config

pytestmark = pytest.mark.gpu
ONE = [dict(side=1)]
TWO = [dict(side=1), dict(side=-1)]
BIMATERIAL = [dict(side=1), dict(side=-1, cs=1.2, cp=2.5)]

CASES = [
    # grids that do not fill the chip: from 64 lags (and modes x lags past 2^18)
    (256, 256, 1.0, ONE, "fp64", 63, 0), (256, 256, 1.0, ONE, "fp64", 64, 1),
    (512, 256, 1.0, ONE, "fp64", 95, 0), (256, 512, 1.3, ONE, "fp64", 96, 1),
    (512, 256, 1.0, ONE, "fp32", 64, 1),
    # square grids that do
    (512, 512, 1.0, ONE, "fp64", 111, 0), (512, 512, 1.0, BIMATERIAL, "fp64", 112, 1),
    (512, 512, 1.0, ONE, "fp32", 79, 0), (512, 512, 1.0, ONE, "fp32", 80, 1),
    (512, 512, 1.0, ONE, "fp32_comp", 64, 1), (512, 512, 1.0, TWO, "fp32", 64, 1),
    # two modes a kernel row, few and many sharing their q
    (512, 512, 1.3, ONE, "fp32", 131, 0), (512, 512, 1.3, ONE, "fp32_comp", 132, 1),
    (512, 512, 1.3, TWO, "fp64", 159, 0), (512, 512, 1.3, TWO, "fp64", 160, 1),
    (1024, 512, 1.0, ONE, "fp64", 255, 0), (512, 1024, 1.0, BIMATERIAL, "fp64", 256, 1),
    (1024, 512, 1.0, TWO, "fp64", 383, 0), (1024, 512, 1.0, TWO, "fp64", 384, 1),
]


@pytest.mark.parametrize("n1,n3,dx3,planes,precision,window,matrix", CASES)
def test_sweep_form_of_a_configuration(n1, n3, dx3, planes, precision, window, matrix, monkeypatch):
    for k in ("KIND", "DEPTH", "CHUNKS", "QUADS"):
        monkeypatch.delenv("SBIM_SWEEP_" + k, raising=False)
    sb = SBIM(Config.from_dict(dict(n1=n1, n3=n3, dx3=dx3, window_cap=window, planes=planes),
                               precision=precision), device="cuda:0")
    info = sb.info()
    sb.close()
    assert info["sweep_matrix_cores"] == matrix
