"""The electron launch's LDS at its limits."""
import pytest

import oracle
from paper_1508_02892_amd import hd, workloads as W
from test_parity_gpu import compare

pytestmark = pytest.mark.gpu


def test_a_variant_that_does_not_fit_leaves_no_error():
    # FP64 on the largest grid with 8,000 EEDF bins needs more LDS than a
    # workgroup has; FP32 with 16,400 fits a narrow workgroup but not a wide one
    p = W.small(precision=W.FP64, n_cells=4096, gap_m=2e-3, n_macro=3000)
    for bins in (8000, 5900):
        with pytest.raises(hd.HdError):
            hd.Discharge(dict(p, n_eedf_bins=bins))
    for q in (p, dict(p, precision=W.FP32, n_eedf_bins=16400)):
        dev, orc = hd.Discharge(q), oracle.Oracle(q, contract=True)
        dev.step(17)
        orc.step(17)
        compare(dev.moments(), dev.particles(), orc)
        dev.close()
