"""Read-out of moments: every array equal to the oracle's whatever else is
asked for, on the smallest and largest grids and with several species."""
import ctypes as C

import numpy as np
import pytest

import oracle
from paper_1508_02892_amd import hd, workloads as W
from test_parity_gpu import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [
    W.small(n_cells=2, n_macro=300, load_lo=0.0, load_hi=1.0),
    W.small(precision=W.FP32, n_cells=4096, n_macro=5000, n_eedf_bins=1),
    W.small_chem(n_cells=255, n_macro=3001, n_eedf_bins=1000),
], ids=["2-cells", "4096-cells", "species"])
def test_each_array_alone_and_all_together(p):
    dev, orc = hd.Discharge(p), oracle.Oracle(p, contract=True)
    dev.step(17)
    orc.step(17)
    whole, g = dev.moments(), orc.grid()
    for k in ("cnt", "phi", "E", "n_e"):
        np.testing.assert_array_equal(whole[k], g[k], err_msg=k)
    np.testing.assert_array_equal(whole["eedf_counts"], orc.accum()["eedf"])
    S = max(1, len(p.get("species", [])))
    for s in range(S if p.get("species") else 0):
        o = orc.species(s)
        nn = p["n_cells"] + 1
        np.testing.assert_array_equal(whole["n_species"][s * nn:(s + 1) * nn], o["n"])
    for k in hd._Moments._ARRS:
        M = hd._Moments(p["n_cells"] + 1, p["n_eedf_bins"], len(p["channels"]), S)
        for other in hd._Moments._ARRS:
            if other != k:
                setattr(M.m, other, None)
        hd._check(hd.lib().hd_moments(dev.h, C.byref(M.m)))
        np.testing.assert_array_equal(M.arrs[k], whole[k], err_msg=k)
        assert M.m.n_live == whole["n_live"] and M.m.pushed == whole["pushed"]
        assert all(not M.arrs[o].any() for o in hd._Moments._ARRS if o != k)


@pytest.mark.parametrize("p", [
    W.small(n_cells=2, n_macro=300, load_lo=0.0, load_hi=1.0),
    W.small(precision=W.FP32, n_cells=4096, n_macro=5000, n_eedf_bins=1),
    W.small_chem(n_cells=255, n_macro=3001, n_eedf_bins=1000),
], ids=["2-cells", "4096-cells", "species"])
def test_every_array_equals_the_oracle(p):
    # the arrays that the test above compares with a second read-out only: n_i,
    # the fluxes, the averages and the normalised EEDF
    dev, orc = hd.Discharge(p), oracle.Oracle(p, contract=True)
    dev.step(17)
    orc.step(17)
    m = dev.moments()
    compare(m, dev.particles(), orc)
    assert m["n_acc"] > 0
    counts = np.asarray(orc.accum()["eedf"], float)
    within = counts[:-1].sum()
    assert within > 0
    width = p["eedf_emax_eV"] / p["n_eedf_bins"]
    # a product and two quotients, each rounded once
    np.testing.assert_allclose(m["eedf"], counts[:-1] / (within * width), rtol=4 * 2.2e-16)
