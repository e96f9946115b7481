"""The electron launch's LDS at its limits: the largest histograms that fit a
workgroup beside the largest grid, and the full fluid's arrays lying over the
table of ranges where both together would cost a workgroup per CU."""
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


LDS = 160 << 10  # bytes of a workgroup


def _al(x):
    return (x + 15) // 16 * 16


def _bins_that_fit(precision, nodes, D):
    """EEDF bins (with one for the energies beyond) that fill the LDS: 1,024
    rows of three channels, E' and the deposit grid at the nodes, eight queues
    of 128 collisions, counters, child counts, D + 1 words for the division of
    work and eight of the scan."""
    real, entry = ((4, 32), (8, 48))[precision]
    used = (_al(1024 * 3 * real) + _al(nodes * real) + _al(nodes * 8) + 8 * 128 * entry + 96 + 1024
            + _al((D + 1) * 4) + 32)
    return (LDS - used) // 16 * 4 - 1


@pytest.mark.parametrize("precision,D", [(W.FP64, 1), (W.FP64, 3), (W.FP32, 1), (W.FP32, 2)])
def test_largest_histogram(precision, D):
    bins = _bins_that_fit(precision, 4097, D)
    ps = [W.small(precision=precision, n_cells=4096, gap_m=2e-3, n_macro=3000 + 700 * i, t_e0_eV=20.0,
                  n_eedf_bins=bins, load_lo=0.0, load_hi=1.0) for i in range(D)]
    b = hd.Batch(ps)
    b.step(17)
    for i in range(D):
        orc = oracle.Oracle(ps[i], contract=True)
        orc.step(17)
        compare(b.moments(i), b.particles(i), orc)
    b.close()
    with pytest.raises(hd.HdError):
        hd.Batch([dict(p, n_eedf_bins=bins + 4) for p in ps])


@pytest.mark.parametrize("precision,cells,groups", [
    # the fluid takes 4 nodes + 896 doubles: on 2,304 nodes half a CU's LDS
    # less 1 KB, so that the table of ranges does not fit beside it
    (W.FP32, 2303, 0), (W.FP32, 2303, 1), (W.FP32, 2303, 4096), (W.FP64, 2303, 0), (W.FP32, 2302, 1),
])
def test_fluid_over_the_table_of_ranges(precision, cells, groups):
    ps = [W.small(precision=precision, ion_model=W.ION_FULL, n_cells=cells, gap_m=1e-3, seed=3 + i,
                  n_macro=n, t_e0_eV=20.0, load_lo=0.0, load_hi=1.0)
          for i, n in enumerate((1, 300, 9000, 2, 30011, 257, 5))]
    b = hd.Batch(ps)
    b.set_launch({"electron_groups": groups})
    b.step(19)
    for i in (0, 1, 4, 6):
        orc = oracle.Oracle(ps[i], contract=True)
        orc.step(19)
        compare(b.moments(i), b.particles(i), orc)
    b.close()


def test_fluid_over_the_table_of_one_discharge():
    # 4,097 units of work on the most workgroups there can be: no more ranges
    # than a discharge has room for the totals of
    nodes = 2304
    fluid = nodes // 32 + 4
    p = W.small(precision=W.FP32, ion_model=W.ION_FULL, n_cells=nodes - 1, gap_m=1e-3, t_e0_eV=20.0,
                n_macro=256 * (4097 - fluid), load_lo=0.0, load_hi=1.0, capacity=256 * 4200)
    dev, orc = hd.Discharge(p), oracle.Oracle(p, contract=True)
    dev.set_launch({"electron_groups": 4096})
    dev.step(5)
    orc.step(5)
    compare(dev.moments(), dev.particles(), orc)
    dev.close()
