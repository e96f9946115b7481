"""The electron launch's division of work against the oracle, bit for bit, at
its edges: sub-chunks of 256 slots with one slot more or less, collisions so
frequent that a sub-chunk's selected electrons do not fit their wave's queue
at once, more sub-chunks in one workgroup than their child counts have room
for in its LDS, more discharges than workgroups or than lanes of a wave, and
each kind of batch that has kernels of its own.
"""
import numpy as np
import pytest

import oracle
from paper_1508_02892_amd import hd, workloads as W
from test_parity_gpu import compare

pytestmark = pytest.mark.gpu

SUB = 256  # slots of a sub-chunk


def _p(n, model=W.ION_DD, precision=0, **kw):
    # hot electrons that ionize, reach both walls and are emitted from them
    return W.small(precision=precision, ion_model=model, n_cells=64, n_macro=n, t_e0_eV=50.0,
                   v_amp_V=2000.0, phase_rad=np.pi / 2, gamma_see=1.0, load_lo=0.0, load_hi=1.0,
                   mu_const=8e-3, **kw)


def _dense(n, model, precision):
    # a collision event is drawn for nearly every electron each step: what a
    # sub-chunk selects often finds no room in its wave's queue of 128
    p = _p(n, model, precision, n_gas_m3=20 * W.N_GAS_1ATM)
    o = oracle.Oracle(p, contract=True)
    assert o.derived()["Pmax"] > 0.6
    return p


_MANY = [_p(n, (W.ION_DD, W.ION_FULL)[i % 2], seed=100 + i)
         for i, n in enumerate((7 * k * k) % 1500 + 1 for k in range(70))]

CASES = (
    # (name, discharges, launch shape)
    [("edge of a sub-chunk %d" % n, [_p(n)], {}) for n in (1, SUB - 1, SUB, SUB + 1, 9 * SUB + 3)]
    + [("dense %d %d v%d" % (pr, m, v), [_dense(8 * SUB + 77, m, pr)], {"electron_variant": v})
       for pr, m, v in ((0, W.ION_DD, 0), (0, W.ION_FULL, 7), (0, W.ION_DD, 8), (1, W.ION_FULL, 1),
                        (1, W.ION_DD, 0))]
    + [("one workgroup of 548 sub-chunks", [_p(140_000)], {"electron_groups": 1, "electron_variant": v})
       for v in (0, 8)]
    + [("70 discharges on %d workgroups" % g, _MANY, {"electron_groups": g}) for g in (1, 3, 70, 100)]
    + [("one kind in a batch", [_p(n, m, seed=n) for n in (300, 5000, 1)], {"electron_groups": g})
       for m in (W.ION_DD, W.ION_FULL) for g in (0, 2)]
)


@pytest.mark.parametrize("name,ps,cfg", CASES, ids=[c[0] for c in CASES])
def test_work_split(name, ps, cfg):
    b = hd.Batch(ps)
    b.set_launch(cfg)
    b.step(3)
    b.step(16)
    for i in range(0, len(ps), max(1, len(ps) // 8)):
        orc = oracle.Oracle(ps[i], contract=True)
        orc.step(19)
        compare(b.moments(i), b.particles(i), orc)
    b.close()


@pytest.mark.parametrize("small,precision,groups", [(130, 0, 64), (700, 1, 0)],
                         ids=["several rounds of ranges", "more discharges than workgroups"])
def test_one_large_discharge_among_many(small, precision, groups):
    # ranges shorter than the large discharge and more of them than workgroups
    ps = [_p(1 + i % 300, seed=200 + i, precision=precision) for i in range(small)]
    ps.insert(small // 2, _p(60_000, precision=precision, seed=9))
    b = hd.Batch(ps)
    b.set_launch({"electron_groups": groups})
    b.step(19)
    for i in (0, small // 2, small):
        orc = oracle.Oracle(ps[i], contract=True)
        orc.step(19)
        compare(b.moments(i), b.particles(i), orc)
    b.close()


@pytest.mark.parametrize("cells", [9, 17, 130, 257, 449, 450, 453, 705, 4096])
def test_partitioned_solve_at_the_edges_of_its_batches(cells):
    # partitions whose rows (less the three that start and end a sweep) are a
    # multiple of the sweeps' batch, or one more or less
    p = W.small(precision=1, ion_model=W.ION_FULL_FIT, n_cells=cells, gap_m=0.5e-3, n_macro=20000,
                load_lo=0.0, load_hi=1.0)
    dev, orc = hd.Discharge(p), oracle.Oracle(p, contract=True)
    dev.step(5)
    orc.step(5)
    compare(dev.moments(), dev.particles(), orc)
    dev.close()
