"""Collisions that outgrow a wave's queue, in every electron kernel that has
that path: a wave queues up to 128 collisions, and when a sub-chunk of 256 slots
brings more than there is room for, their particles are read back from memory.
The gas collides with 0.8 of the electrons in every step whatever their energy
(cross sections with constant collision frequencies), about 200 of a sub-chunk.
All is compared with the oracle bit for bit."""
import numpy as np
import pytest

import oracle
from paper_1508_02892_amd import hd, workloads as W
from test_parity_gpu import compare

pytestmark = pytest.mark.gpu

QUEUE = 128
STEPS = 19  # a sort among them


def _nu(fraction, dt=2e-14):
    """Cross section of constant frequency -ln(1 - fraction) / dt at 1 atm."""
    e = np.maximum(W.energy_grid(4096), 0.05)
    v = np.sqrt(2.0 * e * W.E_CHARGE / 9.1093837015e-31)
    return -np.log1p(-fraction) / dt / (W.N_GAS_1ATM * v)


def _above(sigma, threshold):
    return np.where(W.energy_grid(4096) > threshold, sigma, 0.0)


def _params(attach, precision, n, seed=1):
    s = _nu(0.8)
    if not attach:
        ch = [{"kind": "elastic", "threshold_eV": 0.0, "sigma_m2": 0.8 * s},
              {"kind": "excitation", "threshold_eV": 2.0, "sigma_m2": _above(0.1 * s, 2.0)},
              {"kind": "ionization", "threshold_eV": 15.0, "sigma_m2": _above(0.1 * s, 15.0)}]
        return W.small(precision=precision, n_cells=64, n_macro=n, t_e0_eV=25.0, channels=ch, seed=seed,
                       load_lo=0.0, load_hi=1.0)
    ch = [{"kind": "elastic", "threshold_eV": 0.0, "sigma_m2": 0.8 * s},
          {"kind": "attachment", "threshold_eV": 0.0, "sigma_m2": 0.04 * s, "product": 3},
          {"kind": "ionization", "threshold_eV": 12.0, "sigma_m2": _above(0.08 * s, 12.0), "product": 2},
          {"kind": "ionization", "threshold_eV": 24.6, "sigma_m2": _above(0.08 * s, 24.6), "product": 0}]
    return W.small_chem(precision=precision, n_cells=64, n_macro=n, t_e0_eV=25.0, channels=ch, seed=seed,
                        load_lo=0.0, load_hi=1.0)


NARROW, WIDE = (0, 1, 2, 3, 4, 5, 6), (8, 10, 11, 12, 13, 14)


@pytest.mark.parametrize("attach", [False, True], ids=["three channels", "attachment"])
@pytest.mark.parametrize("precision,variant", [(0, v) for v in NARROW + WIDE] + [(1, v) for v in NARROW])
def test_more_collisions_than_the_queue_holds(attach, precision, variant):
    p = _params(attach, precision, 11 * 256 + 77)
    orc = oracle.Oracle(p, contract=True)
    most, before = 0.0, np.zeros(len(p["channels"]))
    for _ in range(STEPS):
        blocks = -(-len(orc.particles()["cell"]) // 256)
        orc.step(1)
        now = np.asarray(orc.counters()["coll"], float)[:len(before)]
        most = max(most, (now - before).sum() / blocks)
        before = now
    assert most > QUEUE  # some sub-chunk of that step has more than the average
    if attach:
        assert before[1] > 0
    # one workgroup, so that its waves enter sub-chunks with entries queued; as
    # many as there are sub-chunks
    for groups in (1, 0):
        dev = hd.Discharge(p)
        dev.set_launch({"electron_variant": variant, "electron_groups": groups})
        dev.step(STEPS)
        compare(dev.moments(), dev.particles(), orc)
        dev.close()
