"""Releasing a handle whose device state lies in the caller's arena waits for its
own stream, not for the work of others on the device."""
import time

import numpy as np
import pytest
import torch

from paper_1508_02892_amd import hd, workloads as W

pytestmark = pytest.mark.gpu


def test_free_does_not_wait_for_other_streams():
    p = W.small(n_cells=64, n_macro=3000)
    arena = torch.empty(hd.required_bytes(p), dtype=torch.uint8, device="cuda")
    busy = hd.Discharge(W.base_params(precision=W.FP32, n_cells=2048, gap_m=1e-3, n_macro=1 << 22))
    busy.step(64)
    busy.moments()
    steps, took, freed = 4000, 0.0, 1.0
    for _ in range(2):  # the first time round also allocates what later handles reuse
        a = hd.Discharge(p, arena=arena)
        a.step(20)
        want = a.moments()["n_live"]
        assert want > 0
        t0 = time.perf_counter()
        busy.step(steps)
        t1 = time.perf_counter()
        a.close()
        freed = time.perf_counter() - t1
        busy.moments()
        took = time.perf_counter() - t0
    busy.close()
    assert took > 0.05 and freed < 0.25 * took, (freed, took)


def test_kept_buffers_serve_later_handles():
    # buffers of freed arena handles, more of them than are kept, then larger
    # and smaller read-outs in turn
    small, large = W.small(n_cells=16, n_macro=50), W.small(n_cells=300, n_macro=50, n_eedf_bins=5000)
    for n, p in ((70, small), (3, large), (5, small), (12, large)):
        need = (hd.required_bytes(p) + 255) // 256 * 256
        arena = torch.empty(n * need, dtype=torch.uint8, device="cuda")
        ds = [hd.Discharge(p, arena=arena[i * need:(i + 1) * need]) for i in range(n)]
        ref = hd.Discharge(p)
        for d in ds + [ref]:
            d.step(3)
        want = ref.moments()
        for d in ds:
            got = d.moments()
            for k in ("cnt", "phi", "n_i", "eedf_counts"):
                np.testing.assert_array_equal(got[k], want[k])
        for d in ds:
            d.close()
        if n == 3:
            ref.close()  # waits, and frees what is kept
