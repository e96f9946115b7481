"""What the autotuner's key tells apart: batches that run different kernels, and
choices that were kept by a library which divided the work in another way."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

CHILD = """
import json, sys
sys.path.insert(0, sys.argv[2])
from paper_1508_02892_amd import hd, workloads as W
kw = dict(n_cells=128, n_macro=20000, capacity=60000)
three = W.he_channels()
out = []
for second in (three, three[:2]):
    d = hd.Batch([W.small(channels=ch, **kw) for ch in (three, second)])
    out.append(d.autotune(32) if sys.argv[1] == "tune" else d.get_launch())
    d.close()
print(json.dumps(out))
"""


def _child(mode, cache):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CHILD, mode, root], capture_output=True, text=True,
                       timeout=240, env=dict(os.environ, HD_TUNE_CACHE=str(cache)))
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.strip().splitlines()[-1])


def test_kernels_and_division_are_in_the_key(tmp_path):
    cache = tmp_path / "tune.txt"
    default = _child("fresh", cache)
    _child("tune", cache)
    keys = [line.split()[0] for line in cache.read_text().splitlines()]
    assert len(keys) == 2 and keys[0] != keys[1]  # three channels each, or three and two
    # a line whose key ends at the ion models, as it did before the kernels were
    # told apart and the division of work was changed
    old = keys[0][:keys[0].index("/q")]
    cache.write_text("%s 1 77 333 5 8192\n" % old)
    assert _child("fresh", cache) == default
    cache.write_text("%s 1 77 333 5 8192\n" % keys[0])
    fresh = _child("fresh", cache)
    assert fresh[0] == {"electron_variant": 1, "electron_groups": 77, "sort_groups": 333,
                        "append_groups": 5, "sort_tile": 8192}
    assert fresh[1] == default[1]
