"""Which kernels a transport without knobs runs: the pool kernel alone on small
populations, the step kernel's graph on those that fill the GPU, and secondaries that
find no free slot in a pool queued instead.  With an explicit knob the step kernel
runs throughout; that both give the same bits is checked beside."""
import os
import re
import subprocess
import sys

import numpy as np
import pytest

import gv_inputs
from test_gpu_pool import CASES, KEYS

pytestmark = pytest.mark.gpu
KNOBS = dict(basket=256, occupancy=3, inner_steps=4)
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("case", list(CASES))
def test_kernels_that_ran(case):
    import paper_2005_00949_amd as gv
    make, cfg = CASES[case]
    geom, prim = make()
    replays = []
    for knobs in ({}, KNOBS):
        eng = gv.Engine(geom, deposit_mode=gv.DEPOSIT_FIXED, max_steps_per_track=20_000, **cfg, **knobs)
        eng.transport(prim, 0x9003)
        replays.append(eng.stats()["graph_replays"])
        eng.close()
    assert (replays[0] > 0) == case.startswith("slab_bulk"), replays
    assert replays[1] > 0


def spill(precision):
    """Run in a process of its own, whose library prints each launch."""
    import paper_2005_00949_amd as gv
    geom, prim = gv_inputs.single_slab("Pb", 100.0), gv_inputs.beam(4000, 22, 3.0e3)
    out = []
    for knobs in (KNOBS, {}):
        eng = gv.Engine(geom, deposit_mode=gv.DEPOSIT_FIXED, precision=getattr(gv, precision), **knobs)
        e = np.asarray(eng.transport(prim, 11))
        st = eng.stats()
        out.append((e, eng.ledger(), eng.escape_hist(), [st[k] for k in KEYS]))
        eng.close()
    a, b = out
    assert a[3] == b[3]
    assert all(np.array_equal(x, y) for x, y in zip(a[:3], b[:3]))
    print("same bits")


@pytest.mark.parametrize("precision", ["PMIX", "P64"])
def test_secondaries_without_a_slot(precision):
    """4,000 showers in a block of lead: a launch begins with some 40 tracks in each
    pool of 192 slots and multiplies them tenfold."""
    code = (f"import sys; sys.path[:0] = [{ROOT!r}, {os.path.join(ROOT, 'tests')!r}]; "
            f"import test_gpu_pool_paths as t; t.spill({precision!r})")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100,
                       env=dict(os.environ, GV_PROGRESS="1"))
    assert r.returncode == 0 and "same bits" in r.stdout, r.stderr[-2000:]
    spilled = [int(x) for x in re.findall(r"\[gv\] pool.*spilled (\d+)", r.stderr)]
    print(f"\n[{precision}] secondaries queued per pair of launches: {spilled}")
    assert sum(spilled) > 0
