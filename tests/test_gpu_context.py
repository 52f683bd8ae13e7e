"""A context made after another one uses its device memory again: results are
those of a context that starts from nothing, whatever ran before, and close()
gives the memory back.  Fixed-point deposits: no tolerance."""
import ctypes as C

import numpy as np
import pytest

import gv_inputs

pytestmark = pytest.mark.gpu


def _free_bytes():
    lib = C.CDLL("libamdhip64.so.7")
    free, total = C.c_size_t(), C.c_size_t()
    assert lib.hipMemGetInfo(C.byref(free), C.byref(total)) == 0
    return free.value


# detector, primaries, configuration: queues of other sizes and precisions, the
# plain driver, the integration queue, more cells than the context before
def _runs(gv):
    slab = lambda layers: gv_inputs.slab_calorimeter(layers)
    return [
        ("slab", slab(10), gv_inputs.mixed_beam(200, 3, 30.0, 300.0), dict(precision=gv.PMIX)),
        ("plate", gv_inputs.single_slab("Pb", 0.2), gv_inputs.beam(500, 11, 10.0), dict(precision=gv.PMIX)),
        ("deep", slab(30), gv_inputs.mixed_beam(300, 4, 30.0, 300.0), dict(precision=gv.P64)),
        ("plain", slab(5), gv_inputs.mixed_beam(20, 5, 30.0, 300.0),
         dict(driver=gv.DRIVER_PLAIN, precision=gv.P64, capacity=1 << 18)),
        ("rk45", gv_inputs.barrel(field_map=gv_inputs.MAP_SOLENOID), gv_inputs.barrel_beam(20, 6, 300.0),
         dict(precision=gv.PMIX, field_method=gv.FIELD_RK45)),
        ("small queues", slab(10), gv_inputs.mixed_beam(50, 7, 30.0, 300.0),
         dict(precision=gv.PMIX, capacity=1 << 16)),
    ]


def _one(gv, run):
    _, geom, prim, cfg = run
    eng = gv.Engine(geom, deposit_mode=gv.DEPOSIT_FIXED, **cfg)
    assert not eng.escape_hist().any()
    edep = eng.transport(prim, 42)
    s = eng.stats()
    return np.asarray(edep).copy(), [list(s["steps"]), list(s["tracks"]), s["escaped"]], eng


def test_context_after_context_equals_a_first_one():
    import paper_2005_00949_amd as gv
    runs = _runs(gv)
    first = []
    for run in runs:
        edep, stats, eng = _one(gv, run)
        eng.close()
        first.append((edep, stats))
    free0 = _free_bytes()
    for order in ([0, 1, 2, 3, 4, 5], [5, 0, 4, 3, 2, 1, 1]):
        for k in order:
            edep, stats, eng = _one(gv, runs[k])
            assert np.array_equal(edep, first[k][0]), runs[k][0]
            assert stats == first[k][1], runs[k][0]
    eng.close()
    assert _free_bytes() >= free0 - (64 << 20)
