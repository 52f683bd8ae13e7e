"""A context whose predecessor left device memory behind finds room beside other
users of the card: what the predecessor kept (deposit buffers as large as its events
times cells, queues) goes before a call fails for want of memory.  The card is
filled, but for 4 GiB, by an allocation that nothing touches; results are those of an
empty card (fixed-point deposits: no tolerance)."""
import ctypes as C

import numpy as np
import pytest

import gv_inputs

pytestmark = pytest.mark.gpu
GIB = 1 << 30


@pytest.fixture
def hip():
    lib = C.CDLL("libamdhip64.so.7")
    lib.hipMalloc.argtypes = [C.POINTER(C.c_void_p), C.c_size_t]
    lib.hipFree.argtypes = [C.c_void_p]
    return lib


def _free(hip):
    free, total = C.c_size_t(), C.c_size_t()
    assert hip.hipMemGetInfo(C.byref(free), C.byref(total)) == 0
    return free.value


def _wide_context(gv, hip):
    """A context that ran with 16 GiB of deposits (1,024 events x 2^21 cells), 12 GB of
    queues."""
    geom = gv_inputs.single_slab("Pb", 0.2)
    geom["cell"] = np.array([(1 << 21) - 1], dtype=np.int32)
    geom["n_cells"] = 1 << 21
    out = C.c_void_p()
    assert hip.hipMalloc(C.byref(out), 16 * GIB) == 0
    eng = gv.Engine(geom, edep_on_device=1)
    eng.transport(gv_inputs.beam(1024, 11, 10.0), 1, edep_out=out.value)
    assert hip.hipFree(out) == 0


def _fill(hip, leave):
    p = C.c_void_p()
    assert hip.hipMalloc(C.byref(p), _free(hip) - leave) == 0
    return p


def _small(gv, **cfg):
    eng = gv.Engine(gv_inputs.slab_calorimeter(10), deposit_mode=gv.DEPOSIT_FIXED, **cfg)
    e = np.asarray(eng.transport(gv_inputs.mixed_beam(200, 3, 30.0, 300.0), 42)).copy()
    return eng, e


@pytest.mark.parametrize("precision", ["PMIX", "P64"])
def test_queues_find_room_beside_kept_deposits(hip, precision):
    import paper_2005_00949_amd as gv
    cfg = dict(precision=getattr(gv, precision), capacity=3 << 24)   # 18 or 23 GB of queues
    eng, want = _small(gv, **cfg)
    eng.close()
    _wide_context(gv, hip)
    block = _fill(hip, 4 * GIB)
    try:
        eng, got = _small(gv, **cfg)
        assert np.array_equal(got, want)
        again = np.asarray(eng.transport(gv_inputs.mixed_beam(200, 3, 30.0, 300.0), 42))
        assert np.array_equal(again, want)
    finally:
        assert hip.hipFree(block) == 0
        eng.close()


def test_a_call_that_finds_no_room_fails_alone(hip):
    """Queues of 2^30 slots have no room on any card; the next call succeeds."""
    import paper_2005_00949_amd as gv
    eng, want = _small(gv)
    eng.configure(capacity=1 << 30)
    prim = gv_inputs.mixed_beam(200, 3, 30.0, 300.0)
    with pytest.raises(gv.GvError, match="out of memory"):
        eng.transport(prim, 42)
    eng.configure(capacity=0)
    assert np.array_equal(np.asarray(eng.transport(prim, 42)), want)
    eng.close()
