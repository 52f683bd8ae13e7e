"""The pool kernel (stage baskets in LDS, for populations too small to fill the
GPU) against the step kernel, which a transport with an explicit knob uses.

Both run the same stage functions on the same states and draw random numbers
keyed by (event, track, step), so fixed-point deposits and ledgers, every
counter and the escape histogram are equal bit for bit: no tolerance.  Sizes
lie around a wavefront (64 tracks), a workgroup (256) and the pool's slots, and
on both sides of the population where the step kernel takes over."""
import numpy as np
import pytest

import gv_inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gv():
    import paper_2005_00949_amd
    paper_2005_00949_amd.load()
    return paper_2005_00949_amd


KEYS = ("steps", "tracks", "interactions", "escaped", "killed", "rejection_exhausted", "rk_substeps", "rk_rejected")


def _slab(n, field=0.0, layers=10):
    geom = gv_inputs.slab_calorimeter(layers, (0.0, field, 0.0))
    return geom, gv_inputs.mixed_beam(n, 0x9001 + n, 30.0, 300.0)


def _barrel(n, field_map=gv_inputs.MAP_UNIFORM):
    geom = gv_inputs.barrel(field_map=field_map)
    p = gv_inputs.barrel_beam(n, 0x9002 + n, 300.0)
    p["pdg"] = np.array([11, -11, 22], dtype=np.int32)[np.arange(n) % 3]
    return geom, p


def _plate(n):
    return gv_inputs.single_slab("Pb", 0.2), gv_inputs.beam(n, 11, 10.0)


def _edges(n):
    """Below the tracking cut, outside the world, at rest for an e+, along B."""
    geom, p = _slab(n, 4.0)
    p["ekin"][0::5] = 0.05
    p["pos"][1::5] = (0.0, 0.0, -50.0)
    p["pos"][2::5] = (25.0, 0.0, 4.0)
    p["dir"][3::5] = (0.0, 1.0, 0.0)
    return geom, p


CASES = {
    "slab1": (lambda: _slab(1), {}),
    "slab63": (lambda: _slab(63), {}),
    "slab65_field": (lambda: _slab(65, 4.0), {}),
    "slab257_tables": (lambda: _slab(257, 4.0), dict(fs_alias=31)),
    "slab_bulk": (lambda: (gv_inputs.slab_calorimeter(50), gv_inputs.beam(300, 11, 1.0e4)), {}),
    "slab_bulk_stable": (lambda: (gv_inputs.slab_calorimeter(50), gv_inputs.beam(300, 11, 1.0e4)),
                         dict(queue_order=1)),
    "edges": (lambda: _edges(130), {}),
    "plate": (lambda: _plate(3000), {}),
    "barrel": (lambda: _barrel(64), {}),
    "map": (lambda: _barrel(33, gv_inputs.MAP_SOLENOID), {}),
    "map_rk4": (lambda: _barrel(33, gv_inputs.MAP_SOLENOID), dict(field_method=1)),
    "map_rk45": (lambda: _barrel(33, gv_inputs.MAP_SOLENOID), dict(field_method=2)),
    "map_rk45_stable": (lambda: _barrel(33, gv_inputs.MAP_SOLENOID), dict(field_method=2, queue_order=1)),
}


@pytest.mark.parametrize("prec", ["p64", "pmix"])
@pytest.mark.parametrize("case", list(CASES))
def test_pool_equals_step_kernel(gv, case, prec):
    make, cfg = CASES[case]
    geom, prim = make()
    out = []
    for knobs in ({}, dict(basket=256, occupancy=3, inner_steps=4)):
        eng = gv.Engine(geom, precision=gv.P64 if prec == "p64" else gv.PMIX, deposit_mode=gv.DEPOSIT_FIXED,
                        max_steps_per_track=20_000, **cfg, **knobs)
        e = eng.transport(prim, 0x9003)
        st = eng.stats()
        out.append((e, eng.ledger(), eng.escape_hist(), [st[k] for k in KEYS], st))
        eng.close()
    a, b = out
    print(f"\n[{case} {prec}] steps {a[4]['total_steps']}, launches {a[4]['kernel_launches']} "
          f"(step kernel {b[4]['kernel_launches']})")
    assert a[3] == b[3]
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])
    # and the pool's own counters: never more steps than lanes offered
    assert 0 < a[4]["total_steps"] <= a[4]["lane_slots"]


def test_pool_windows(gv):
    """One event in flight per window gives what all in flight give."""
    geom, prim = _slab(40, 4.0)
    eng = gv.Engine(geom, precision=gv.PMIX, deposit_mode=gv.DEPOSIT_FIXED)
    ref, ref_l = eng.transport(prim, 7), eng.ledger()
    eng.configure(max_events_in_flight=1)
    assert np.array_equal(eng.transport(prim, 7), ref) and np.array_equal(eng.ledger(), ref_l)
