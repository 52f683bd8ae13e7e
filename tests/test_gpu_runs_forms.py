"""Runs of vacuum steps in the fields that no other test has: along no axis, along an
axis in the negative sense, along x in the barrel, and a bending tolerance so small
that a step may turn by less than the run's helix holds for (no run is taken then).
Against the same steps taken one by one, which a transport with a trace does: the
same expressions, no tolerance."""
import numpy as np
import pytest

import gv_inputs
from test_gpu_runs import KEYS, RK45, _barrel, _slab

pytestmark = pytest.mark.gpu


def _case(geom, prim, B, seed):
    """The primaries of test_gpu_runs turned to circle about B."""
    geom = dict(geom, B=np.array(B, dtype=np.float64))
    b = geom["B"] / np.linalg.norm(geom["B"])
    d = np.random.default_rng(seed).normal(size=(len(prim), 3))
    d -= (1.0 - 1e-3) * np.outer(d @ b, b)
    prim = prim.copy()
    prim["dir"] = d / np.linalg.norm(d, axis=1, keepdims=True)
    return geom, prim


def _slab_in(B):
    return _case(*_slab(2), B, 11)


def _barrel_in(B, field_map=gv_inputs.MAP_UNIFORM):
    return _case(*_barrel(field_map), B, 12)


FINE = dict(chord_tol_cm=1e-10)
CASES = {
    "slab oblique": (lambda: _slab_in((1.5, 3.0, -2.0)), {}),
    "slab in the xy plane": (lambda: _slab_in((2.0, -3.0, 0.0)), {}),
    "slab -x": (lambda: _slab_in((-4.0, 0.0, 0.0)), {}),
    "slab -y": (lambda: _slab_in((0.0, -4.0, 0.0)), {}),
    "slab -z": (lambda: _slab_in((0.0, 0.0, -4.0)), {}),
    "slab fine": (lambda: _slab_in((0.0, 4.0, 0.0)), FINE),
    "barrel oblique": (lambda: _barrel_in((0.7, -0.5, 3.6)), {}),
    "barrel x": (lambda: _barrel_in((3.8, 0.0, 0.0)), {}),
    "barrel -z": (lambda: _barrel_in((0.0, 0.0, -3.8)), {}),
    "barrel fine": (lambda: _barrel_in((0.0, 0.0, 3.8)), FINE),
    "barrel oblique rk45": (lambda: _barrel_in((0.7, -0.5, 3.6)), dict(field_method=RK45)),
    "map -z": (lambda: _barrel_in((0.0, 0.0, -3.8), gv_inputs.MAP_SOLENOID), {}),
    "map -z rk45": (lambda: _barrel_in((0.0, 0.0, -3.8), gv_inputs.MAP_SOLENOID), dict(field_method=RK45)),
    "map fine": (lambda: _barrel_in((0.0, 0.0, 3.8), gv_inputs.MAP_SOLENOID), FINE),
}


@pytest.mark.parametrize("precision", ["PMIX", "P64"])
@pytest.mark.parametrize("cap", [700, 12000])
@pytest.mark.parametrize("case", list(CASES))
def test_runs_equal_single_steps(case, cap, precision):
    import paper_2005_00949_amd as gv
    make, cfg = CASES[case]
    geom, prim = make()
    out = []
    for trace in (0, 1):
        eng = gv.Engine(geom, precision=getattr(gv, precision), deposit_mode=gv.DEPOSIT_FIXED, trace_cap=trace,
                        max_steps_per_track=cap, **cfg)
        e = eng.transport(prim, 99)
        s = eng.stats()
        out.append((np.asarray(e), eng.ledger(), eng.escape_hist(), s))
        eng.close()
    (e0, l0, h0, s0), (e1, l1, h1, s1) = out
    print(f"\n[{case} {precision}] steps {s0['total_steps']}, by the helper {s0['helper_steps']}")
    assert cap < 1000 or s0["helper_steps"] > 0
    for k in KEYS:
        assert s0[k] == s1[k], k
    assert np.array_equal(e0, e1) and np.array_equal(l0, l1) and np.array_equal(h0, h1)
