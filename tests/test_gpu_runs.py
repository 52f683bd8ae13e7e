"""Runs of vacuum steps (a looper's steps taken in one loop) against the same
steps taken one by one, which a transport with a trace does: both evaluate the
same expressions, so fixed-point deposits, ledgers, counters, the escape
histogram and the step at which a looper is given up are equal bit for bit (no
tolerance).  Loopers start in every gap of the barrel, near its walls, and beside
the slab stack; the looper cap lies inside, at the edge of and beyond a run."""
import numpy as np
import pytest

import gv_inputs

pytestmark = pytest.mark.gpu

KEYS = ("steps", "tracks", "escaped", "killed", "rk_substeps", "rk_rejected")


def _prim(pos, seed, ekin, axis=2):
    n = len(pos)
    rng = np.random.default_rng(seed)
    d = rng.normal(size=(n, 3))
    d[:, axis] *= 1e-3          # turning about the field, hardly moving along it
    p = np.zeros(n, dtype=gv_inputs.PRIMARY_DTYPE)
    p["pdg"] = np.array([11, -11], dtype=np.int32)[np.arange(n) % 2]
    p["event"] = np.arange(n, dtype=np.int32)
    p["ekin"] = ekin * 10.0 ** rng.uniform(-1.0, 0.5, n)
    p["pos"] = pos
    p["dir"] = d / np.linalg.norm(d, axis=1, keepdims=True)
    return p


def _barrel(field_map):
    geom = gv_inputs.barrel(field_map=field_map)
    b = geom["bounds"]
    gaps = [(b[v], b[v + 1]) for v in range(len(b) - 1) if geom["material"][v] < 0]
    # the middle of each gap, and 1 um and 0.1 mm from either wall
    r = [x for lo, hi in gaps for x in (0.5 * (lo + hi), lo + 1e-4, lo + 1e-2, hi - 1e-4, hi - 1e-2)] + [0.0]
    phi = np.linspace(0.0, 6.0, len(r))
    pos = np.stack([np.array(r) * np.cos(phi), np.array(r) * np.sin(phi), np.linspace(-300.0, 300.0, len(r))], axis=1)
    return geom, _prim(pos, 5, 2.0)


def _slab(axis):
    B = [0.0, 0.0, 0.0]
    B[axis] = 4.0
    geom = gv_inputs.slab_calorimeter(10, tuple(B))
    ex, ey = geom["env"]
    wx, wy, z0, z1 = geom["world"]
    lo, hi = geom["bounds"][0], geom["bounds"][-1]
    rng = np.random.default_rng(3)
    pos = [(rng.uniform(-wx, wx), rng.uniform(-wy, wy), z0 + f * (lo - z0)) for f in (0.01, 0.3, 0.9, 0.999)]
    pos += [(rng.uniform(-wx, wx), rng.uniform(-wy, wy), hi + f * (z1 - hi)) for f in (0.01, 0.3, 0.9)]
    pos += [(s * (ex + f * (wx - ex)), 0.5 * ey, 0.5 * (lo + hi)) for s in (-1, 1) for f in (1e-4, 0.2, 0.8)]
    return geom, _prim(np.array(pos), 6, 2.0, axis)


RK45 = 2
CASES = {
    "barrel rk45": lambda: _barrel(gv_inputs.MAP_UNIFORM),
    "barrel map rk45": lambda: _barrel(gv_inputs.MAP_SOLENOID),
    "barrel": lambda: _barrel(gv_inputs.MAP_UNIFORM),
    "barrel map": lambda: _barrel(gv_inputs.MAP_SOLENOID),
    "slab x": lambda: _slab(0),
    "slab y": lambda: _slab(1),
    "slab z": lambda: _slab(2),
}


@pytest.mark.parametrize("precision", ["PMIX", "P64"])
@pytest.mark.parametrize("cap", [1, 700, 12000])
@pytest.mark.parametrize("case", list(CASES))
def test_runs_equal_single_steps(case, cap, precision):
    import paper_2005_00949_amd as gv
    geom, prim = CASES[case]()
    out = []
    for trace in (0, 1):
        eng = gv.Engine(geom, precision=getattr(gv, precision), deposit_mode=gv.DEPOSIT_FIXED, trace_cap=trace,
                        max_steps_per_track=cap, field_method=RK45 if "rk45" in case else 0)
        e = eng.transport(prim, 99)
        s = eng.stats()
        out.append((np.asarray(e), eng.ledger(), eng.escape_hist(), s))
        eng.close()
    (e0, l0, h0, s0), (e1, l1, h1, s1) = out
    if cap > 1000:
        assert s0["helper_steps"] > 0
    for k in KEYS:
        assert s0[k] == s1[k], k
    assert np.array_equal(e0, e1) and np.array_equal(l0, l1) and np.array_equal(h0, h1)
