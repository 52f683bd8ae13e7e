"""The step kernel on loopers: more of them than the helper takes, circling in the
vacuum beside the slab stack.  A transport with explicit knobs (step kernel from end
to end) and one without (pool kernel, helper, step kernel) take the same steps:
fixed-point scores, counters and escape histogram are equal, no tolerance.

Times: a wavefront of loopers takes 1.6 us per step in the vacuum form and 3.2 us in
the general one, and nothing but this chain bounds the call; the line is drawn
halfway, at 2.4 us."""
import numpy as np
import pytest

import gv_inputs

pytestmark = pytest.mark.gpu

KEYS = ("steps", "tracks", "interactions", "escaped", "killed", "rejection_exhausted")
KNOBS = dict(basket=256, occupancy=3, inner_steps=4)
STEPS = 20_000


def loopers(n, field_map=None):
    """n e-/e+ turning about the field, in front of the slab stack or (field_map) in
    the gaps of the barrel."""
    rng = np.random.default_rng(n)
    p = np.zeros(n, dtype=gv_inputs.PRIMARY_DTYPE)
    p["pdg"] = np.array([11, -11], dtype=np.int32)[np.arange(n) % 2]
    p["event"] = np.arange(n, dtype=np.int32)
    p["ekin"] = 10.0 ** rng.uniform(-0.9, 0.0, n)
    d = rng.normal(size=(n, 3))
    if field_map is None:
        geom, axis = gv_inputs.slab_calorimeter(10, (0.0, 4.0, 0.0)), 1
        p["pos"] = np.stack([rng.uniform(-25, 25, n), rng.uniform(-25, 25, n), rng.uniform(-9.0, -3.0, n)], axis=1)
    else:
        geom, axis = gv_inputs.barrel(field_map=field_map), 2
        b = geom["bounds"]
        gaps = np.array([(b[v], b[v + 1]) for v in range(1, len(b) - 1) if geom["material"][v] < 0])
        lo, hi = gaps[np.arange(n) % len(gaps)].T
        r, phi = lo + rng.uniform(0.3, 0.7, n) * (hi - lo), rng.uniform(0.0, 6.28, n)
        p["pos"] = np.stack([r * np.cos(phi), r * np.sin(phi), rng.uniform(-50, 50, n)], axis=1)
    d[:, axis] *= 1e-4
    p["dir"] = d / np.linalg.norm(d, axis=1, keepdims=True)
    return geom, p


def run(gv, geom, prim, **cfg):
    eng = gv.Engine(geom, deposit_mode=gv.DEPOSIT_FIXED, **cfg)
    ms = []
    for _ in range(2):
        e = eng.transport(prim, 7)
        st = eng.stats()
        ms.append(st["kernel_ms"])
    out = (np.asarray(e).copy(), eng.ledger(), eng.escape_hist(), [st[k] for k in KEYS], min(ms))
    eng.close()
    return out


def assert_same(a, b):
    assert a[3] == b[3]
    assert all(np.array_equal(x, y) for x, y in zip(a[:3], b[:3]))


@pytest.mark.parametrize("n", [257, 2500])
@pytest.mark.parametrize("cfg", [dict(KNOBS), dict(KNOBS, queue_order=1), dict(capacity=1 << 24), dict(graph_steps=8)],
                         ids=["knobs", "stable", "capacity", "graph"])
def test_step_kernel_steps_loopers_in_the_vacuum_form(n, cfg):
    import paper_2005_00949_amd as gv
    geom, prim = loopers(n)
    a = run(gv, geom, prim, max_steps_per_track=STEPS, **cfg)
    b = run(gv, geom, prim, max_steps_per_track=STEPS)
    assert_same(a, b)
    us = a[4] * 1e3 / STEPS
    print(f"\n{n} loopers: {us:.2f} us per step")
    assert us < 2.4


@pytest.mark.parametrize("precision", ["PMIX", "P64"])
def test_step_kernel_steps_loopers_of_the_barrel(precision):
    import paper_2005_00949_amd as gv
    geom, prim = loopers(300, gv_inputs.MAP_UNIFORM)
    cfg = dict(precision=getattr(gv, precision), max_steps_per_track=2_000)
    assert_same(run(gv, geom, prim, **cfg, **KNOBS), run(gv, geom, prim, **cfg))


# (loopers, field map, method, looper cap): on either side of the numbers up to which
# one wavefront per looper takes them, and many more
MANY = {
    "uniform 1100": (1100, None, 0, 4000),
    "uniform 4200": (4200, None, 0, 20_000),
    "barrel 2100": (2100, gv_inputs.MAP_UNIFORM, 0, 4000),
    "map 1500": (1500, gv_inputs.MAP_SOLENOID, 0, 4000),
    "map 5000": (5000, gv_inputs.MAP_SOLENOID, 0, 4000),
    "rk45 1025": (1025, gv_inputs.MAP_SOLENOID, 2, 1000),
    "rk45 uniform 1500": (1500, gv_inputs.MAP_UNIFORM, 2, 1000),
    "rk4 uniform 1500": (1500, gv_inputs.MAP_UNIFORM, 1, 50),
}


@pytest.mark.parametrize("precision", ["PMIX", "P64"])
@pytest.mark.parametrize("case", list(MANY))
def test_many_loopers_without_knobs(case, precision):
    """Loopers alone take no longer without knobs than in the step kernel: 1.25 leaves
    the two launches of the pool kernel that find out (0.5 ms) and the noise of either
    call a fifth each; the pool kernel alone took 1.4 times (4,200 in a uniform field)
    to 4 times as long."""
    import paper_2005_00949_amd as gv
    n, field_map, method, cap = MANY[case]
    geom, prim = loopers(n, field_map)
    cfg = dict(precision=getattr(gv, precision), max_steps_per_track=cap, field_method=method)
    a = run(gv, geom, prim, **cfg)
    b = run(gv, geom, prim, **cfg, **KNOBS)
    print(f"\n{case} {precision}: {a[4]:.2f} ms, with knobs {b[4]:.2f} ms")
    assert_same(a, b)
    if b[4] > 5.0:
        assert a[4] < 1.25 * b[4]
