"""Performance cases of the transport library: calls that its users make, over
the range of sizes they make them at.

A program that uses the library sets a detector up once (gv_init and
gv_configure, one context per process), then transports batch after batch of
new primaries and reads each event's deposits, its energy ledger and the step
and track counts.  So a pass of most cases here is one `Engine.transport` of
host primaries plus `ledger` and `stats`, on an engine that is kept between
passes.  The other public calls have a case of their own: setting a detector
up and using it once, and the allocation-free queue compaction.

A case is a dict of plain values:

  kind      "slab" (lead / liquid-argon stack), "plate" (one slab of one
            material), "barrel" (cylindrical shells), "setup" (a new plate
            detector every pass) or "compact" (queue compaction)
  events    primaries, one per event
  e_lo/e_hi kinetic energy in MeV, log-uniform (mono-energetic when equal)
  beam      "e-" or "mixed" (e-, e+, gamma in turn)
  field     tesla (slab: across the stack; barrel: along the axis)
  map       barrel: "uniform" or "solenoid"
  method    field propagation: "helix", "rk4" or "rk45"
  precision "mixed" or "fp64"
  order, deposit, tables   queue order, deposit mode, table sampling
  on_device deposits into a device tensor instead of host memory
"""
from __future__ import annotations

import math

import numpy as np
import torch

import gv_inputs
import paper_2005_00949_amd as gv

METHODS = {"helix": gv.FIELD_HELIX, "rk4": gv.FIELD_RK4, "rk45": gv.FIELD_RK45}

DEFAULTS = dict(kind="slab", events=100, e_lo=1.0e3, e_hi=1.0e3, beam="e-", layers=10, field=0.0, map="uniform",
                method="helix", precision="mixed", order="arrival", deposit="float", tables=False, on_device=False,
                material="Pb", thickness=0.2)


def listed():
    return [
        # One event at a time, as an event loop that feeds the library from a
        # generator calls it: latency of a transport, launches and host work.
        dict(name="one_event", kind="slab", events=1, layers=10, e_lo=1.0e3, e_hi=1.0e3),
        # A small batch without field (the repository's c1).
        dict(name="slab_small", kind="slab", events=100, layers=10, e_lo=1.0e3, e_hi=1.0e3),
        # A sampling calorimeter without field, 10 GeV electrons (c2): the
        # ordinary batch; deposits to host memory.
        dict(name="slab_ordinary", kind="slab", events=1000, layers=50, e_lo=1.0e4, e_hi=1.0e4),
        # The same detector in 4 T with the reproducible options: fixed-point
        # deposits, stable queues, table sampling (a c3-like batch of odd size).
        dict(name="slab_reproducible", kind="slab", events=333, layers=10, field=4.0, e_lo=1.0e4, e_hi=1.0e4,
             order="stable", deposit="fixed", tables=True, on_device=True),
        # One GPU's share of the large batch, all in FP64 (validation runs).
        dict(name="slab_fp64", kind="slab", events=1250, layers=50, field=4.0, beam="mixed", e_lo=100.0, e_hi=1.0e5,
             precision="fp64", on_device=True),
        # The largest: the benchmark's batch (c4).
        dict(name="slab_large", kind="slab", events=10000, layers=50, field=4.0, beam="mixed", e_lo=100.0,
             e_hi=1.0e5, on_device=True),
        # The cylindrical detector in a uniform solenoidal field (c5): showers
        # at large radius and electrons that spiral along the beam pipe.
        dict(name="barrel_uniform", kind="barrel", events=500, field=3.8, e_lo=5.0e4, e_hi=5.0e4, on_device=True),
        # The same detector in the field map of a finite solenoid, helix in the
        # local field (c5m).
        dict(name="barrel_map", kind="barrel", events=2000, field=3.8, map="solenoid", e_lo=5.0e4, e_hi=5.0e4,
             on_device=True),
        # ... and integrated by adaptive Runge-Kutta, fewer events.
        dict(name="barrel_map_rk45", kind="barrel", events=100, field=3.8, map="solenoid", method="rk45", e_lo=5.0e4,
             e_hi=5.0e4, on_device=True),
        # Transmission and reflection of many low-energy electrons through one
        # plate (t5): a large number of very short histories.
        dict(name="plate_many", kind="plate", events=20000, material="Pb", thickness=0.2, e_lo=10.0, e_hi=10.0),
        # A scan over detectors: set up, transport a small batch, read the
        # escape histogram; every pass pays for the set-up.
        dict(name="setup_scan", kind="setup", events=500, material="Pb", thickness=0.2, e_lo=10.0, e_hi=10.0),
        # The three-way queue compaction for callers that cannot allocate, at
        # a ragged population of a running shower.
        dict(name="compact", kind="compact", n=1000003, block=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["slab", "slab", "slab", "barrel", "barrel", "plate", "setup", "compact"])
    if kind == "compact":
        return dict(kind=kind, n=_log_int(rng, 1, 4000000), block=rng.choice([64, 128, 256]))
    if kind in ("plate", "setup"):
        material, t_lo, t_hi = rng.choice([("Pb", 0.02, 1.0), ("PbWO4", 0.03, 2.0), ("lAr", 0.2, 10.0),
                                           ("Si", 0.03, 5.0), ("brass", 0.03, 2.0), ("polystyrene", 0.2, 10.0)])
        e = round(math.exp(rng.uniform(math.log(1.0), math.log(100.0))), 3)
        return dict(kind=kind, events=_log_int(rng, 1, 20000 if kind == "plate" else 2000), material=material,
                    thickness=round(math.exp(rng.uniform(math.log(t_lo), math.log(t_hi))), 4), e_lo=e, e_hi=e,
                    precision=rng.choice(["mixed", "mixed", "fp64"]))
    precision = rng.choice(["mixed", "mixed", "fp64"])
    case = dict(kind=kind, beam=rng.choice(["e-", "mixed"]), precision=precision,
                order=rng.choice(["arrival", "arrival", "stable"]), deposit=rng.choice(["float", "fixed"]),
                tables=rng.choice([False, True]), on_device=rng.choice([False, True]))
    if kind == "slab":
        case["layers"] = rng.randint(5, 50)
        case["field"] = rng.choice([0.0, 0.0, 4.0, 4.0, 2.0])
        case["e_lo"] = round(math.exp(rng.uniform(math.log(50.0), math.log(5.0e4))), 2)
        case["e_hi"] = case["e_lo"] if rng.random() < 0.5 else 1.0e5
        most = 2.0e7 if precision == "mixed" else 6.0e6
    else:
        case["field"] = rng.choice([3.8, 2.0])
        case["map"] = rng.choice(["uniform", "solenoid"])
        case["method"] = rng.choice(["helix", "rk45", "rk4"]) if case["map"] == "solenoid" else "helix"
        case["e_lo"] = case["e_hi"] = round(math.exp(rng.uniform(math.log(1.0e3), math.log(5.0e4))), 1)
        most = 2.0e7 if case["method"] == "helix" and precision == "mixed" else 3.0e6
    case["events"] = max(1, min(5000, _log_int(rng, 1.0, most / _mean_energy(case))))
    return case


def _mean_energy(case):
    lo, hi = case["e_lo"], case["e_hi"]
    return lo if lo == hi else (hi - lo) / math.log(hi / lo)


# ---------------------------------------------------------------------------
# the engine: one context per process, kept while the detector and the run
# options stay the same
# ---------------------------------------------------------------------------
_current = [None, None]


def _geometry(c):
    if c["kind"] == "slab":
        return gv_inputs.slab_calorimeter(c["layers"], (0.0, c["field"], 0.0))
    if c["kind"] == "barrel":
        return gv_inputs.barrel((0.0, 0.0, c["field"]),
                                gv_inputs.MAP_SOLENOID if c["map"] == "solenoid" else gv_inputs.MAP_UNIFORM)
    return gv_inputs.single_slab(c["material"], c["thickness"])


def _new_engine(c):
    return gv.Engine(_geometry(c), driver=gv.DRIVER_BATCHED,
                     precision=gv.P64 if c["precision"] == "fp64" else gv.PMIX,
                     field_method=METHODS[c["method"]], edep_on_device=1 if c["on_device"] else 0,
                     queue_order=gv.ORDER_STABLE if c["order"] == "stable" else gv.ORDER_ARRIVAL,
                     deposit_mode=gv.DEPOSIT_FIXED if c["deposit"] == "fixed" else gv.DEPOSIT_FLOAT,
                     fs_alias=gv.FS_ALL if c["tables"] else 0)


def _engine(c):
    key = tuple(sorted((k, v) for k, v in c.items() if k not in ("events", "e_lo", "e_hi", "beam", "name")))
    if _current[0] != key:
        _current[1] = _new_engine(c)
        _current[0] = key
    return _current[1]


def _primaries(c, seed):
    n = c["events"]
    if c["kind"] == "barrel":
        p = gv_inputs.barrel_beam(n, seed, c["e_lo"])
        if c["beam"] == "mixed":
            p["pdg"] = np.array([11, -11, 22], dtype=np.int32)[np.arange(n) % 3]
        return p
    if c["beam"] == "mixed" or c["e_lo"] != c["e_hi"]:
        p = gv_inputs.mixed_beam(n, seed, c["e_lo"], c["e_hi"])
        if c["beam"] != "mixed":
            p["pdg"] = 11
        return p
    return gv_inputs.beam(n, gv_inputs.PDG_ELECTRON, c["e_lo"])


def prepare(case, seed):
    c = dict(DEFAULTS, **case)
    if c["kind"] == "compact":
        # output codes of a running shower's tracks: most survive in the queue
        # of their type (queues are read type by type), some make secondaries
        n = c["n"]
        g = torch.Generator(device="cuda").manual_seed(seed)
        u = torch.rand((n, 3), generator=g, device="cuda")
        kind = torch.randint(0, 3, (n, 2), generator=g, device="cuda", dtype=torch.int8)
        own = (torch.arange(n, device="cuda") * 10 // max(n, 1)).clamp(max=9)
        own = torch.where(own < 7, 0, torch.where(own < 9, 1, 2)).to(torch.int8)
        codes = torch.full((n, 3), -1, dtype=torch.int8, device="cuda")
        codes[:, 0] = torch.where(u[:, 0] < 0.85, own, -1)
        codes[:, 1] = torch.where(u[:, 1] < 0.12, kind[:, 0], -1)
        codes[:, 2] = torch.where((u[:, 1] < 0.12) & (u[:, 2] < 0.4), kind[:, 1], -1)
        return dict(case=c, codes=codes, index=torch.zeros(9 * n, dtype=torch.int32, device="cuda"),
                    counts=torch.zeros(4, dtype=torch.int32, device="cuda"))
    state = dict(case=c, seed=int(seed), primaries=_primaries(c, seed))
    if c["kind"] != "setup":
        eng = _engine(c)
        if c["on_device"]:
            state["edep"] = torch.zeros((c["events"], eng.n_cells), dtype=torch.float64, device="cuda")
    return state


def run(state):
    c = state["case"]
    if c["kind"] == "compact":
        gv.compact3_noalloc(state["codes"].data_ptr(), c["n"], c["block"], state["index"].data_ptr(),
                            state["counts"].data_ptr(), torch.cuda.current_stream().cuda_stream)
        return {"index": state["index"], "counts": state["counts"]}
    if c["kind"] == "setup":
        _current[0] = None
        eng = _new_engine(c)
    else:
        eng = _engine(c)
    if c["on_device"]:
        edep = state["edep"]
        eng.transport(state["primaries"], state["seed"], edep.data_ptr())
    else:
        edep = eng.transport(state["primaries"], state["seed"])
    stats = eng.stats()
    out = {"edep": edep, "ledger": eng.ledger(), "steps": stats["steps"], "tracks": stats["tracks"],
           "interactions": stats["interactions"]}
    if c["kind"] in ("plate", "setup"):
        out["escapes"] = eng.escape_hist()
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
# Steps of a shower per GeV of primary energy with the repository's cuts
# (counted), and arithmetic of one step: cross sections, distance to the next
# boundary, move, and for charged steps scattering and energy loss, averaged
# over the mix of photon and charged steps.
STEPS_PER_GEV = 9950.0
FLOPS_PER_STEP = 250.0


def work(case):
    c = dict(DEFAULTS, **case)
    if c["kind"] == "compact":
        # codes in, one index out per code that is not -1 (about 1.02 a track)
        return {"bytes": 3.0 * c["n"] + 4.0 * 1.02 * c["n"] + 16.0, "flops": 0.0}
    cells = {"slab": 2 * c["layers"], "barrel": 51}.get(c["kind"], 1)
    if c["kind"] in ("plate", "setup"):
        steps = 9.0 * c["events"]
    else:
        steps = max(1.0, STEPS_PER_GEV * c["events"] * _mean_energy(c) * 1.0e-3)
    # primaries in, deposits and ledger out; tracks need never leave the chip
    return {"bytes": 64.0 * c["events"] + 8.0 * c["events"] * (cells + 4), "flops": FLOPS_PER_STEP * steps}


def exact(case, seed):
    """Transports are random histories whose steps depend on the rounding of
    the ones before: 64-bit arithmetic takes other histories, so there is no
    value to compare with.  The compaction is a stable partition."""
    c = dict(DEFAULTS, **case)
    if c["kind"] != "compact":
        return None
    n = c["n"]
    codes = prepare(case, seed)["codes"].reshape(-1)
    index = torch.zeros(9 * n, dtype=torch.int32, device="cuda")
    counts = torch.zeros(4, dtype=torch.int32, device="cuda")
    for q in range(3):
        at = torch.nonzero(codes == q).reshape(-1)
        index[q * 3 * n: q * 3 * n + len(at)] = (at // 3 * 4 + at % 3).to(torch.int32)
        counts[q] = len(at)
    return {"index": index, "counts": counts}
