"""What the autotuner of the knobs left at 0 compares and keeps (batches of at
least 4096 primaries): statements about the choice and its counters, no timing."""
import numpy as np
import pytest

import gv_inputs

pytestmark = pytest.mark.gpu


def _low(n, seed=5):
    """Showers that stay below the population the step kernel takes."""
    return gv_inputs.mixed_beam(n, seed, 30.0, 300.0)


def test_batch_that_never_fills_the_gpu_keeps_the_defaults():
    """Between the thresholds that baskets of 64 and of 256 would have (32,768 and
    131,072 tracks on 256 CUs), no candidate has step-kernel work to be timed by:
    the defaults stand and the pool kernel keeps the batch.  A batch of the same
    size that does fill the GPU afterwards is tuned."""
    import paper_2005_00949_amd as gv
    eng = gv.Engine(gv_inputs.slab_calorimeter(50, (0.0, 4.0, 0.0)), max_steps_per_track=2000)
    for k in range(2):
        eng.transport(_low(6000), k)
        s = eng.stats()
        assert (s["basket"], s["occupancy"], s["inner_steps"]) == (256, 3, 4), s["basket"]
        assert s["graph_replays"] == 0
    assert s["autotune_ms"] == 0.0          # and the search is not repeated
    high = gv_inputs.beam(4200, 11, 1.0e4)
    eng.transport(high, 3)                  # finds the untimed choice and shows that it is of another kind
    assert eng.stats()["graph_replays"] > 0
    eng.transport(high, 4)
    s = eng.stats()
    assert s["tuned"] == 1 and s["autotune_ms"] > 0.0
    eng.transport(high, 5)
    s = eng.stats()
    assert s["tuned"] == 1 and s["autotune_ms"] == 0.0
    eng.close()


def test_choice_is_made_anew_for_another_kernel():
    """A choice timed on the helix's step kernel with the pool kernel beside it says
    nothing about the integrators' kernels, nor about a transport that a trace or a
    capacity keeps in the step kernel from end to end."""
    import paper_2005_00949_amd as gv
    eng = gv.Engine(gv_inputs.slab_calorimeter(20, (0.0, 4.0, 0.0)), max_steps_per_track=2000)
    prim = gv_inputs.beam(4096, 11, 3.0e3)
    for change in ({}, dict(field_method=gv.FIELD_RK45), dict(trace_cap=1)):
        eng.configure(**change)
        eng.transport(prim, 1)
        s = eng.stats()
        assert s["tuned"] == 1 and s["autotune_ms"] > 0.0, change
        eng.transport(prim, 2)
        s = eng.stats()
        assert s["tuned"] == 1 and s["autotune_ms"] == 0.0, change
    # a capacity has the step kernel from end to end too: the trace's choice serves
    eng.configure(trace_cap=0, capacity=1 << 24)
    eng.transport(prim, 1)
    s = eng.stats()
    assert s["tuned"] == 1 and s["autotune_ms"] == 0.0
    eng.close()


def test_trials_that_fall_behind_end_early():
    """Sixteen trials of half a batch, run to the end, take at least eight times the
    kernel time of the batch (no knobs are much better than the ones it runs with);
    trials that end once they have fallen behind take less."""
    import paper_2005_00949_amd as gv
    eng = gv.Engine(gv_inputs.slab_calorimeter(50), max_steps_per_track=2000)
    prim = gv_inputs.beam(4200, 11, 1.0e4)
    eng.transport(prim, 1)
    tune = eng.stats()["autotune_ms"]
    kernel = []
    for k in range(3):
        eng.transport(prim, 2 + k)
        kernel.append(eng.stats()["kernel_ms"])
    print(f"\nautotune {tune:.0f} ms, batch {min(kernel):.1f} ms")
    assert 0.0 < tune < 8.0 * min(kernel)
    eng.close()
