"""The range bin on tables of other spacings than the usual 100 nodes per decade:
the energy after a continuous loss against a binary search over the library's own
range table in numpy (FP64, the same expressions: no tolerance), for every step that
leaves the track moving, so down to the range at the tracking cut; and the cost of a
fine table, on which the guess of the bin is several bins off."""
import ctypes as C

import numpy as np
import pytest

import gv_inputs

pytestmark = pytest.mark.gpu


def _spec(bpd):
    return dict(bins_per_decade=bpd, n_nodes=8 * bpd + 1)


def _table(gv, eng, which, n):
    """All nodes of one table of material 0 (FP64)."""
    out = np.zeros(n)
    io = gv.DebugIO()
    io.material, io.which, io.precision = 0, gv.TABLE_IDS[which], gv.P64
    io.values = out.ctypes.data
    rc = eng.lib.gv_debug_step(gv.DBG_TABLE, n, C.byref(io))
    assert rc == 0, eng.lib.gv_last_error()
    return out


@pytest.mark.parametrize("pdg", [1, 2])
@pytest.mark.parametrize("bpd", [5, 25, 100, 400, 1000])
@pytest.mark.parametrize("material", ["Pb", "polystyrene"])
def test_energy_after_loss(material, bpd, pdg):
    import paper_2005_00949_amd as gv
    spec = _spec(bpd)
    eng = gv.Engine(gv_inputs.single_slab(material, 1.0e4), table_spec=spec, precision=gv.P64)
    E = _table(gv, eng, "nodes", spec["n_nodes"])
    R = _table(gv, eng, "R_em" if pdg == 1 else "R_ep", spec["n_nodes"])
    rng = np.random.default_rng(bpd + pdg)
    n = 20000
    # half over the whole table, half where a step may take most of the range
    T = np.exp(np.concatenate([rng.uniform(np.log(0.11), np.log(0.99 * E[-1]), n // 2),
                               rng.uniform(np.log(0.11), np.log(5.0), n // 2)]))
    st = dict(type=np.full(n, pdg), pos=np.tile([0.0, 0.0, 5.0e3], (n, 1)), dir=np.tile([0.0, 0.0, 1.0], (n, 1)),
              ekin=T, event=np.arange(n), tid=np.arange(n), nstep=np.zeros(n))
    o = eng.debug_step(st, 7, gv.P64, stage=gv.DBG_THRU_ELOSS)
    eng.close()
    i = np.clip(np.searchsorted(E, T, side="right") - 1, 0, len(E) - 2)
    w = (T - E[i]) / (E[i + 1] - E[i])
    full = R[i] + (R[i + 1] - R[i]) * w
    r = full - o["step"]
    use = (o["step"] >= 0.011 * full) & (o["ekin"] > 0.0)
    assert use.sum() > n // 10 and (r[use] < 0.2 * full[use]).any()
    T, r = T[use], r[use]
    k = np.clip(np.searchsorted(R, r, side="right") - 1, 0, len(R) - 2)
    left = np.where(r <= R[0], E[0] * r / R[0], E[k] + (E[k + 1] - E[k]) * (r - R[k]) / (R[k + 1] - R[k]))
    assert np.array_equal(o["ekin"][use], T - (T - left))


def test_a_fine_table_costs_no_more():
    """A search over ten times the nodes takes a third more loads (log2); a walk from
    a guess ten times as many bins off took nearly twice the kernel time."""
    import paper_2005_00949_amd as gv
    prim = gv_inputs.beam(20000, 11, 10.0)
    best = {}
    for bpd in (100, 1000):
        eng = gv.Engine(gv_inputs.single_slab("Pb", 0.2), table_spec=_spec(bpd), precision=gv.PMIX, basket=256,
                        occupancy=3, inner_steps=4)
        ms = []
        for k in range(8):
            eng.transport(prim, 1)
            ms.append(eng.stats()["kernel_ms"])
        best[bpd] = min(ms)
        eng.close()
    print(f"\nkernel time at 100 and 1000 nodes per decade: {best[100]:.3f} and {best[1000]:.3f} ms")
    assert best[1000] < 1.33 * best[100]
