"""The energy after a continuous loss, found from a guess of the range bin,
against a binary search over the library's own range table in numpy: steps from
1 % of the range to nearly all of it, energies from the tracking cut to the end
of the table.  FP64: the same expressions on the same table, no tolerance.  Mixed
precision: float divisions are good to 2.5 ulp; the fraction in the bin and the
range interpolated with it carry 6, the range left (at least a fifth of the range)
five times that, and the last interpolation 6 more: 36, within 64 ulp of T."""
import numpy as np
import pytest

import gv_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pdg", [1, 2])
@pytest.mark.parametrize("precision", ["P64", "PMIX"])
@pytest.mark.parametrize("material", ["Pb", "polystyrene"])
def test_energy_after_loss(material, precision, pdg):
    import paper_2005_00949_amd as gv
    prec = getattr(gv, precision)
    F = np.float64 if precision == "P64" else np.float32
    eng = gv.Engine(gv_inputs.single_slab(material, 1.0e4), precision=prec)
    E = eng.debug_table(0, "nodes", prec).astype(F)
    R = eng.debug_table(0, "R_em" if pdg == 1 else "R_ep", prec).astype(F)
    rng = np.random.default_rng(pdg)
    n = 20000
    lo, hi = 1.1 * gv_inputs.TABLE_SPEC["t_track"], 0.99 * float(E[-1])
    T = np.exp(rng.uniform(np.log(lo), np.log(hi), n)).astype(F)
    st = dict(type=np.full(n, pdg), pos=np.tile([0.0, 0.0, 5.0e3], (n, 1)), dir=np.tile([0.0, 0.0, 1.0], (n, 1)),
              ekin=T.astype(np.float64), event=np.arange(n), tid=np.arange(n), nstep=np.zeros(n))
    o = eng.debug_step(st, 7, prec, stage=gv.DBG_THRU_ELOSS)
    i = np.clip(np.searchsorted(E, T, side="right") - 1, 0, len(E) - 2)
    w = (T - E[i]) / (E[i + 1] - E[i])
    full = R[i] + (R[i + 1] - R[i]) * w
    s = o["step"].astype(F)
    r = full - s
    use = (s >= F(0.011) * full) & (r >= F(0.2) * full) & (o["ekin"] > 0.0)
    assert use.sum() > n // 10
    T, r = T[use], r[use]
    k = np.clip(np.searchsorted(R, r, side="right") - 1, 0, len(R) - 2)
    left = E[k] + (E[k + 1] - E[k]) * (r - R[k]) / (R[k + 1] - R[k])
    want = (T - (T - left)).astype(np.float64)
    tol = 0.0 if precision == "P64" else 64 * 2.0**-24 * T.astype(np.float64)
    print(f"[{material} {precision}] {use.sum()} steps, worst {np.abs(o['ekin'][use] - want).max():.3g}")
    assert (np.abs(o["ekin"][use] - want) <= tol).all()
