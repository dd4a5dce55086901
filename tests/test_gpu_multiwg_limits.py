"""Which launches the multi-workgroup forward serves, and on how many workgroups.

Results are compared bitwise with one workgroup's.
"""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _sim(sc, **kw):
    from paper_2106_05306_amd.sim import Sim
    kw.setdefault("precision", "mixed")
    return Sim.from_scene(sc, device=DEV, **kw)


def _one_workgroup(sc, monkeypatch, **kw):
    with monkeypatch.context() as mp:
        mp.setenv("DIFFCLOTH_FWD_WGS", "0")
        s = _sim(sc, **kw)
        assert s.stats()["fwd_workgroups"] == 1
        x, v, _ = s.forward(sc.steps)
        out = x.clone(), v.clone()
        s.close()
    return out


def _low(sc):
    sc.X = sc.X - np.array([0.0, 0.27, 0.0])        # in contact from the first steps on
    return sc


@pytest.mark.parametrize("cus", [1, 32, 64])
def test_workgroups_that_wait_for_each_other_fit_the_device(monkeypatch, cus):
    # as on a partition of `cus` compute units: all workgroups of a launch can be resident there
    from paper_2106_05306_amd.sim import batch_forward
    scs = [_low(scenes.c2_sphere_drop(0, n=n, steps=st)) for n, st in ((40, 4), (28, 6))]
    ref = [_one_workgroup(sc, monkeypatch) for sc in scs]
    monkeypatch.setenv("DIFFCLOTH_TEST_CUS", str(cus))
    limit = cus - min(64, cus // 4)
    sims = [_sim(sc) for sc in scs]
    for sc, s, (rx, rv) in zip(scs, sims, ref):
        wgs = s.stats()["fwd_workgroups"]
        assert wgs <= limit and (wgs > 1) == (cus >= 32)
        x, v, _ = s.forward(sc.steps)
        assert torch.equal(x, rx) and torch.equal(v, rv)
        xT, vT = (torch.full((s.m, 3), float("nan"), dtype=torch.float64, device=DEV) for _ in range(2))
        s.forward_noalloc(sc.steps, xT, vT)
        assert torch.equal(xT, rx) and torch.equal(vT, rv)
        assert s.stats()["fwd_workgroups"] == wgs    # nobody gave up
    for (x, v), (rx, rv) in zip(batch_forward(sims, [sc.steps for sc in scs]), ref):
        assert torch.equal(x, rx) and torch.equal(v, rv)
    for s in sims:
        s.close()
