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


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kw", [{}, dict(warm_start=True), dict(fwd_tol=1e-7, fwd_max_iters=4000)],
                         ids=["", "warm", "converged"])
def test_one_block_members_leave_a_batch_on_many_workgroups(monkeypatch, precision, kw):
    # sheets of one to 32 nodes (a tree of one level) beside larger ones: all of
    # them on the multi-workgroup kernel, which gives up where the larger
    # one's last workgroup is withheld
    from paper_2106_05306_amd import _binding as B
    from paper_2106_05306_amd.sim import batch_advance, batch_forward
    scs = [_low(scenes.c2_sphere_drop(0, n=n, steps=st)) for n, st in ((2, 3), (5, 9), (28, 4))]
    scs.append(scenes.tiny_scene(4, steps=7, obstacle="plane", height=0.002))
    ref = [_one_workgroup(sc, monkeypatch, precision=precision, **kw) for sc in scs]
    monkeypatch.setenv("DIFFCLOTH_MW_SPIN", "2000000")
    sims = [_sim(sc, precision=precision, **kw) for sc in scs]
    assert [s.stats()["fwd_workgroups"] > 1 for s in sims] == [False, False, True, False]
    for (x, v), (rx, rv) in zip(batch_forward(sims, [sc.steps for sc in scs]), ref):
        assert torch.equal(x, rx) and torch.equal(v, rv)
    for sc, s in zip(scs, sims):
        s.job_forward(sc.steps)
    left = [sc.steps for sc in scs]
    while sum(left) > 0:
        on = [i for i in range(4) if left[i] > 0]
        for i, k in zip(on, batch_advance([sims[i] for i in on], [2] * len(on))):
            left[i] = k
    for sc, s, (rx, rv) in zip(scs, sims, ref):
        x, v = s.state(sc.steps)
        assert torch.equal(x, rx) and torch.equal(v, rv)
    monkeypatch.setenv("DIFFCLOTH_MW_TEST_ABSENT", "1")
    with pytest.raises(B.SimError) as e:
        batch_forward(sims, [sc.steps for sc in scs])
    assert e.value.code == B.SIM_ESYNC
    for s in sims:
        s.close()


def test_barrier_counts_after_16_million_launches(monkeypatch):
    # a launch's counts start 2^40 above the last one's: the 2^24th would start below them
    from paper_2106_05306_amd.sim import batch_advance, batch_forward
    sc = _low(scenes.c2_sphere_drop(0, n=28, steps=4))
    rx, rv = _one_workgroup(sc, monkeypatch)
    monkeypatch.setenv("DIFFCLOTH_TEST_LAUNCHES", str(2 ** 24 - 3))
    passes = {"forward": lambda s: s.forward(sc.steps)[:2], "batch": lambda s: batch_forward([s], [sc.steps])[0]}

    def job(s):
        s.job_forward(sc.steps)
        while batch_advance([s], [1])[0] > 0:
            pass
        return s.state(sc.steps)

    passes["job"] = job
    for run in passes.values():
        s = _sim(sc)
        assert s.stats()["fwd_workgroups"] > 1
        for _ in range(6):
            x, v = run(s)
            assert torch.equal(x, rx) and torch.equal(v, rv)
        assert s.stats()["fwd_workgroups"] > 1
        s.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("lds,threads,wgs", [("1", "64", 2), ("0", "64", 2), ("0", "256", 5), ("1", "256", 16),
                                             ("0", "512", 16), ("1", "448", 7)])
def test_factor_from_lds_or_memory_on_any_number_of_threads(monkeypatch, precision, lds, threads, wgs):
    # 24 x 24: two workgroups of 64 threads have more rows, items and nodes than threads
    sc = _low(scenes.c2_sphere_drop(0, n=24, steps=4))
    rx, rv = _one_workgroup(sc, monkeypatch, precision=precision)
    monkeypatch.setenv("DIFFCLOTH_FWD_WGS", str(wgs))
    monkeypatch.setenv("DIFFCLOTH_MW_LDS", lds)
    monkeypatch.setenv("DIFFCLOTH_MW_THREADS", threads)
    s = _sim(sc, precision=precision)
    assert s.stats()["fwd_workgroups"] == wgs
    x, v, _ = s.forward(sc.steps)
    assert torch.equal(x, rx) and torch.equal(v, rv)
    s.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("scs", [
    [scenes.stacked_sheets(3, steps=9), scenes.stacked_sheets(14, steps=5), scenes.stacked_sheets(4, steps=7, ground=True)],
    [_low(scenes.discretized_sphere_drop(0, n=5, steps=9, level=1)), scenes.wind_napkin(0, n=4, steps=8),
     _low(scenes.discretized_sphere_drop(0, n=21, steps=5, level=1))],
], ids=["pairs", "mesh"])
def test_one_block_members_with_pairs_mesh_obstacles_and_forces(monkeypatch, scs, precision):
    from paper_2106_05306_amd import _binding as B
    from paper_2106_05306_amd.sim import batch_forward
    ref = [_one_workgroup(sc, monkeypatch, precision=precision) for sc in scs]
    monkeypatch.setenv("DIFFCLOTH_MW_SPIN", "2000000")
    sims = [_sim(sc, precision=precision) for sc in scs]
    assert sum(s.stats()["fwd_workgroups"] > 1 for s in sims) == 1
    for (x, v), (rx, rv) in zip(batch_forward(sims, [sc.steps for sc in scs]), ref):
        assert torch.equal(x, rx) and torch.equal(v, rv)
    monkeypatch.setenv("DIFFCLOTH_MW_TEST_ABSENT", "1")
    with pytest.raises(B.SimError) as e:
        batch_forward(sims, [sc.steps for sc in scs])
    assert e.value.code == B.SIM_ESYNC
    for s in sims:
        s.close()
