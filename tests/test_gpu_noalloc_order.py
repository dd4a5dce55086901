"""The allocation-free forward beside a handle's other passes.

Its barriers and work memory are the library's own array, so it may come before
any recorded pass of the handle, and a captured one may be replayed while the
handle runs: every pass is compared bitwise with one workgroup's.
"""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _sim(sc, **kw):
    from paper_2106_05306_amd.sim import Sim
    return Sim.from_scene(sc, device=DEV, precision="mixed", **kw)


def _one_workgroup(sc, monkeypatch, **kw):
    monkeypatch.setenv("DIFFCLOTH_FWD_WGS", "0")
    s = _sim(sc, **kw)
    assert s.stats()["fwd_workgroups"] == 1
    xT, vT, _ = s.forward(sc.steps)
    out = xT.clone(), vT.clone()
    s.close()
    monkeypatch.delenv("DIFFCLOTH_FWD_WGS")
    return out


def _noalloc(s, steps):
    xT, vT = (torch.full((s.m, 3), float("nan"), dtype=torch.float64, device=DEV) for _ in range(2))
    s.forward_noalloc(steps, xT, vT)
    return xT, vT


@pytest.mark.parametrize("n", [24, 48])
@pytest.mark.parametrize("then", ["forward", "batch_forward", "batch_advance"])
def test_first_recorded_pass_after_noalloc(monkeypatch, n, then):
    from paper_2106_05306_amd.sim import batch_advance, batch_forward
    sc = scenes.c2_sphere_drop(0, n=n, steps=6)
    rx, rv = _one_workgroup(sc, monkeypatch)
    s = _sim(sc)                                     # fresh: the allocation-free pass comes first
    assert s.stats()["fwd_workgroups"] > 1
    ax, av = _noalloc(s, sc.steps)
    if then == "forward":
        x, v, _ = s.forward(sc.steps)
    elif then == "batch_forward":
        (x, v), = batch_forward([s], [sc.steps])
    else:
        s.job_forward(sc.steps)
        while batch_advance([s], [4])[0] > 0:
            pass
        x, v = s.state(sc.steps)
    bx, bv = _noalloc(s, sc.steps)
    torch.cuda.synchronize()
    for a, b in ((ax, av), (x, v), (bx, bv)):
        assert torch.equal(a, rx) and torch.equal(b, rv)
    s.close()


def test_captured_pass_replayed_while_the_handle_runs(monkeypatch):
    # replays on a stream of their own, several at a time beside forward and
    # adjoint passes of the same handle, and alone between them
    sc = scenes.c2_sphere_drop(0, n=32, steps=6)
    rx, rv = _one_workgroup(sc, monkeypatch)
    st, side = torch.cuda.Stream(), torch.cuda.Stream()
    seed = torch.tensor(np.random.default_rng(2).normal(size=(sc.n_nodes, 3)), device=DEV)
    with torch.cuda.stream(st):
        s = _sim(sc, stream=st)
        assert s.stats()["fwd_workgroups"] > 1
        s.forward(sc.steps)
        ref = s.backward(seed)["dx0"].clone()
        xT, vT = (torch.zeros((s.m, 3), dtype=torch.float64, device=DEV) for _ in range(2))
        st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        s.forward_noalloc(sc.steps, xT, vT)
    for _ in range(4):
        with torch.cuda.stream(side):
            xT.zero_()
            vT.zero_()
            for _ in range(3):
                g.replay()
        with torch.cuda.stream(st):
            for _ in range(3):
                x, v, _ = s.forward(sc.steps)
                d = s.backward(seed)["dx0"]
                st.synchronize()
                assert torch.equal(x, rx) and torch.equal(v, rv) and torch.equal(d, ref)
        side.synchronize()
        assert torch.equal(xT, rx) and torch.equal(vT, rv)
    torch.cuda.synchronize()
    s.close()


@pytest.mark.parametrize("absent", ["2", "3"])      # at the first barrier, or in the second step
@pytest.mark.parametrize("warm", [False, True])
def test_pass_that_gave_up_runs_again(monkeypatch, absent, warm):
    # (a workgroup withheld by the host: the others' waits end at their limit)
    sc = scenes.c2_sphere_drop(0, n=24, steps=6)
    sc.X = sc.X - np.array([0.0, 0.27, 0.0])        # in contact from the first steps on
    rx, rv = _one_workgroup(sc, monkeypatch, warm_start=warm)
    monkeypatch.setenv("DIFFCLOTH_MW_SPIN", "2000000")
    s = _sim(sc, warm_start=warm)
    assert s.stats()["fwd_workgroups"] > 1
    for a in (absent, "0", absent):
        monkeypatch.setenv("DIFFCLOTH_MW_TEST_ABSENT", a)
        xT, vT = _noalloc(s, sc.steps)
        torch.cuda.synchronize()
        assert torch.equal(xT, rx) and torch.equal(vT, rv)
    s.close()


def test_captured_pass_of_a_handle_that_keeps_to_one_workgroup_since(monkeypatch):
    # a replay takes the descriptor of the handle's latest call, which then chose another kernel
    sc = scenes.c2_sphere_drop(0, n=24, steps=6)
    rx, rv = _one_workgroup(sc, monkeypatch)
    monkeypatch.setenv("DIFFCLOTH_MW_SPIN", "2000000")
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        s = _sim(sc, stream=st)
        xT, vT = (torch.zeros((s.m, 3), dtype=torch.float64, device=DEV) for _ in range(2))
        s.forward_noalloc(sc.steps, xT, vT)
        st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        s.forward_noalloc(sc.steps, xT, vT)
    for later in range(3):
        with torch.cuda.stream(st):
            if later == 1:
                monkeypatch.setenv("DIFFCLOTH_MW_TEST_ABSENT", "2")
                s.forward(sc.steps)
                monkeypatch.delenv("DIFFCLOTH_MW_TEST_ABSENT")
                assert s.stats()["fwd_workgroups"] == 1
            if later == 2:
                s.forward_noalloc(sc.steps, xT, vT)
            for _ in range(2):
                xT.zero_()
                vT.zero_()
                g.replay()
                st.synchronize()
                assert torch.equal(xT, rx) and torch.equal(vT, rv)
    s.close()
