"""Forward passes whose multi-workgroup launch gives up at a barrier.

The host forces it with the barrier's own limit (0 ticks: every wait that is
not over at once ends) or by withholding a workgroup; every kernel returns
normally, and no GPU work is broken on purpose.
"""
import time

import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
KEYS = ("dx0", "dv0", "dw_edge", "dmu")


def _sim(sc, **kw):
    from paper_2106_05306_amd.sim import Sim
    kw.setdefault("precision", "mixed")
    return Sim.from_scene(sc, device=DEV, **kw)


def _seed(sc):
    return torch.tensor(np.random.default_rng(2).normal(size=(sc.n_nodes, 3)), device=DEV)


def _one_workgroup(sc, monkeypatch, **kw):
    with monkeypatch.context() as mp:
        mp.setenv("DIFFCLOTH_FWD_WGS", "0")
        s = _sim(sc, **kw)
        assert s.stats()["fwd_workgroups"] == 1
        traj = s.forward(sc.steps, trajectory=True)[2].clone()
        g = s.backward(_seed(sc))
        out = traj, {k: g[k].clone() for k in KEYS}
        s.close()
    return out


def test_overlapped_factorisation_after_a_launch_that_gave_up(monkeypatch):
    # the records of the first, failed attempt are new memory, and its steps
    # are factored behind it all the same
    sc = scenes.discretized_sphere_drop(0, n=24, steps=24, level=1)
    kw = dict(adj_solver="direct", adj_tol=1e-10, adj_max_iters=10)
    traj, g = _one_workgroup(sc, monkeypatch, **kw)
    monkeypatch.setenv("DIFFCLOTH_FWD_WGS", "16")
    monkeypatch.setenv("DIFFCLOTH_MW_SPIN", "0")
    junk = [torch.full((64 << 20,), 0x55, dtype=torch.uint8, device=DEV) for _ in range(4)]
    s = _sim(sc, **kw)
    del junk                                         # what the records are allocated from
    t = s.forward(sc.steps, trajectory=True)[2]
    assert torch.equal(t, traj)
    out = s.backward(_seed(sc))
    for k in KEYS:
        assert torch.equal(out[k], g[k]), k
    s.close()


def test_launches_behind_one_that_gave_up_do_not_wait_again(monkeypatch):
    from paper_2106_05306_amd import _binding as B
    sc = scenes.c2_sphere_drop(0, n=24, steps=24)
    limit = 0.25
    monkeypatch.setenv("DIFFCLOTH_FWD_WGS", "8")
    monkeypatch.setenv("DIFFCLOTH_MW_SPIN", str(int(limit * 1e8)))
    monkeypatch.setenv("DIFFCLOTH_MW_TEST_ABSENT", "1")
    s = _sim(sc, checkpoint_every=2)                 # twelve launches
    t0 = time.perf_counter()
    with pytest.raises(B.SimError) as e:
        s.forward(sc.steps)
    assert e.value.code == B.SIM_ESYNC
    assert time.perf_counter() - t0 < 4 * limit
    s.close()


def test_a_handle_that_gave_up_keeps_to_one_workgroup(monkeypatch):
    sc = scenes.c2_sphere_drop(0, n=24, steps=6)
    limit = 0.25
    traj, _ = _one_workgroup(sc, monkeypatch)
    monkeypatch.setenv("DIFFCLOTH_FWD_WGS", "8")
    monkeypatch.setenv("DIFFCLOTH_MW_SPIN", str(int(limit * 1e8)))
    monkeypatch.setenv("DIFFCLOTH_MW_TEST_ABSENT", "2")
    s = _sim(sc)
    assert s.stats()["fwd_workgroups"] == 8
    took = []
    for _ in range(3):
        t0 = time.perf_counter()
        t = s.forward(sc.steps, trajectory=True)[2]
        took.append(time.perf_counter() - t0)
        assert torch.equal(t, traj)
        assert s.stats()["fwd_workgroups"] == 1
    assert took[0] >= limit and max(took[1:]) < limit, took
    s.close()


def _batch(monkeypatch, **kw):
    """Scenes for a batch, in contact from the first steps on, their results on
    one workgroup, and handles of which the second never waits for others."""
    scs = [scenes.c2_sphere_drop(0, n=n, steps=st) for n, st in ((28, 7), (10, 9), (40, 5))]
    for sc in scs:
        sc.X = sc.X - np.array([0.0, 0.27, 0.0])
    ref = [_one_workgroup(sc, monkeypatch, **kw) for sc in scs]
    monkeypatch.setenv("DIFFCLOTH_MW_SPIN", "2000000")
    sims = []
    for sc in scs:
        with monkeypatch.context() as mp:
            if sc.n_nodes <= 100:
                mp.setenv("DIFFCLOTH_FWD_WGS", "1")
            sims.append(_sim(sc, **kw))
    assert [s.stats()["fwd_workgroups"] > 1 for s in sims] == [True, False, True]
    return scs, ref, sims


@pytest.mark.parametrize("absent", ["2", "3"])      # at the first barrier, or in the second step
def test_batch_members_that_gave_up_run_again(monkeypatch, absent):
    from paper_2106_05306_amd.sim import batch_backward, batch_forward
    scs, ref, sims = _batch(monkeypatch)
    monkeypatch.setenv("DIFFCLOTH_MW_TEST_ABSENT", absent)
    for _ in range(2):
        outs = batch_forward(sims, [sc.steps for sc in scs])
        for sc, (traj, _), s, (x, _) in zip(scs, ref, sims, outs):
            assert torch.equal(x, traj[-1]) and s.stats()["fwd_workgroups"] == 1
            assert all(torch.equal(s.state(n)[0], traj[n]) for n in range(sc.steps + 1))
    for s, (_, g), out in zip(sims, ref, batch_backward(sims, [_seed(sc) for sc in scs])):
        for k in KEYS:
            assert torch.equal(out[k], g[k]), k
        s.close()


@pytest.mark.parametrize("warm", [False, True])
@pytest.mark.parametrize("at", [0, 1])
def test_job_chunks_that_gave_up_run_again(monkeypatch, warm, at):
    # the larger two give up in the second step of their chunk number `at`, while an adjoint job
    # advances beside them; each chunk counts once
    from paper_2106_05306_amd.sim import batch_advance
    scs, ref, sims = _batch(monkeypatch, warm_start=warm)
    iters = []
    for sc in scs:
        with monkeypatch.context() as mp:
            mp.setenv("DIFFCLOTH_FWD_WGS", "0")
            s = _sim(sc, warm_start=warm)
            s.forward(sc.steps)
            iters.append(s.stats()["fwd_iters_total"])
            s.close()
    adj = _sim(scs[1], warm_start=warm)
    adj.job_forward(scs[1].steps)
    while batch_advance([adj], [16])[0] > 0:
        pass
    adj.job_backward(_seed(scs[1]))
    for sc, s in zip(scs, sims):
        s.job_forward(sc.steps)
    left = batch_advance(sims, [2, 2, 2]) if at else [sc.steps for sc in scs]
    assert [s.stats()["fwd_workgroups"] > 1 for s in sims] == [True, False, True]
    monkeypatch.setenv("DIFFCLOTH_MW_TEST_ABSENT", "3")
    n = 0
    while sum(left) > 0:
        on = [i for i in range(3) if left[i] > 0]
        group = [sims[i] for i in on] + ([adj] if n < 3 else [])
        got = batch_advance(group, [2] * len(on) + ([3] if n < 3 else []))
        for i, k in zip(on, got):
            assert k == max(0, left[i] - 2)
            left[i] = k
        if n < 3:
            assert got[-1] == 9 - 3 * (n + 1)
        n += 1
    assert n >= 3
    assert [s.stats()["fwd_workgroups"] for s in sims] == [1, 1, 1]
    g = adj.job_grads()
    for k in KEYS:
        assert torch.equal(g[k], ref[1][1][k]), k
    adj.close()
    for sc, s, (traj, _), it in zip(scs, sims, ref, iters):
        assert all(torch.equal(s.state(j)[0], traj[j]) for j in range(sc.steps + 1))
        assert s.stats()["fwd_iters_total"] == it
        s.close()


@pytest.mark.parametrize("solver", ["iterative", "direct"])
@pytest.mark.parametrize("first", ["backward", "state", "modes"])
def test_replayed_segments_that_gave_up_run_again(monkeypatch, solver, first):
    sc = scenes.c2_sphere_drop(0, n=24, steps=11)
    sc.X = sc.X - np.array([0.0, 0.27, 0.0])        # in contact from the first steps on
    kw = dict(adj_solver=solver, adj_tol=1e-9, adj_max_iters=40)
    traj, g = _one_workgroup(sc, monkeypatch, **kw)
    with monkeypatch.context() as mp:
        mp.setenv("DIFFCLOTH_FWD_WGS", "0")
        r = _sim(sc, **kw)
        r.forward(sc.steps)
        modes = [r.modes(n) for n in range(sc.steps)]
        r.close()
    assert any((m != 0).any() for m in modes)
    monkeypatch.setenv("DIFFCLOTH_FWD_WGS", "16")
    monkeypatch.setenv("DIFFCLOTH_MW_SPIN", "2000000")
    s = _sim(sc, checkpoint_every=4, **kw)
    assert torch.equal(s.forward(sc.steps, trajectory=True)[2], traj)
    assert s.stats()["fwd_workgroups"] == 16
    monkeypatch.setenv("DIFFCLOTH_MW_TEST_ABSENT", "3")
    seed = _seed(sc)
    check = {"backward": lambda: [torch.equal(v, g[k]) for o in [s.backward(seed)] for k, v in o.items() if k in KEYS],
             "state": lambda: [torch.equal(s.state(n)[0], traj[n]) for n in range(sc.steps + 1)],
             "modes": lambda: [np.array_equal(s.modes(n), modes[n]) for n in range(sc.steps)]}
    assert all(check[first]())
    assert s.stats()["fwd_workgroups"] == 1
    assert all(all(c()) for c in check.values())
    s.close()
