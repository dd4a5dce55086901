"""The Krylov fallback of the iterative adjoint at the edges of its dot products.

A wavefront takes 64 entries of a vector, eight basis vectors at a time, and
wavefronts that a short vector leaves idle take other basis vectors: sizes
below one wavefront (12 entries), just above one (75), where two and one group
of wavefronts fit (363, 588), at most one entry a thread (972) and more (1083),
each with up to 60 basis vectors and restarts.  One adjoint step per mesh
against the oracle's direct solve at the GPU's recorded state.  The solver stops
at |P^-1 (g - A z)| <= tol |P^-1 g|, so z is within kappa_2(P^-1 A) tol of the
solution in the 2-norm; a factor of 10 covers the gradients formed from it.
"""
import numpy as np
import pytest
import scipy.sparse as sp

import scenes
from oracle import diffcloth_oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOL = 1e-12


def _kappa(model, rec):
    h, m = model.h, model.m
    Hm = (O._kron3(h * h * model.K_s) - O.delta_P(model, rec.x1)).toarray()
    Tb = np.tile(np.eye(3), (m, 1, 1))
    if rec.contact.nodes.size:
        Tb[rec.contact.nodes] = O.contact_jacobian_blocks(rec.contact, h)
    A = np.diag(np.repeat(model.mass, 3)) + Hm @ O._blockdiag3(np.transpose(Tb, (0, 2, 1))).toarray()
    P = np.diag(np.repeat(model.mass, 3)) + O._kron3(h * h * model.K_s).toarray()
    return np.linalg.cond(np.linalg.solve(P, A))


@pytest.mark.parametrize("n", [2, 5, 11, 14, 18, 19])
def test_krylov_solve_matches_the_oracle(n):
    from paper_2106_05306_amd.sim import Sim
    sc = scenes.c1_napkin(0, n=n, steps=2)
    sc.X = sc.X - np.array([0.0, 0.1995, 0.0])              # half a millimetre above the ground: contact at once
    sc.v0 = np.random.default_rng(n).normal(0.0, 0.05, sc.X.shape)
    sc.v0[sc.attach] = 0.0
    s = Sim.from_scene(sc, device=DEV, precision="fp64", adj_solver="iterative", adj_tol=TOL, adj_max_iters=3000)
    s.forward(2)
    model = O.Model(sc)
    x0, v0 = (t.cpu().numpy() for t in s.state(1))
    x1, v1 = (t.cpu().numpy() for t in s.state(2))
    rec = O.forward_step(model, x0, v0, 1)
    at_gpu = O.StepRecord(x0, v0, x1, v1, rec.contact, rec.iters)
    gx, gv = np.random.default_rng(5).normal(size=(2, sc.n_nodes, 3))
    out = s.adjoint_step(1, torch.tensor(gx, device=DEV), torch.tensor(gv, device=DEV))
    st = s.stats()
    print(n, "krylov", st["adj_krylov_total"], "fixed point", st["adj_iters_total"], flush=True)
    assert out["status"] in (0, 1)                           # 1: by the fallback
    dx, dv, dw, dmu, _ = O.backward_step(model, at_gpu, gx, gv, 1)
    bound = 10 * _kappa(model, at_gpu) * TOL
    for key, ref in (("dx0", dx), ("dv0", dv), ("dw_edge", dw[:model.n_spring])):
        got = out[key].cpu().numpy()
        assert np.linalg.norm(got - ref) <= bound * max(np.linalg.norm(ref), 1e-300), key
    s.close()
