"""The small-mesh edge loop where nodes have many edges: degrees on both sides of a
batch of slots, of the limit above which a wavefront adds up a node's sums, and of a
round of 512 visits, several such nodes in one chunk of 32.  Against the oracle to
1e-12 (normwise per variable), and the same bits on every run."""
import numpy as np
import pytest
import torch

import oracle
import paper_1403_7209_amd as pk
from tests._util import normwise

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-12


@pytest.mark.parametrize("degrees", [(1, 2, 3, 4, 5, 7, 8, 9), (29, 30, 31, 32, 33), (60, 200, 140, 40, 70),
                                     (511, 512, 513), (1, 1025, 300)])
@pytest.mark.parametrize("N", [1040, 2000])
def test_nodes_of_many_edges(N, degrees):
    print(f"[hubs {degrees} of {N} nodes]", flush=True)
    rng = np.random.default_rng(7)
    hubs = len(degrees)
    e = [np.stack([np.full(d, h), hubs + rng.choice(N - hubs, min(d, N - hubs), replace=False)], 1)
         if d <= N - hubs else
         np.stack([np.full(d, h), hubs + np.arange(d) % (N - hubs)], 1) for h, d in enumerate(degrees)]
    i = np.arange(N - 1)
    e2n = np.concatenate(e + [np.stack([i, i + 1], 1)]).astype(np.int32)
    e2n[::2] = e2n[::2, ::-1].copy()
    E = len(e2n)
    w, dx, vol = rng.normal(size=(3, E)), 1e-3 * rng.normal(size=(3, E)), 0.5 + rng.random(N)
    rho, pr, u = 0.9 + 0.2 * rng.random(N), 0.9 + 0.2 * rng.random(N), 0.6 * rng.random((3, N)) - 0.3
    q = np.concatenate([rho[None], rho * u, (pr / 0.4 + 0.5 * rho * (u * u).sum(0))[None],
                        (rho * rng.random(N))[None]])
    rbar = rng.normal(size=(6, N))
    G = oracle.gradient(e2n, q, w)
    qb, nb = oracle.adjoint(e2n, q, w, rbar)
    dt = oracle.dt(e2n, q, w, vol)
    q1, ss1 = oracle.rk_iteration(e2n, q, w, vol, dt)
    ctx = pk.Context(DEV)
    # in the order given: the hubs lie in one chunk
    p = pk.FluxProblem(ctx, e2n, w, vol, q, renumber="none", halo_order=False)
    p.set_edge_vectors(dx)
    f64 = dict(dtype=torch.float64, device=DEV)
    runs = []
    for _ in range(2):
        r, gr, r2, qbar = (torch.empty(k, N, **f64) for k in (6, 18, 6, 6))
        nbar = torch.empty(3, E, **f64)
        p.residual(p.qa, r, pk.OWNER, pk.WRITE)
        p.gradient(p.qa, gr, pk.OWNER, pk.WRITE)
        p.residual2(p.qa, p.nodes_in(G), r2, pk.OWNER, pk.WRITE)
        ctx.edge_flux_adjoint(p.edges, p.e2n, p.dat(p.qa), p.w, p.dat(p.nodes_in(rbar)), p.dat(qbar),
                              p.dat(nbar, edges=True), p.gamma, pk.OWNER, pk.WRITE)
        step = p.compute_dt(0.5, pk.OWNER)
        q0 = p.qa.clone()
        p.rk_iteration(dt, pk.OWNER)
        ctx.sync()
        runs.append((r, gr, r2, qbar, nbar, p.qa.clone(), p.ss.clone()))
        p.qa.copy_(q0)
        assert abs(step - dt) <= TOL * dt
    assert all(torch.equal(a, b) for a, b in zip(*runs))
    r, gr, r2, qbar, nbar, qn, ss = runs[0]
    for t, want in ((r, oracle.residual(e2n, q, w)), (gr, G), (qbar, qb), (qn, q1),
                    (r2, oracle.residual2(e2n, q, G, vol, w, dx))):
        assert normwise(p.nodes_out(t), want) <= TOL
    assert normwise(p.nodes_out(nbar, edges=True), nb) <= TOL
    assert normwise(ss.cpu().numpy().T, ss1.T) <= TOL
