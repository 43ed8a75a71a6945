"""The fixed-order edge loop (coloured variant, and every loop of a small mesh's
owner variant) against the oracle, at the edges of its chunks and rounds:
meshes of fewer nodes than a chunk, of one chunk more, with a last chunk of one
node, at both sides of the small-mesh limits (24,576 nodes for the owner variant,
98,304 for the coloured one), cluster sizes with and without a compile-time
instance, and a node with more edges than a round has visits.  Results must be the same bits on every run."""
import numpy as np
import pytest
import torch

import meshgen
import oracle
import paper_1403_7209_amd as pk
from tests._util import normwise

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-12  # normwise per variable, as for every FP64 loop


class Graph:
    """Edges between random or given nodes, with random weights and volumes."""

    def __init__(self, N, e2n, seed=5):
        rng = np.random.default_rng(seed)
        self.N, self.e2n = N, np.asarray(e2n, np.int32)
        self.w = rng.normal(size=(3, len(self.e2n)))
        self.vol = 0.5 + rng.random(N)
        self.dx = 0.001 * rng.normal(size=(3, len(self.e2n)))
        rho, p = 0.9 + 0.2 * rng.random(N), 0.9 + 0.2 * rng.random(N)
        u = 0.6 * rng.random((3, N)) - 0.3
        self.q = np.concatenate([rho[None], rho * u, (p / 0.4 + 0.5 * rho * (u * u).sum(0))[None],
                                 (rho * rng.random(N))[None]])


def chain(N):  # every node to its next and its next but two
    i = np.arange(N)
    e = np.concatenate([np.stack([i[:-1], i[1:]], 1), np.stack([i[:-3], i[3:]], 1)])
    return Graph(N, e)


def star(N):  # node 0 in every edge, the orientation alternating
    e = np.stack([np.zeros(N - 1, int), np.arange(1, N)], 1)
    e[::2] = e[::2, ::-1]
    return Graph(N, e)


def box(n):
    m = meshgen.build_mesh(n, 0, 0.2)
    g = Graph(m.N, m.e2n)
    g.w, g.vol, g.dx = m.w, m.vol, meshgen.edge_vectors(m)
    return g


CASES = {  # graph, cluster size, variants
    "one-chunk": (lambda: box(6), 512, (pk.COLOURED,)),
    "fine-513": (lambda: chain(513), 512, (pk.COLOURED, pk.OWNER)),
    "fine-33-of-64": (lambda: chain(65), 64, (pk.COLOURED, pk.OWNER)),
    "fine-box11": (lambda: box(11), 512, (pk.COLOURED, pk.OWNER)),
    "owner-limit": (lambda: chain(24576), 512, (pk.COLOURED, pk.OWNER)),
    "fine-limit": (lambda: chain(98304), 512, (pk.COLOURED,)),
    "above-limit": (lambda: chain(98305), 512, (pk.COLOURED,)),
    "run-time-chunk": (lambda: chain(98305), 200, (pk.COLOURED,)),
    "box47-of-64": (lambda: box(47), 64, (pk.COLOURED,)),
    "box47": (lambda: box(47), 512, (pk.COLOURED,)),
    # no two-level colouring: only the owner variant
    "star": (lambda: star(1500), 512, (pk.OWNER,)),
}


def close(p, t, ref, edges=False):
    return normwise(p.nodes_out(t, edges=edges), ref) <= TOL


@pytest.mark.parametrize("name", list(CASES))
def test_loops_and_iteration(name):
    make, K, variants = CASES[name]
    g = make()
    print(f"[fixed order {name}: {g.N} nodes, {len(g.e2n)} edges]", flush=True)
    ctx = pk.Context(DEV)
    p = pk.FluxProblem(ctx, g.e2n, g.w, g.vol, g.q, cluster_size=K)
    p.set_edge_vectors(g.dx)
    res = oracle.residual(g.e2n, g.q, g.w)
    G = oracle.gradient(g.e2n, g.q, g.w)
    res2 = oracle.residual2(g.e2n, g.q, G, g.vol, g.w, g.dx)
    rbar = np.random.default_rng(3).normal(size=(6, g.N))
    qb, nb = oracle.adjoint(g.e2n, g.q, g.w, rbar)
    dt = oracle.dt(g.e2n, g.q, g.w, g.vol)
    q1, ss1 = oracle.rk_iteration(g.e2n, g.q, g.w, g.vol, dt)
    f64 = dict(dtype=torch.float64, device=DEV)
    for v in variants:
        runs = []
        for _ in range(2):
            r, gr, r2 = torch.zeros(6, g.N, **f64), torch.zeros(18, g.N, **f64), torch.zeros(6, g.N, **f64)
            q, n = torch.zeros(6, g.N, **f64), torch.zeros(3, len(g.e2n), **f64)
            p.residual(p.qa, r, v)
            p.gradient(p.qa, gr, v)
            p.residual2(p.qa, p.nodes_in(G), r2, v)
            ctx.edge_flux_adjoint(p.edges, p.e2n, p.dat(p.qa), p.w, p.dat(p.nodes_in(rbar)),
                                  p.dat(q), p.dat(n, edges=True), p.gamma, v)
            ctx.sync()
            runs.append((r, gr, r2, q, n))
        assert all(torch.equal(a, b) for a, b in zip(*runs))
        assert close(p, r, res) and close(p, gr, G) and close(p, r2, res2)
        assert close(p, q, qb) and close(p, n, nb, edges=True)
        assert abs(p.compute_dt(0.5, v) - dt) <= 1e-12 * dt
        q0 = p.qa.clone()
        out = []
        for _ in range(2):
            p.qa.copy_(q0)
            p.rk_iteration(dt, v)
            ctx.sync()
            out.append((p.qa.clone(), p.ss.clone()))
        p.qa.copy_(q0)
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
        assert close(p, out[0][0], q1)
        assert normwise(out[0][1].cpu().numpy().T, ss1.T) <= TOL
        if v == pk.OWNER:  # WRITE overwrites
            r = torch.full((6, g.N), 1e30, **f64)
            p.residual(p.qa, r, v, res_access=pk.WRITE)
            ctx.sync()
            assert close(p, r, res)


@pytest.mark.parametrize("N", [24577, 65536, 98304, 131072, 131073])
def test_owner_workgroup_widths(N):
    """The owner variant above the small-mesh limit and on both sides of one
    workgroup per CU (256 clusters; 128 for the gradient's two halves)."""
    g = chain(N)
    print(f"[owner widths: {g.N} nodes]", flush=True)
    ctx = pk.Context(DEV)
    f64 = dict(dtype=torch.float64, device=DEV)
    res, G = oracle.residual(g.e2n, g.q, g.w), oracle.gradient(g.e2n, g.q, g.w)
    rbar = np.random.default_rng(3).normal(size=(6, g.N))
    qb, nb = oracle.adjoint(g.e2n, g.q, g.w, rbar)
    dt = oracle.dt(g.e2n, g.q, g.w, g.vol)
    q1, ss1 = oracle.rk_iteration(g.e2n, g.q, g.w, g.vol, dt)
    p = pk.FluxProblem(ctx, g.e2n, g.w, g.vol, g.q)
    p.set_edge_vectors(g.dx)
    r, gr, r2 = torch.empty(6, g.N, **f64), torch.empty(18, g.N, **f64), torch.empty(6, g.N, **f64)
    q, n = torch.zeros(6, g.N, **f64), torch.zeros(3, len(g.e2n), **f64)
    p.residual(p.qa, r, pk.OWNER, res_access=pk.WRITE)
    p.gradient(p.qa, gr, pk.OWNER, pk.WRITE)
    p.residual2(p.qa, p.nodes_in(G), r2, pk.OWNER, pk.WRITE)
    ctx.edge_flux_adjoint(p.edges, p.e2n, p.dat(p.qa), p.w, p.dat(p.nodes_in(rbar)), p.dat(q),
                          p.dat(n, edges=True), p.gamma, pk.OWNER)
    ctx.sync()
    assert close(p, r, res) and close(p, gr, G) and close(p, q, qb) and close(p, n, nb, edges=True)
    assert close(p, r2, oracle.residual2(g.e2n, g.q, G, g.vol, g.w, g.dx))
    assert abs(p.compute_dt(0.5, pk.OWNER) - dt) <= 1e-12 * dt
    p.rk_iteration(dt, pk.OWNER)
    ctx.sync()
    assert close(p, p.qa, q1) and normwise(p.ss.cpu().numpy().T, ss1.T) <= TOL
    # the coloured iteration's partial sums share the buffer with other rows
    p.qa.copy_(p.nodes_in(g.q))
    p.rk_iteration(dt)
    ctx.sync()
    assert close(p, p.qa, q1) and normwise(p.ss.cpu().numpy().T, ss1.T) <= TOL


def test_coloured_iteration_takes_up_the_residual():
    """What p.res holds enters the first stage, and p.res is zero afterwards, fused or not."""
    g = box(9)
    ctx = pk.Context(DEV)
    p = pk.FluxProblem(ctx, g.e2n, g.w, g.vol, g.q)
    q0, src = p.qa.clone(), torch.randn(6, g.N, dtype=torch.float64, device=DEV)
    out = []
    for fused in (False, True):
        p.qa.copy_(q0)
        p.res.copy_(src)
        p.rk_iteration(1e-4, fused=fused)
        ctx.sync()
        out.append((p.qa.cpu().numpy(), p.ss.cpu().numpy()))
        assert not p.res.any()
    assert normwise(out[1][0], out[0][0]) <= TOL and normwise(out[1][1].T, out[0][1].T) <= TOL


def test_coloured_iteration_fp32_and_local_steps():
    g = box(9)
    ctx = pk.Context(DEV)
    for fp32, tol in ((False, TOL), (True, 1e-5)):
        p = pk.FluxProblem(ctx, g.e2n, g.w, g.vol, g.q, fp32=fp32)
        q0, out = p.qa.clone(), []
        for fused in (False, True):
            p.qa.copy_(q0)
            p.compute_local_dt()
            p.rk_iteration_local(fused=fused)
            ctx.sync()
            out.append((p.qa.double().cpu().numpy(), p.ss.cpu().numpy()))
        assert normwise(out[1][0], out[0][0]) <= tol and normwise(out[1][1].T, out[0][1].T) <= tol
