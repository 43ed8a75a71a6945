"""FP32 storage: which way round an edge is evaluated.

FP32 arithmetic does not give F(a, b, w) = -F(b, a, -w) to the bit, so a loop that
evaluates an edge once for each end has to do so in the same direction as the
loops that evaluate it once: the coloured variant's two increments of an edge
cancel exactly, and the owner variant turns the edges between two clusters, and
only those, whichever of its loops a mesh's size selects.

The increments are FP32 values added up in FP64, so two loops that evaluate every
edge alike agree to the rounding of FP64 sums of at most a few dozen terms:
1e-13 of the largest increment, where one edge turned round shows as 1e-8.  The
sums of a node's residuals cancel to some 1/30 of its increments: 1e-12."""
import numpy as np
import pytest
import torch

import meshgen
import paper_1403_7209_amd as pk
from tests._util import normwise

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-12


def box(n):
    """A closed box in an order of its own clusters: (e2n, w, vol, q)."""
    m = meshgen.build_mesh(n, 0, 0.2)
    q = meshgen.state(m.N, m.perm)
    ctx = pk.Context(None)
    nodes, edges = ctx.decl_set(m.N, "nodes"), ctx.decl_set(m.E, "edges")
    e2n = ctx.decl_map(edges, nodes, 2, m.e2n, 0, "e2n")
    ctx.plan(e2n, renumber="morton", coords=m.xyz)
    new = ctx.get_perm(nodes, m.N)
    out = np.empty_like(q), np.empty_like(m.vol)
    out[0][:, new], out[1][new] = q, m.vol
    return new[m.e2n].astype(np.int32), m.w, out[1], out[0]


def with_chain(g, N):
    """The graph with a chain of further nodes, N in all."""
    e2n, w, vol, q = g
    n0, rng = len(vol), np.random.default_rng(2)
    i = np.arange(n0, N - 1, dtype=np.int32)
    more = N - n0
    return (np.concatenate([e2n, np.stack([i, i + 1], 1)]),
            np.concatenate([w, 1e-3 * rng.normal(size=(3, len(i)))], 1),
            np.concatenate([vol, np.ones(more)]), np.concatenate([q, q[:, rng.integers(0, n0, more)]], 1))


def problem(g, K=512, **kw):
    return pk.FluxProblem(pk.Context(DEV), g[0], g[1], g[2], g[3], fp32=True, cluster_size=K, **kw)


def residual(p, variant):
    r = torch.zeros(6, p.N, dtype=torch.float64, device=DEV)
    p.residual(p.qa, r, variant)
    lam = p.lam.zero_()
    p.ctx.edge_specrad(p.edges, p.e2n, p.dat(p.qa), p.w, p.lam_d, p.gamma, variant)
    p.ctx.sync()
    return p.nodes_out(r), p.nodes_out(lam[None])


def first_norms(p, variant):
    p.rk_iteration(1e-4, variant)
    p.ctx.sync()
    return p.ss[0].cpu().numpy()


# below and above the sizes where the small-mesh loop ends, for the coloured variant
# (47^3 = 103,823 nodes) and for the owner variant (30^3 = 27,000)
@pytest.mark.parametrize("n", [8, 9, 16, 47])
def test_coloured_residual_conserves(n):
    print(f"[fp32 conservation {n}^3]", flush=True)
    p = problem(box(n))
    r, _ = residual(p, pk.COLOURED)
    assert (np.abs(r.sum(axis=1)) <= TOL * np.abs(r).sum(axis=1)).all()


@pytest.mark.parametrize("n,N", [(8, 512), (9, 729), (16, 4096), (16, 100000)])
def test_coloured_agrees_with_one_evaluation_per_edge(n, N):
    """The fixed-order loops against the mini-partitions, which a plan without owner
    clusters runs: residual, spectral radii and the first stage's norms."""
    g = box(n)
    if N > n ** 3:
        g = with_chain(g, N)
    print(f"[fp32 coloured {n}^3 of {N} nodes]", flush=True)
    a, b = problem(g), problem(g, K=0)
    (ra, la), (rb, lb) = residual(a, pk.COLOURED), residual(b, pk.COLOURED)
    assert normwise(ra, rb) <= TOL and normwise(la, lb) <= TOL
    assert normwise(first_norms(a, pk.COLOURED), first_norms(b, pk.COLOURED)) <= TOL


@pytest.mark.parametrize("n,K", [(9, 512), (16, 512), (16, 64), (16, 200), (26, 512)])
def test_owner_of_a_small_mesh_agrees_with_the_clusters(n, K):
    """A small mesh's loop against the loop over clusters, which the same nodes run in
    a mesh of 30,000: the same clusters of consecutive nodes in both."""
    g = box(n)
    n0 = n ** 3
    print(f"[fp32 owner {n}^3 K={K}]", flush=True)
    n1 = (n0 + K - 1) // K * K  # the chain starts a cluster of its own
    pad = (g[0], g[1], np.concatenate([g[2], np.ones(n1 - n0)]),
           np.concatenate([g[3], g[3][:, :n1 - n0]], 1))
    a, b = problem(g, K, renumber="none"), problem(with_chain(pad, 30000), K, renumber="none")
    (ra, la), (rb, lb) = residual(a, pk.OWNER), residual(b, pk.OWNER)
    assert normwise(ra, rb[:, :n0]) <= TOL and normwise(la, lb[:, :n0]) <= TOL
    ss = first_norms(a, pk.OWNER)
    assert normwise(ss, (rb[:, :n0] ** 2).sum(axis=1)) <= TOL
