"""The link form of the geometry reverse (meshes whose tets close a ring around
every edge) against the oracle: boxes so small that every difference wraps,
chunks that end at a block of 2,048 nodes, an order that scatters a node's
neighbours (chunks cut by their LDS), volume adjoints that are zero, equal or
arbitrary, an output that already holds values; the same bits on every run."""
import numpy as np
import pytest
import torch

import meshgen
import oracle
import paper_1403_7209_amd as pk
from tests._util import normwise

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-12  # normwise per variable, as for the record form

CASES = [(3, 0, "morton", 512), (4, 1, "rcm", 64), (8, 1, "morton", 1024), (12, 0, "none", 512),
         (13, 0, "morton", 512), (16, 1, "rcm", 256), (20, 0, "none", 512), (24, 1, "morton", 512)]


@pytest.mark.parametrize("n,split,order,K", CASES)
def test_link_reverse(n, split, order, K):
    m = meshgen.build_mesh(n, split, 0.2)
    print(f"[link reverse {n}^3 {order} K={K}]", flush=True)
    t2n = m.tets()
    t2e = meshgen.tet_edges(m, t2n)
    p = pk.FluxProblem(pk.Context(DEV), m.e2n, m.w, m.vol, np.ones((6, m.N)), renumber=order,
                       coords=m.xyz, cluster_size=K, tets=t2n, tet_edges=t2e)
    x = p.nodes_in(m.xyz)
    rng = np.random.default_rng(n)
    wbar = rng.normal(size=(3, m.E))
    for volbar in (np.zeros(m.N), np.full(m.N, 2.5), rng.normal(size=m.N)):
        ref = oracle.geometry_adjoint(m.e2n, t2n, t2e, m.xyz, wbar, volbar)
        start = np.abs(ref).max() * rng.normal(size=(3, m.N))
        out = []
        for _ in range(2):
            xbar = p.nodes_in(start)
            p.geometry_adjoint(x, p.nodes_in(wbar, edges=True),
                               p.nodes_in(volbar[None])[0].contiguous(), xbar)
            p.ctx.sync()
            out.append(xbar)
        assert torch.equal(*out)
        assert normwise(p.nodes_out(out[0]), start + ref) <= TOL
