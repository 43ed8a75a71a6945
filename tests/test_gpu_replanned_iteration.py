"""An iteration after the edge map has been planned again with other clusters: the
coloured variant runs whichever way the plan of now has, fused over fixed-order lists
or as separate loops.  Against the oracle to 1e-12, normwise per variable."""
import numpy as np
import pytest

import meshgen
import oracle
import paper_1403_7209_amd as pk
from tests._util import normwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first", [512, 0, 1024])
@pytest.mark.parametrize("second", [0, 1024, 256])
def test_coloured_iteration_after_replanning(first, second):
    print(f"[replanned, clusters of {first} then {second}]", flush=True)
    m = meshgen.build_mesh(8, 1, 0.2)
    q = meshgen.state(m.N, m.perm)
    p = pk.FluxProblem(pk.Context("cuda:0"), m.e2n, m.w, m.vol, q, cluster_size=first)
    dt = oracle.dt(m.e2n, q, m.w, m.vol)
    want, ss = oracle.rk_iteration(m.e2n, q, m.w, m.vol, dt)
    for K in (first, second):
        if K == second:
            p.ctx.plan(p.e2n, cluster_size=second)
            p.node_new, p.edge_new = p.ctx.get_perm(p.nodes, p.N), p.ctx.get_perm(p.edges, p.E)
            p.w_t.copy_(p.nodes_in(m.w, edges=True))
            p.vol_t.copy_(p.nodes_in(m.vol[None])[0])
        p.qa.copy_(p.nodes_in(q))
        p.rk_iteration(dt)
        p.ctx.sync()
        assert normwise(p.nodes_out(p.qa), want) <= 1e-12
        assert normwise(p.ss.cpu().numpy().T, ss.T) <= 1e-12
    assert np.isfinite(p.rms()).all()
