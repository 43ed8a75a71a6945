"""The ring kernel of the geometry loop with its batches split over several
workgroups per chunk: meshes of 1, 7, 16 and 27 chunks (8 groups, some without a
batch), one of 275 (4 groups), against the oracle and, bit for bit, against a
second run."""
import numpy as np
import pytest
import torch

import meshgen
import oracle
import paper_1403_7209_amd as pk
from tests._util import normwise

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-12  # normwise per variable, as for the one-workgroup form


@pytest.mark.parametrize("n,K", [(5, 512), (15, 512), (20, 512), (12, 64), (26, 64)])
def test_ring_groups(n, K):
    m = meshgen.build_mesh(n, 0, 0.2)
    print(f"[ring groups {n}^3 K={K}: {(m.N + K - 1) // K} chunks]", flush=True)
    t2n = m.tets()
    t2e = meshgen.tet_edges(m, t2n)
    p = pk.FluxProblem(pk.Context(DEV), m.e2n, m.w, m.vol, np.ones((6, m.N)), renumber="morton",
                       coords=m.xyz, cluster_size=K, tets=t2n, tet_edges=t2e)
    w_ref, vol_ref = oracle.geometry(m.e2n, t2n, t2e, m.xyz)
    x, out = p.nodes_in(m.xyz), []
    for _ in range(2):
        w = torch.full((3, m.E), 1e30, dtype=torch.float64, device=DEV)
        vol = torch.full((m.N,), 1e30, dtype=torch.float64, device=DEV)
        p.geometry(x, w, vol, access=pk.WRITE)
        p.ctx.sync()
        out.append((w, vol))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert normwise(p.nodes_out(w, edges=True), w_ref) <= TOL
    assert normwise(p.nodes_out(vol[None]), vol_ref[None]) <= TOL
