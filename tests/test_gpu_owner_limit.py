"""Where the owner variant leaves the small-mesh loop: at 48 clusters, whatever their
size.  The small-mesh loop also serves the coloured variant there, in FP64 with the
same bits; the loop over clusters adds up in another order.  Both sides against the
oracle to 1e-12, normwise per variable."""
import numpy as np
import pytest
import torch

import oracle
import paper_1403_7209_amd as pk
from tests._util import normwise

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("K", [64, 100, 256, 512])
def test_limit_in_clusters(K, over):
    N = 48 * K + over
    print(f"[owner limit: {N} nodes, K={K}]", flush=True)
    rng = np.random.default_rng(K)
    i = np.arange(N)
    e2n = np.concatenate([np.stack([i, (i + d) % N], 1) for d in (1, 5, 17, 40)]).astype(np.int32)
    w = rng.normal(size=(3, len(e2n)))
    rho, u = 0.9 + 0.2 * rng.random(N), 0.6 * rng.random((3, N)) - 0.3
    q = np.concatenate([rho[None], rho * u, (2.5 + 0.5 * rho * (u * u).sum(0))[None], rho[None]])
    p = pk.FluxProblem(pk.Context(DEV), e2n, w, np.ones(N), q, cluster_size=K)
    assert p.info["nclusters"] == 48 + over and p.info["coloured_ok"]
    out = []
    for v in (pk.OWNER, pk.COLOURED):
        r = torch.zeros(6, N, dtype=torch.float64, device=DEV)
        p.residual(p.qa, r, v)
        p.ctx.sync()
        out.append(r)
    ref = oracle.residual(e2n, q, w)
    assert all(normwise(p.nodes_out(r), ref) <= 1e-12 for r in out)
    assert torch.equal(*out) == (over == 0)
