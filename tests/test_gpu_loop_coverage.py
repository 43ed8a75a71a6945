"""Instances of the edge loops that no other test reaches: the owner loop over
clusters of sizes without a compile-time instance, on meshes above the small-mesh
limit; its workgroups of 1024 and 768 threads with many cut visits per cluster
(boxes in RCM order), in both storage forms; and the mini-partitions of the
coloured variant (plans without owner clusters, or with large ones), every loop and
bit for bit.  Against the oracle: FP64 to 1e-12, FP32 storage from rounded inputs to
1e-5, normwise per variable."""
import functools

import numpy as np
import pytest
import torch

import meshgen
import oracle
import paper_1403_7209_amd as pk
from tests._util import normwise

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = {False: 1e-12, True: 1e-5}


@functools.lru_cache(maxsize=1)
def reference(n, split):
    """A box and the oracle's results on it: {fp32: ...} for the loops with an FP32 form."""
    m = meshgen.build_mesh(n, split, 0.2)
    q = meshgen.state(m.N, m.perm)
    rbar = np.random.default_rng(3).normal(size=(6, m.N))
    dx = meshgen.edge_vectors(m)
    G = oracle.gradient(m.e2n, q, m.w)
    ref = dict(rbar=rbar, dx=dx, G=G, res2=oracle.residual2(m.e2n, q, G, m.vol, m.w, dx),
               adj=oracle.adjoint(m.e2n, q, m.w, rbar))
    for fp32 in (False, True):
        q_, w_ = (x.astype(np.float32).astype(np.float64) if fp32 else x for x in (q, m.w))
        dt = oracle.dt(m.e2n, q_, w_, m.vol)
        ref[fp32] = dict(res=oracle.residual(m.e2n, q_, w_), dt=dt,
                         it=oracle.rk_iteration(m.e2n, q_, w_, m.vol, dt))
    return m, q, ref


def check(n, split, variant, fixed_order=False, **plan):
    m, q, ref = reference(n, split)
    print(f"[{n}^3 variant {variant} {plan}]", flush=True)
    ctx = pk.Context(DEV)
    if plan.get("renumber") == "morton":
        plan["coords"] = m.xyz
    p64 = pk.FluxProblem(ctx, m.e2n, m.w, m.vol, q, **plan)
    p32 = pk.FluxProblem(ctx, m.e2n, m.w, m.vol, q, fp32=True, like=p64)
    p64.set_edge_vectors(ref["dx"])
    f64 = dict(dtype=torch.float64, device=DEV)

    def close(t, want, tol, edges=False):
        return normwise(p64.nodes_out(t, edges=edges), want) <= tol

    def results(p):  # the loops of both storage forms
        r = torch.zeros(6, m.N, **f64)
        p.residual(p.qa, r, variant)
        dt = p.compute_dt(0.5, variant)
        q0 = p.qa.clone()
        p.rk_iteration(ref[p.fp32]["dt"], variant)
        p.ctx.sync()
        out = r, torch.full((1,), dt, **f64), p.qa.clone(), p.ss.clone()
        p.qa.copy_(q0)
        return out

    def results64():
        p = p64
        G, r2, qb = (torch.zeros(k, m.N, **f64) for k in (18, 6, 6))
        nb = torch.zeros(3, m.E, **f64)
        p.gradient(p.qa, G, variant)
        p.residual2(p.qa, p.nodes_in(ref["G"]), r2, variant)
        ctx.edge_flux_adjoint(p.edges, p.e2n, p.dat(p.qa), p.w, p.dat(p.nodes_in(ref["rbar"])),
                              p.dat(qb), p.dat(nb, edges=True), p.gamma, variant)
        ctx.sync()
        return G, r2, qb, nb

    for p in (p64, p32):
        tol, want = TOL[p.fp32], ref[p.fp32]
        r, dt, q1, ss = out = results(p)
        assert close(r, want["res"], tol), (p.fp32, "residual")
        assert abs(dt.item() - want["dt"]) <= tol * want["dt"]
        assert close(q1, want["it"][0], tol), (p.fp32, "iteration")
        assert normwise(ss.cpu().numpy().T, want["it"][1].T) <= tol
        if fixed_order:
            assert all(torch.equal(a, b) for a, b in zip(out, results(p)))
    G, r2, qb, nb = out = results64()
    assert close(G, ref["G"], TOL[False]) and close(r2, ref["res2"], TOL[False])
    assert close(qb, ref["adj"][0], TOL[False]) and close(nb, ref["adj"][1], TOL[False], edges=True)
    if fixed_order:
        assert all(torch.equal(a, b) for a, b in zip(out, results64()))
    return p64


@pytest.mark.parametrize("K", [64, 96, 200, 256, 500])
def test_owner_run_time_cluster_sizes(K):
    """27,000 nodes: above the limit below which the small-mesh loop takes over."""
    p = check(30, 0, pk.OWNER, renumber="morton", cluster_size=K)
    # the stage through the entry point that allocates nothing
    out, qa = [], p.dat(p.qa)
    for call in (p.ctx.edge_flux_stage, p.ctx.edge_flux_stage_noalloc):
        q1 = torch.empty_like(p.qa)
        ss = torch.zeros(6, dtype=torch.float64, device=DEV)
        call(p.edges, p.e2n, qa, p.w, qa, p.vol, p.dat(q1), 1e-4, ss, p.gamma)
        p.ctx.sync()
        out.append((p.nodes_out(q1), ss.cpu().numpy()))
    assert normwise(out[1][0], out[0][0]) <= TOL[False] and normwise(out[1][1], out[0][1]) <= TOL[False]


@pytest.mark.parametrize("n", [47, 55])
def test_owner_wide_workgroups_with_many_cut_visits(n):
    """RCM order: 203 clusters (1024 threads) and 325 (768 for the flux), whose cut
    visits take several rounds."""
    check(n, 0, pk.OWNER)


def test_coloured_fixed_order_fp32_above_the_small_mesh_limit():
    check(47, 0, pk.COLOURED, fixed_order=True)


@pytest.mark.parametrize("bs,csort", [(64, False), (256, True), (512, False), (1024, True)])
@pytest.mark.parametrize("K", [0, 1024])
def test_coloured_mini_partitions(K, bs, csort):
    check(8, 1, pk.COLOURED, fixed_order=True, cluster_size=K, block_size=bs, colour_sort=csort)


def test_coloured_mini_partitions_rk_separate_loops():
    """Large partitions over more than one round of threads, and Morton order."""
    check(20, 0, pk.COLOURED, fixed_order=True, renumber="morton", cluster_size=0, block_size=1024)
