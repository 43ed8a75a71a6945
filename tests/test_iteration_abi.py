"""Argument checks of opf_rk_iteration that need no GPU: every handle is checked
before it is used, and what cannot run is an error code."""
import ctypes

import numpy as np
import pytest

import paper_1403_7209_amd as pk


@pytest.fixture()
def host():
    ctx = pk.Context(None)
    nodes, edges = ctx.decl_set(4, "nodes"), ctx.decl_set(3, "edges")
    e2n = ctx.decl_map(edges, nodes, 2, np.array([[0, 1], [1, 2], [2, 3]], np.int32), 0, "e2n")
    ctx.plan(e2n)
    out = ctypes.c_int32()

    def dat(s, dim):
        assert ctx.lib.opf_decl_dat(ctx._ctx, s, dim, 0, None, 8, b"", ctypes.byref(out)) == 0
        return out.value

    d = dict(q=dat(nodes, 6), n=dat(edges, 3), vol=dat(nodes, 1), dt=-1, qb=dat(nodes, 6),
             qc=dat(nodes, 6), res=-1)
    alpha, ss = (ctypes.c_double * 5)(*pk.RK_ALPHA), ctypes.c_void_p(4096)

    def call(variant=pk.OWNER, alpha=alpha, ss=ss, **over):
        a = {**d, **over}
        return ctx.lib.opf_rk_iteration(ctx._ctx, edges, e2n, a["q"], a["n"], a["vol"], a["dt"],
                                        a["qb"], a["qc"], a["res"], 1.4, alpha, ss, variant, None)

    call.res = dat(nodes, 6)
    return call


def test_a_host_only_context_cannot_run(host):
    assert host() == pk.EDEVICE
    assert host(pk.COLOURED, res=host.res) == pk.EDEVICE


@pytest.mark.parametrize("bad", [-1, 999, -7])
@pytest.mark.parametrize("name", ["q", "n", "vol", "qb", "qc"])
def test_invalid_handles(host, name, bad):
    assert host(**{name: bad}) == pk.EINVAL


def test_other_invalid_arguments(host):
    assert host(dt=999) == pk.EINVAL
    assert host(pk.COLOURED, res=999) == pk.EINVAL
    assert host(pk.COLOURED) == pk.EINVAL and host(res=host.res) == pk.EINVAL
    for v in (pk.ATOMIC, pk.FLAT, pk.COLOURED_LDS_ATOMIC, 17, -1):
        assert host(v) == pk.EINVAL
    assert host(alpha=None) == pk.EINVAL and host(ss=None) == pk.EINVAL
