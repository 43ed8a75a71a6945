"""opf_rk_iteration refuses a bad argument before it launches anything: every dat's
set, dimension and type, those of the second stage buffer (first used by the second
stage) among them.  On a host-only context the refusal comes before the missing
device; on a GPU the state buffers and the residual are left as they were."""
import ctypes

import numpy as np
import pytest
import torch

import meshgen
import paper_1403_7209_amd as pk

NAMES = ("q", "n", "vol", "qb", "qc", "res")
DIMS = dict(q=6, n=3, vol=1, qb=6, qc=6, res=6)
DEV = "cuda:0"


def bad_dats(name):
    """(dimension, type, on the other set) of a dat in place of `name`, and the status."""
    d, edges = DIMS[name], name == "n"
    out = [((d + 1, pk.F64, edges), pk.ESIZE), ((d, pk.F64, not edges), pk.EINVAL)]
    if name != "q":  # the state's type is the loop's
        out.append(((d, pk.F32, edges), pk.ETYPE))
    return out


@pytest.mark.parametrize("name", NAMES)
def test_shapes_and_types_without_a_device(name):
    ctx = pk.Context(None)
    nodes, edges = ctx.decl_set(4, "nodes"), ctx.decl_set(3, "edges")
    e2n = ctx.decl_map(edges, nodes, 2, np.array([[0, 1], [1, 2], [2, 3]], np.int32), 0, "e2n")
    ctx.plan(e2n)
    out = ctypes.c_int32()

    def dat(dim, dtype, on_edges):
        assert ctx.lib.opf_decl_dat(ctx._ctx, edges if on_edges else nodes, dim, dtype, None, 8, b"",
                                    ctypes.byref(out)) == 0
        return out.value

    alpha = (ctypes.c_double * 5)(*pk.RK_ALPHA)
    for variant in (pk.OWNER, pk.COLOURED):
        if name == "res" and variant == pk.OWNER:
            continue
        a = {k: dat(DIMS[k], pk.F64, k == "n") for k in NAMES}
        if variant == pk.OWNER:
            a["res"] = -1

        def call():
            return ctx.lib.opf_rk_iteration(ctx._ctx, edges, e2n, a["q"], a["n"], a["vol"], -1, a["qb"],
                                            a["qc"], a["res"], 1.4, alpha, ctypes.c_void_p(4096),
                                            variant, None)

        assert call() == pk.EDEVICE
        for spec, status in bad_dats(name):
            a[name] = dat(*spec)
            assert call() == status


@pytest.mark.parametrize("n", [0, 4, 6])
def test_five_coefficients(n):
    """Fewer used to be filled up with zeros."""
    ctx = pk.Context(None)
    with pytest.raises(ValueError):
        ctx.rk_iteration(0, 0, 0, 0, 0, 0, 0, [0.1] * n, None)


@pytest.mark.gpu
@pytest.mark.parametrize("variant", [pk.OWNER, pk.COLOURED])
def test_nothing_is_launched_for_a_bad_second_buffer(variant):
    m = meshgen.build_mesh(6, 0, 0.2)
    p = pk.FluxProblem(pk.Context(DEV), m.e2n, m.w, m.vol, meshgen.state(m.N, m.perm))
    print(f"[bad second buffer, variant {variant}]", flush=True)
    f64 = dict(dtype=torch.float64, device=DEV)
    p.res.normal_()
    qb, res, ss = torch.full_like(p.qa, 7.0), p.res.clone(), torch.full((5, 6), 7.0, **f64)
    bad = [p.dat(torch.empty(7, p.N, **f64)), p.dat(torch.empty(6, p.E, **f64), edges=True),
           p.dat(torch.empty(6, p.N, dtype=torch.float32, device=DEV))]
    for qc in bad:
        with pytest.raises(pk.OpfError):
            p.ctx.rk_iteration(p.edges, p.e2n, p.dat(p.qa), p.w, p.vol, p.dat(qb), qc, [1e-4] * 5, ss,
                               res=p.res_d if variant == pk.COLOURED else -1, variant=variant)
        p.ctx.sync()
        assert (qb == 7.0).all() and (ss == 7.0).all() and torch.equal(p.res, res)
