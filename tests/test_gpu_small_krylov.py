"""Captured GMRES iterations whose Krylov steps run in one block (at most 1024
unknowns): fewer unknowns than a wavefront, a remainder, exactly the limit and one
past it.  Eager launches take the separate kernels with the same arithmetic, so
everything is compared bitwise; a batch runs the solves side by side."""
import numpy as np
import pytest

import inputs

pytestmark = pytest.mark.gpu

pbm = pytest.importorskip("paper_2108_10481_amd")

MESHES = {10: lambda: inputs.bipyramid(3, 4.0, 4.0), 724: lambda: inputs.star_surface(4, 6, 5.0)[0],
          1024: lambda: inputs.bipyramid(510, 4.0, 4.0), 1026: lambda: inputs.bipyramid(511, 4.0, 4.0)}


def _same(a, b):
    assert a["iterations"] == b["iterations"] and a["dG"] == b["dG"] and a["status"] == b["status"]
    assert np.array_equal(a["phi"], b["phi"]) and np.array_equal(a["dphi"], b["dphi"])


@pytest.mark.parametrize("precision", [pbm.PB_FP64, pbm.PB_FP32])
@pytest.mark.parametrize("sizes", [(10,), (724,), (1024,), (1026,), (10, 1024, 724), (724, 1026)])
def test_small_iterations_match_eager(sizes, precision):
    meshes = [MESHES[n]() for n in sizes]
    assert [2 * m.n_vertices for m in meshes] == list(sizes)
    sets = [inputs.charges_ball(40 + k, 5, 1.0) for k in range(len(sizes))]
    sets = [(c.xyz, c.q) for c in sets]

    def handles(**kw):
        opt = pbm.pb_default_options(formulation=pbm.PB_JUFFER, precision=precision, operator_mode=pbm.PB_MATRIX_FREE,
                                     max_iter=40, **kw)
        return [pbm.MeshHandle(m.xyz, m.tri, opt) for m in meshes]

    eager = [pbm.pb_mesh_solve(h, *c) for h, c in zip(handles(use_graph=0), sets)]
    hs = handles()
    single = [pbm.pb_mesh_solve(h, *c) for h, c in zip(hs, sets)]
    again = [pbm.pb_mesh_solve(h, *c) for h, c in zip(hs, sets)]
    batch = pbm.pb_solve_batch(hs, sets)
    for e, s, a, b in zip(eager, single, again, batch):
        assert e["iterations"] >= 2
        _same(e, s)
        _same(s, a)
        _same(s, b)


@pytest.mark.parametrize("precision", [pbm.PB_FP64, pbm.PB_FP32])
@pytest.mark.parametrize("sizes", [(70,), (600,), (724,), (768,), (770,), (724, 70), (768, 770)])
def test_long_solves_change_kernels(sizes, precision):
    """Solves that run on past the iterations one block serves: the separate kernels
    take over between two checks, bitwise as eager launches throughout, also in a
    second solve and in batches."""
    meshes = [inputs.bipyramid(n // 2 - 2, 4.0, 4.0) for n in sizes]
    sets = [inputs.charges_ball(80 + k, 5, 1.0) for k in range(len(sizes))]
    sets = [(c.xyz, c.q) for c in sets]

    def handles(**kw):
        opt = pbm.pb_default_options(precision=precision, tol=1e-300, max_iter=57, preconditioner=pbm.PB_PREC_NONE, **kw)
        return [pbm.MeshHandle(m.xyz, m.tri, opt) for m in meshes]

    eager = [pbm.pb_mesh_solve(h, *c) for h, c in zip(handles(use_graph=0), sets)]
    hs = handles()
    single = [pbm.pb_mesh_solve(h, *c) for h, c in zip(hs, sets)]
    again = [pbm.pb_mesh_solve(h, *c) for h, c in zip(hs, sets)]
    batch = pbm.pb_solve_batch(hs, sets)
    for e, s, a, b in zip(eager, single, again, batch):
        assert e["iterations"] == 57
        _same(e, s)
        _same(s, a)
        _same(s, b)
