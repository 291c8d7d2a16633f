"""Charges and evaluation points so far away that their squared distances
overflow: their projections and potentials are zero to rounding, and the other
points of the call are unaffected."""
import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu

pbm = pytest.importorskip("paper_2108_10481_amd")
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("far", [1e153, 1e155, 1e200, 1.7e308])
def test_distant_points(far):
    m = inputs.icosphere(4, 2.0)
    rng = np.random.default_rng(61)
    tr = rng.standard_normal(2 * m.n_vertices)
    pts = inputs.charges_ball(62, 6, 1.0).xyz
    pts[1] = [far, 0.0, 0.0]
    pts[4] = [-far, far, -far]
    near = [0, 2, 3, 5]
    q = rng.uniform(-1.0, 1.0, 6)
    with pbm.MeshHandle(m.xyz, m.tri, pbm.pb_default_options()) as h:
        v = pbm.pb_mesh_reaction_potential(h, tr[:m.n_vertices], tr[m.n_vertices:], pts)
        ref = pbm.pb_mesh_reaction_potential(h, tr[:m.n_vertices], tr[m.n_vertices:], pts[near])
        b = pbm.pb_mesh_rhs(h, pts, q)
        bref = pbm.pb_mesh_rhs(h, pts[near], q[near])
        t, p = torch.from_numpy(tr).cuda(), torch.from_numpy(pts).cuda()
        out = torch.zeros(6, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        pbm.pb_mesh_reaction_potential_noalloc(h, t.data_ptr(), 6, p.data_ptr(), out.data_ptr())
        pbm.pb_mesh_synchronize(h)
    assert np.array_equal(out.cpu().numpy(), v)
    assert np.abs(v[[1, 4]]).max() < 1e-140
    assert np.abs(v[near] - ref).max() <= 1e-14 * np.abs(ref).max()
    assert np.abs(b - bref).max() <= 1e-14 * np.abs(bref).max()


@pytest.mark.parametrize("freq", [1, 4, 6, 7])
@pytest.mark.parametrize("npts", [1, 7, 65, 512, 513])
def test_small_potentials(freq, npts):
    """Few points of a small mesh (a block per point) and one past either limit: against
    the oracle, and bitwise the allocation-free entry point."""
    m = inputs.icosphere(freq, 2.0)
    tr = np.random.default_rng(67).standard_normal(2 * m.n_vertices)
    pts = inputs.charges_ball(68, npts, 1.0).xyz
    with pbm.MeshHandle(m.xyz, m.tri, pbm.pb_default_options()) as h:
        v = pbm.pb_mesh_reaction_potential(h, tr[:m.n_vertices], tr[m.n_vertices:], pts)
        t, p = torch.from_numpy(tr).cuda(), torch.from_numpy(pts).cuda()
        out = torch.zeros(npts, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        pbm.pb_mesh_reaction_potential_noalloc(h, t.data_ptr(), npts, p.data_ptr(), out.data_ptr())
        pbm.pb_mesh_synchronize(h)
    assert np.array_equal(out.cpu().numpy(), v)
    ref = oracle.reaction_potential(m, tr[:m.n_vertices], tr[m.n_vertices:], pts)
    assert np.abs(v - ref).max() <= 1e-13 * np.abs(ref).max() * np.sqrt(m.n_triangles)
