"""The treecode on tiles (FP32, theta <= 0.8), at the edges of its pieces: proxy
counts below, at and over a staged block (27, 216, 512), a ragged last tile,
no separated cluster, the largest theta of the path and one past it, every sum of
kernels, no screening.  The reference is the FP64 direct product.

Tolerance: twice the FP64 treecode's own error at the same degree and theta (its
clusters have other bounds but pass the same test), and the rounding: a pair's
r^2 = |S|^2 - 2 S.X + |X|^2 keeps its rounding (1.5 x 2^-24) times at most
((1 + theta) / (1 - theta))^2, the kernels r^-3 one and a half times that; 1e-6
for the rest, as in the direct FP32 product."""
import numpy as np
import pytest

import inputs

pytestmark = pytest.mark.gpu

pbm = pytest.importorskip("paper_2108_10481_amd")


@pytest.fixture(scope="module")
def mesh():
    return inputs.star_surface(4, 14, 5.0)[0]


@pytest.mark.parametrize("degree,theta", [(2, 0.01), (2, 0.3), (2, 0.8), (2, 0.81), (5, 0.5), (7, 0.5)])
@pytest.mark.parametrize("form", [pbm.PB_DIRECT_EXT_PERM, pbm.PB_JUFFER, pbm.PB_MULLER_EXT])
@pytest.mark.parametrize("kappa", [0.0, 0.125])
def test_tiled_treecode_matches_direct(mesh, degree, theta, form, kappa):
    x = np.random.default_rng(29).standard_normal(2 * mesh.n_vertices)

    def product(precision, **kw):
        opt = pbm.pb_default_options(formulation=form, precision=precision, kappa=kappa, **kw)
        with pbm.MeshHandle(mesh.xyz, mesh.tri, opt) as h:
            y = pbm.pb_mesh_apply(h, x)
            assert np.array_equal(y, pbm.pb_mesh_apply(h, x))
        return y

    tree = dict(operator_mode=pbm.PB_TREECODE, tree_degree=degree, tree_theta=theta)
    ref = product(pbm.PB_FP64, operator_mode=pbm.PB_MATRIX_FREE)
    scale, top = np.linalg.norm(ref), np.abs(ref).max()
    d64 = product(pbm.PB_FP64, **tree) - ref
    d32 = product(pbm.PB_FP32, **tree) - ref
    lost = ((1 + theta) / (1 - theta)) ** 2 if theta <= 0.8 else 0.0
    tol = 1.5 * 1.5 * 2.0 ** -24 * lost + 1e-6
    print("%.2e %.2e" % (np.linalg.norm(d64) / scale, np.linalg.norm(d32) / scale))
    assert np.linalg.norm(d32) < 2 * np.linalg.norm(d64) + tol * scale
    assert np.abs(d32).max() < 2 * np.abs(d64).max() + 10 * tol * top


def test_memory_stays_bounded_at_small_theta():
    """Nearly every pair of tiles direct: the handle stays within its estimate (a slot
    per pair would take 20 GB)."""
    m = inputs.star_surface(4, 100, 28.0)[0]      # 200000 triangles
    opt = pbm.pb_default_options(precision=pbm.PB_FP32, operator_mode=pbm.PB_TREECODE, tree_degree=2, tree_theta=0.01)
    with pbm.MeshHandle(m.xyz, m.tri, opt) as h:
        assert h.info()["device_bytes"] <= pbm.pb_estimate_device_bytes(m.xyz, m.tri, opt)


@pytest.mark.parametrize("form", [pbm.PB_DIRECT_EXT_PERM, pbm.PB_JUFFER])
@pytest.mark.parametrize("theta,degree", [(0.01, 2), (0.25, 7)])
def test_general_path_on_the_tile_order(form, theta, degree):
    """Under a memory budget that leaves the tiles' slots out, the general path runs
    on the triangles' k-d order; tolerance as above."""
    m = inputs.star_surface(4, 32, 9.0)[0]        # 20480 triangles, 320 tiles
    x = np.random.default_rng(31).standard_normal(2 * m.n_vertices)
    tree = dict(operator_mode=pbm.PB_TREECODE, tree_degree=degree, tree_theta=theta, source_chunks=1)
    out = []
    for kw in (dict(), dict(tree), dict(tree, precision=pbm.PB_FP32), dict(tree, precision=pbm.PB_FP32)):
        opt = pbm.pb_default_options(formulation=form, **kw)
        if len(out) == 3:
            opt.memory_budget = pbm.pb_estimate_device_bytes(m.xyz, m.tri, opt)
        with pbm.MeshHandle(m.xyz, m.tri, opt) as h:
            out.append(pbm.pb_mesh_apply(h, x))
    ref, y64, tiled, general = out
    assert not np.array_equal(tiled, general)
    scale, err64 = np.linalg.norm(ref), np.linalg.norm(y64 - ref)
    for y in (tiled, general):
        assert np.linalg.norm(y - ref) < 2 * err64 + (2e-7 + 2e-6) * scale
