"""GPU: the far field that evaluates every unordered triangle pair once, at the
edges of its tiles (64 triangles, in FP32 in groups of 16): less than one group, one tile and a remainder, many tiles with
a ragged last one and separated tile pairs.  The reference is the FP64 oracle's
dense system.

Tolerances: FP64 1e-12, FP32 2e-6 (a kernel value carries a few FP32 roundings
of 6e-8, sums of a few thousand of them in one slot and FP64 across slots stay
below ten of them)."""
import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu

pbm = pytest.importorskip("paper_2108_10481_amd")

MESHES = {"ico1": lambda: inputs.icosphere(1, 2.0),          # 20 triangles
          "bipyramid33": lambda: inputs.bipyramid(33, 2.0, 2.0),   # 66: one tile and two triangles
          "star6": lambda: inputs.star_surface(4, 6, 5.0)[0]}    # 720: 12 tiles, the last of 16


@pytest.fixture(scope="module")
def cases():
    return {name: make() for name, make in MESHES.items()}


@pytest.mark.parametrize("name", sorted(MESHES))
@pytest.mark.parametrize("form", [pbm.PB_DIRECT_EXT_PERM, pbm.PB_JUFFER, pbm.PB_PMCHWT_EXT])
@pytest.mark.parametrize("kappa", [0.0, 0.125])
def test_product_at_tile_edges(cases, name, form, kappa):
    m = cases[name]
    A = oracle.system_matrix(m, 4.0, 80.0, kappa, form)
    x = np.random.default_rng(23).standard_normal(2 * m.n_vertices)
    ref = A @ x
    for precision, sym, tol in ((pbm.PB_FP64, 0, 1e-12), (pbm.PB_FP32, 0, 2e-6), (pbm.PB_FP32, -1, 2e-6)):
        opt = pbm.pb_default_options(formulation=form, precision=precision, kappa=kappa, far_symmetric=sym)
        with pbm.MeshHandle(m.xyz, m.tri, opt) as h:
            y = pbm.pb_mesh_apply(h, x)
            again = pbm.pb_mesh_apply(h, x)
        assert np.array_equal(y, again)
        assert np.linalg.norm(y - ref) < tol * np.linalg.norm(ref), (precision, sym)
        assert np.abs(y - ref).max() < 10 * tol * np.abs(ref).max(), (precision, sym)


@pytest.mark.parametrize("freq", [5, 8, 9, 10])   # 500, 1280, 1620, 2000 triangles: 4, 2, 2 parts, whole items
@pytest.mark.parametrize("form", [pbm.PB_DIRECT_EXT_PERM, pbm.PB_JUFFER])
def test_parts_of_items(freq, form):
    """FP32 items cut into parts by column groups, against the FP64 product per
    ordered pair (PB_AUTO stays on it); the tolerance is the one above."""
    m = inputs.star_surface(4, freq, 5.0)[0]
    x = np.random.default_rng(31).standard_normal(2 * m.n_vertices)
    out = []
    for precision, mode in ((pbm.PB_FP64, pbm.PB_AUTO), (pbm.PB_FP32, pbm.PB_MATRIX_FREE)):
        opt = pbm.pb_default_options(formulation=form, precision=precision, operator_mode=mode)
        with pbm.MeshHandle(m.xyz, m.tri, opt) as h:
            out.append(pbm.pb_mesh_apply(h, x))
    ref, y = out
    assert np.linalg.norm(y - ref) < 2e-6 * np.linalg.norm(ref)
    assert np.abs(y - ref).max() < 2e-5 * np.abs(ref).max()
