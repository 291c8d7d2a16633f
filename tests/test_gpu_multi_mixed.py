"""Mixed-precision batches whose matrix products are split over the columns.

The 16-bit product of the inner sweeps and the accurate product of the
refinement sweeps serve all systems of a batch at once and cut the columns into
parts.  Sizes: fewer rows than one tile of either, row counts that leave a
remainder, more steps than parts; batches of one, of several, full, and full
plus one.  A single solve of the same handle refines against the same FP32
matrix to the same tolerance tau, so two solutions differ by at most
2 tau |P^-1 A|^-1 |pb| <= 2 tau cond |x|; cond < 1e3 for these surfaces,
which at tau = 1e-10 bounds the relative difference by 2e-7.
"""
import numpy as np
import pytest

import inputs

pytestmark = pytest.mark.gpu

pbm = pytest.importorskip("paper_2108_10481_amd")

MESHES = {"bipyramid3": lambda: inputs.bipyramid(3, 4.0, 4.0),      # 10 rows
          "ico1": lambda: inputs.icosphere(1, 4.0),                  # 24
          "bipyramid33": lambda: inputs.bipyramid(33, 4.0, 4.0),    # 70
          "star6": lambda: inputs.star_surface(4, 6, 5.0)[0]}        # 724


@pytest.mark.parametrize("nb", [1, 3, 16, 17])
@pytest.mark.parametrize("prec", [pbm.PB_MIXED_BF16, pbm.PB_MIXED_FP16])
@pytest.mark.parametrize("name,form", [("bipyramid3", pbm.PB_JUFFER), ("ico1", pbm.PB_DIRECT_EXT_PERM),
                                       ("bipyramid33", pbm.PB_DIRECT_EXT_PERM), ("star6", pbm.PB_JUFFER)])
def test_batched_products_match_single_solves(name, form, prec, nb):
    m = MESHES[name]()
    sets = [inputs.charges_ball(300 + k, 5, 1.0) for k in range(nb)]
    opt = pbm.pb_default_options(formulation=form, precision=prec, operator_mode=pbm.PB_ASSEMBLED, tol=1e-10,
                                 max_iter=400)
    with pbm.MeshHandle(m.xyz, m.tri, opt) as h:
        multi = pbm.pb_solve_multi(h, [(c.xyz, c.q) for c in sets])
        single = [pbm.pb_mesh_solve(h, c.xyz, c.q) for c in sets]
    for a, b in zip(multi, single):
        assert a["status"] == pbm.PB_OK and a["rel_residual"] <= 1.001e-10
        for f in ("phi", "dphi"):
            assert np.abs(a[f] - b[f]).max() <= 2e-7 * np.linalg.norm(b[f])
