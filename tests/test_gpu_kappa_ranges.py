"""Screening constants far outside the physical range, where coordinates scaled by
kappa, their cubes and exponents leave the range of a number format.  A tiny
positive kappa is no screening to rounding, a huge one leaves the Laplace
kernels alone; neither may give infinities or NaN.

FP32 far fields are held to the FP64 assembled far field (unscaled coordinates,
the library's exponential) with the repository's bound for FP32 far fields, 2e-5;
the treecode adds its own error, below 1e-6 at degree 7 and theta 0.5.  What is
below FP32's range (Yukawa kernels alone at a huge kappa: 1e-125) is zero there."""
import numpy as np
import pytest

import inputs

pytestmark = pytest.mark.gpu

pbm = pytest.importorskip("paper_2108_10481_amd")

TINY = float(np.finfo(np.float32).tiny)
FORMS = [(pbm.PB_DIRECT_INT, 1.0, 1.0), (pbm.PB_JUFFER, 1.0, 1.0), (pbm.PB_MULLER_EXT, 1.0, 1.0),
         (pbm.PB_CFIE_EXT, 0.0, 1.0), (pbm.PB_CFIE_EXT, 0.0, 0.0)]   # the last two: some, no Laplace terms


def _opts(form, kappa, **kw):
    return pbm.pb_default_options(formulation=form[0], cfie_alpha=form[1], cfie_beta=form[2], kappa=kappa, **kw)


def _far(m, x, opt):
    with pbm.MeshHandle(m.xyz, m.tri, opt) as h:
        return pbm.pb_mesh_apply(h, x, pbm.PB_APPLY_FAR_ONLY), h.info()


@pytest.fixture(scope="module")
def star6():
    return inputs.star_surface(4, 6, 5.0)[0]       # 720 triangles


@pytest.fixture(scope="module")
def star14():
    return inputs.star_surface(4, 14, 5.0)[0]      # 3920


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("kappa", [1e-300, 1e-20, 1e-14, 1e-13, 1e-12, 1e-10, 1e-9, 1e-6, 1e3, 1e8, 1e12])
def test_fp32_far_field(star6, star14, form, kappa):
    for m, modes in ((star6, (dict(), dict(far_symmetric=1), dict(far_symmetric=-1))),
                     (star14, (dict(), dict(operator_mode=pbm.PB_TREECODE, tree_degree=7, tree_theta=0.5)))):
        x = np.random.default_rng(41).standard_normal(2 * m.n_vertices)
        ref, _ = _far(m, x, _opts(form, kappa, operator_mode=pbm.PB_ASSEMBLED))
        for kw in modes:
            y, _ = _far(m, x, _opts(form, kappa, precision=pbm.PB_FP32, **kw))
            assert np.isfinite(y).all(), (m.n_triangles, kw)
            assert np.linalg.norm(y - ref) <= 2.1e-5 * np.linalg.norm(ref) + TINY, (m.n_triangles, kw)


@pytest.mark.parametrize("form", FORMS[:2])
def test_fp32_graded_edges(form):
    """Short edges on a large surface: the screening is not below rounding across
    it, and distances of the short edges' size have cubes out of range."""
    m = inputs.bipyramid(510, 4.0, 4.0)
    x = np.random.default_rng(43).standard_normal(2 * m.n_vertices)
    ref, _ = _far(m, x, _opts(form, 1e-9, operator_mode=pbm.PB_ASSEMBLED))
    for sym in (0, 1):
        y, info = _far(m, x, _opts(form, 1e-9, precision=pbm.PB_FP32, far_symmetric=sym))
        assert info["far_symmetric"] == 0
        assert np.linalg.norm(y - ref) <= 2.1e-5 * np.linalg.norm(ref)


def test_batch_with_negligible_screening():
    """Requests without screening to rounding beside screened ones, twice the same
    meshes: bitwise their single solves."""
    reqs = []
    for k, kappa in enumerate((1e-14, 0.125, 1e-14, 1e6)):
        m, shape = inputs.star_surface(7 + k // 2, 5 + k // 2, 5.0)
        c = inputs.charges_in_star(30 + k, 5, shape)
        reqs.append((pbm.MeshHandle(m.xyz, m.tri, pbm.pb_default_options(kappa=kappa, precision=pbm.PB_FP32)), (c.xyz, c.q)))
    hs, sets = [r[0] for r in reqs], [r[1] for r in reqs]
    single = [pbm.pb_mesh_solve(h, *s) for h, s in zip(hs, sets)]
    for _ in range(2):
        for a, b in zip(single, pbm.pb_solve_batch(hs, sets)):
            assert a["status"] == pbm.PB_OK and np.isfinite(a["dG"])
            assert a["dG"] == b["dG"] and a["iterations"] == b["iterations"] and np.array_equal(a["phi"], b["phi"])


@pytest.mark.parametrize("kappa", [2e8, 1e9, 3e9, 4.5e9, 1e10, 1e12])
def test_near_blocks_at_huge_kappa(star6, kappa):
    """Sauter-Schwab blocks past the exponent range of the near field's exponential:
    at 4 Gauss points r is above 1e-6 edge lengths at every point, so exp(-kappa r)
    is below exp(-100) of the Laplace kernel's value, K_Y's by a further kappa r;
    the Laplace blocks do not see kappa."""
    t = np.repeat(np.arange(6, dtype=np.int32), star6.n_triangles)
    s = np.tile(np.arange(star6.n_triangles, dtype=np.int32), 6)
    share = (star6.tri[t][:, :, None] == star6.tri[s][:, None, :]).any(axis=(1, 2))
    t, s = t[share], s[share]
    with pbm.MeshHandle(star6.xyz, star6.tri, pbm.pb_default_options(kappa=kappa)) as h:
        b = pbm.pb_mesh_near_blocks(h, t, s)
    with pbm.MeshHandle(star6.xyz, star6.tri, pbm.pb_default_options(kappa=0.125)) as h:
        ref = pbm.pb_mesh_near_blocks(h, t, s)
    assert np.isfinite(b).all()
    assert np.abs(b[:, 2:]).max() <= 1e-30 * np.abs(ref[:, :2]).max()
    assert np.abs(b[:, :2] - ref[:, :2]).max() <= 1e-14 * np.abs(ref[:, :2]).max()


@pytest.mark.parametrize("precision", [pbm.PB_FP64, pbm.PB_FP32])
def test_solve_at_huge_kappa(star6, precision):
    """The solution no longer depends on kappa once every exponential has
    underflowed: kappa 1e12 against 1e8, to the solver's tolerance."""
    c = inputs.charges_ball(51, 5, 1.0)
    out = []
    for kappa in (1e8, 1e12):
        with pbm.MeshHandle(star6.xyz, star6.tri, pbm.pb_default_options(kappa=kappa, precision=precision, tol=1e-7)) as h:
            out.append(pbm.pb_mesh_solve(h, c.xyz, c.q))
    a, b = out
    assert a["status"] == b["status"] == pbm.PB_OK
    assert abs(a["dG"] - b["dG"]) <= 1e-5 * abs(a["dG"])


@pytest.mark.parametrize("alpha,beta", [(1e-42, 1.0), (1.0, 1e-42), (1e-30, 1e-30), (1e-11, 1e-13), (1e-42, 0.0)])
@pytest.mark.parametrize("mode", [pbm.PB_MATRIX_FREE, pbm.PB_TREECODE])
def test_fp32_tiny_combined_field_constants(star14, alpha, beta, mode):
    """Combined fields whose Laplace terms are tiny beside the Yukawa ones, over the
    range of FP32 as a ratio, against the FP64 matrix-free far field; bounds as above."""
    x = np.random.default_rng(47).standard_normal(2 * star14.n_vertices)
    form = (pbm.PB_CFIE_EXT, alpha, beta)
    ref, _ = _far(star14, x, _opts(form, 0.125))
    y, _ = _far(star14, x, _opts(form, 0.125, precision=pbm.PB_FP32, operator_mode=mode, tree_degree=7, tree_theta=0.5))
    assert np.isfinite(y).all()
    assert np.linalg.norm(y - ref) <= 2.1e-5 * np.linalg.norm(ref)
