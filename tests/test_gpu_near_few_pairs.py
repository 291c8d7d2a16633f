"""Sauter-Schwab blocks where the pairs are few: one wavefront per pair (any small
number of pairs at these orders), blocks of 64 pairs with eight or four
wavefronts, at every order that changes the choice, pair counts that leave blocks
ragged, and both ranges of the exponential.  The reference is the oracle; the
tolerance is that of the near-field test at order 4."""
import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu

pbm = pytest.importorskip("paper_2108_10481_amd")


def _pairs(m):
    fans = [[] for _ in range(m.n_vertices)]
    for t, v in enumerate(m.tri):
        for k in v:
            fans[k].append(t)
    return np.array([(t, s) for t, v in enumerate(m.tri) for s in sorted(set(fans[v[0]] + fans[v[1]] + fans[v[2]]))],
                    dtype=np.int32)


@pytest.fixture(scope="module")
def mesh():
    m = inputs.icosphere(8, 3.0)                  # 1280 triangles
    return m, _pairs(m)


@pytest.mark.parametrize("kappa", [0.125, 2.0])
@pytest.mark.parametrize("order", [1, 2, 3, 4, 6, 8])
@pytest.mark.parametrize("count", [1, 3, 70, 5000, None])
def test_blocks(mesh, order, kappa, count):
    m, pairs = mesh
    pairs = pairs[:count]
    with pbm.MeshHandle(m.xyz, m.tri, pbm.pb_default_options(kappa=kappa, singular_order=order)) as h:
        got = pbm.pb_mesh_near_blocks(h, pairs[:, 0], pairs[:, 1])
    pick = np.unique(np.concatenate([np.arange(min(4, len(pairs))), np.arange(len(pairs))[-4:],
                                     np.random.default_rng(order).integers(0, len(pairs), 8)]))
    for k in pick:
        t, s = (int(v) for v in pairs[k])
        VL, KL, _ = oracle.pair_block(m, t, s, 0.0, order)
        VY, KY, _ = oracle.pair_block(m, t, s, kappa, order)
        ref = np.stack([VL, KL, VY, KY])
        assert np.abs(got[k] - ref).max() < 1e-13 * np.abs(ref[0]).max(), (t, s)
