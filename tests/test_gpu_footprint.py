"""What a handle holds on the device, and what it falls back to where a memory
budget has no room for a faster path's workspace."""
import numpy as np
import pytest

import inputs

pytestmark = pytest.mark.gpu

pbm = pytest.importorskip("paper_2108_10481_amd")


@pytest.mark.parametrize("npts", [range(1, 65), (1, 5000, 5001, 5003, 9000, 3, 20000, 100000, 100000)])
@pytest.mark.parametrize("budget", [False, True])
def test_potentials_of_growing_point_sets(npts, budget):
    """Evaluating one point set after another, each a little larger, does not
    accumulate workspaces: beside the points themselves (7 doubles each, kept for the
    largest set, one buffer per growth) at most one buffer of 2^18 sums and one
    value per point."""
    m = inputs.icosphere(16, 5.0)                 # 5120 triangles
    tr = np.random.default_rng(3).standard_normal(2 * m.n_vertices)
    opt = pbm.pb_default_options()
    if budget:
        opt.memory_budget = pbm.pb_estimate_device_bytes(m.xyz, m.tri, opt)
    pts = inputs.charges_ball(5, max(npts), 4.0).xyz
    with pbm.MeshHandle(m.xyz, m.tri, opt) as h:
        before = h.info()["device_bytes"]
        first = None
        for n in npts:
            v = pbm.pb_mesh_reaction_potential(h, tr[:m.n_vertices], tr[m.n_vertices:], pts[:n])
            first = v[0] if first is None else first
            assert abs(v[0] - first) <= 1e-12 * abs(first)
        grown, top = [], 0
        for n in npts:
            if n > top:
                grown.append(max(56 * n, 256))
                top = n
        held = h.info()["device_bytes"] - before
    assert held <= sum(grown) + 8 * (2 ** 18 + max(npts))
