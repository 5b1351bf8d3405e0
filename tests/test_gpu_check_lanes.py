"""The lane-per-configuration exact check at the edges of its work items (64 configurations) and of its obstacle levels
(clusters of at most 16 obstacles, groups of 8 clusters, 64 clusters to a mask word)."""
import numpy as np
import pytest

import oracle
from paper_2604_13323_amd import scenes as S

from parity import from_dev, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1, 63, 64, 65, 700])
@pytest.mark.parametrize("n_obs", [1, 16, 17, 130, 1100])
@pytest.mark.parametrize("family", ["arm7_axis", "dual14_rel"])
def test_verdicts_match_lane_groups_and_oracle(family, n_obs, n):
    """Same verdicts as the lane groups', and as the oracle's outside the 1e-5 m band of FP32 positions."""
    import paper_2604_13323_amd as M
    sc = S.arm7_axis_scene(1, n_obs) if family == "arm7_axis" else S.dual14_rel_scene(2, n_obs)
    if n_obs > 200:
        sc.obstacles[:, 3] *= 0.25  # so that about half the configurations are in collision
    elif n_obs < 20:
        sc.obstacles[:, :3] *= 0.4
    q = np.random.default_rng(n_obs * 1000 + n).uniform(-2, 2, (n, sc.d))
    G = M.Problem(sc.to_blob())
    for dtype in (torch.float32, torch.float64):
        qd = to_dev(q, dtype)
        v = G.check(qd)
        for lanes in (4, 64):
            G.set_check_lanes(lanes)
            assert torch.equal(G.check(qd), v), lanes
        G.set_check_lanes(0)
        vo, sd = oracle.Problem(sc.to_blob()).check(from_dev(qd).T)
        out = np.abs(sd) > 1e-5
        assert (from_dev(v).astype(int)[out] == vo[out]).all()
