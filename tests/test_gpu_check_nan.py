"""The exact check where coordinates are NaN: the box tests let every box pass, so the walk over groups and clusters of
obstacles must end with the last one that exists (an incomplete read of four groups, of eight clusters, one or both words
of the cluster mask), and the finite configurations of the same wave keep their verdicts."""
import numpy as np
import pytest

import oracle
from paper_2604_13323_amd import scenes as S

from parity import from_dev, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def scene(family, n_obs):
    if family == "arm7_axis":
        return S.arm7_axis_scene(1, n_obs)
    sc = S.humanoid36_scene(3, slab_x=(0.42, 0.5), slab_h=(1.0, 1.2))
    obs = np.concatenate([sc.obstacles + [0.0, 0.0, dz, 0.0] for dz in (0.0, 0.3, 0.6)])  # shelves in reach of the hands
    sc.obstacles = np.ascontiguousarray(obs[np.random.default_rng(n_obs).permutation(len(obs))[:n_obs]])
    return sc


@pytest.mark.parametrize("n_obs", [1, 16, 17, 130, 200, 1100])
@pytest.mark.parametrize("family", ["arm7_axis", "humanoid36"])
def test_nan_configurations_among_finite_ones(family, n_obs):
    """A comparison with NaN is false, so such a configuration is free in every form of the check; the others' verdicts
    equal those of a batch without it, and the oracle's outside the 1e-5 m band of FP32 positions."""
    import paper_2604_13323_amd as M
    sc = scene(family, n_obs)
    rng = np.random.default_rng(n_obs)
    q = rng.uniform(-2, 2, (131, sc.d)) if family == "arm7_axis" else sc.qref + 0.15 * rng.standard_normal((131, sc.d))
    bad = np.zeros(len(q), bool)
    bad[[0, 3, 40, 63, 90, 130]] = True
    G = M.Problem(sc.to_blob())
    for dtype in (torch.float32, torch.float64):
        want = G.check(to_dev(q, dtype))
        qn = q.copy()
        qn[bad] = np.nan
        qn[40] = q[40]
        qn[40, sc.d // 3] = np.nan  # one coordinate: the links behind it
        qd = to_dev(qn, dtype)
        got = {}
        for lanes in (0, 1, 4, 64):
            G.set_check_lanes(lanes)
            got[lanes] = from_dev(G.check(qd)).astype(int)
        G.set_check_lanes(0)
        keep = ~bad
        assert (got[0][keep] == from_dev(want).astype(int)[keep]).all()
        vo, sd = oracle.Problem(sc.to_blob()).check(from_dev(to_dev(q, dtype)).T)
        out = keep & (np.abs(sd) > 1e-5)
        assert (got[0][out] == vo[out]).all()
        whole = [0, 3, 63, 90, 130]
        assert (got[0][whole] == 0).all()
        for lanes in (1, 4, 64):
            assert (got[lanes] == got[0]).all(), lanes
