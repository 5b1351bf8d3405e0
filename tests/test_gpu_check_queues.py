"""The exact check's work items on short and long queues: a link's clusters split over waves while the queue is short, the
36-DoF trees' links, the crowded arm that takes lane groups by itself. Verdicts are those of the lane groups, and of the
oracle outside the 1e-5 m band of FP32 positions."""
import numpy as np
import pytest

import oracle
from paper_2604_13323_amd import scenes as S

from parity import from_dev, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def tree_scene(family, n_obs):
    """Shelf spheres in reach of the hands."""
    make = S.humanoid36_scene if family == "humanoid36" else S.digit36_scene
    sc = make(3, slab_x=(0.42, 0.5), slab_h=(1.0, 1.2))
    obs = np.concatenate([sc.obstacles + [0.0, 0.0, dz, 0.0] for dz in (0.0, 0.3, 0.6)])
    sc.obstacles = np.ascontiguousarray(obs[np.random.default_rng(n_obs).permutation(len(obs))[:n_obs]])
    return sc


def check_all(sc, q, need_both):
    import paper_2604_13323_amd as M
    G = M.Problem(sc.to_blob())
    qd = to_dev(q, torch.float32)
    v = G.check(qd)
    for lanes in (1, 4, 64):
        G.set_check_lanes(lanes)
        assert torch.equal(G.check(qd), v), lanes
    vo, sd = oracle.Problem(sc.to_blob()).check(from_dev(qd).T)
    out = np.abs(sd) > 1e-5
    assert (from_dev(v).astype(int)[out] == vo[out]).all()
    if need_both:
        assert 0 < vo.sum() < len(vo)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 700])
@pytest.mark.parametrize("n_obs", [1, 16, 17, 130, 1100])
@pytest.mark.parametrize("family", ["humanoid36", "digit36"])
def test_trees(family, n_obs, n):
    sc = tree_scene(family, n_obs)
    q = sc.qref + 0.15 * np.random.default_rng(n_obs * 1000 + n).standard_normal((n, sc.d))
    check_all(sc, q, n == 700 and n_obs > 100)


@pytest.mark.parametrize("n", [9, 600, 2100, 4200, 20000])
@pytest.mark.parametrize("n_obs,scale", [(200, 0.4), (1100, 0.25), (1100, 1.0)])
def test_arm_queue_lengths(n_obs, scale, n):
    """Every split of an arm's items (64 clusters' waves down to one), and the crowded arm (scale 1)."""
    sc = S.arm7_axis_scene(1, n_obs)
    sc.obstacles[:, 3] *= scale
    check_all(sc, np.random.default_rng(n).uniform(-2, 2, (n, sc.d)), scale < 1 and n > 9)
