"""Single steps of the tree families' leaf-to-root walks far from the manifold, against the FP64 oracle: pose errors
whose rotation needs the angle itself (beyond the series of asin(s)/s at sin^2 < 0.01), joint angles several turns
away (the sine table's reduction), and the damped step, whose lambda is transformed with the row basis."""
import numpy as np
import pytest

import oracle
from paper_2604_13323_amd import scenes as S

from parity import from_dev, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SCENES = dict(humanoid=lambda: S.humanoid36_scene(3), digit=lambda: S.digit36_scene(5), dual=lambda: S.dual14_rel_scene(2))


@pytest.mark.parametrize("lam", [0.0, 1e-2])
@pytest.mark.parametrize("name,spread,turns", [
    (name, spread, turns) for name in sorted(SCENES) for spread, turns in [(0.02, 0), (0.4, 0), (0.4, 40)]])
def test_one_fp64_step_matches_oracle(name, spread, turns, lam):
    """Tolerance: both sides solve the same system in FP64; the forward error is kappa_2(G) 2^-53 times a small constant
    and the step, so 1e-9 (1 + |step|) where kappa_2 < 1e5, plus the 2^-53 |q| of angles turned by up to 40 turns times
    the step's own sensitivity, |step| kappa_2^(1/2) (below 1e-9 too)."""
    import paper_2604_13323_amd as M
    sc = SCENES[name]()
    P = oracle.Problem(sc.to_blob())
    rng = np.random.default_rng(11)
    rev = np.array([j.jtype == S.JOINT_REV for j in sc.joints])
    q = sc.qref + rng.standard_normal((130, sc.d)) * np.where(rev, spread, 0.1 * spread)
    q[:, rev] += 2 * np.pi * rng.integers(-turns, turns + 1, (130, rev.sum()))
    G = M.Problem(sc.to_blob())
    r = G.project(to_dev(q, torch.float64), tol=1e-13, max_iter=1, lam=lam, check=False)
    torch.cuda.synchronize()
    qo, st, it, _ = P.project(q, tol=1e-13, max_iter=1, lam=lam)
    sv = np.linalg.svd(P.jacobian(q), compute_uv=False)  # (the Digit set's dropped rows are zero rows)
    k2 = (sv[:, 0] / np.where(sv > 1e-10 * sv[:, :1], sv, np.inf).min(axis=1)) ** 2
    step = np.linalg.norm(qo - q, axis=1)
    keep = (k2 < 1e5) & (step < 10.0) & (it == 1)
    assert keep.sum() > 60, (keep.sum(), np.median(k2))
    assert (from_dev(r.iters)[keep] == 1).all()
    err = np.abs(from_dev(r.q).T - qo).max(axis=1)
    assert (err[keep] < 1e-9 * (1.0 + step[keep])).all(), err[keep].max()
