"""The condition estimate in the rows of the projection kernels: against the oracle's Jacobian turned into those rows, and
as what decides which configurations of an FP32 step continue in FP64."""
import numpy as np
import pytest

import oracle
from paper_2604_13323_amd import scenes as S

from parity import from_dev, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SCENES = dict(humanoid=lambda: S.humanoid36_scene(3), digit=lambda: S.digit36_scene(5), dual=lambda: S.dual14_rel_scene(2),
              axis=lambda: S.arm7_axis_scene(1))


def inputs(name, n=600):
    sc = SCENES[name]()
    rng = np.random.default_rng(5)
    q0 = sc.qref if sc.qref is not None else rng.uniform(-2, 2, (n, sc.d))
    return sc, q0 + 0.4 * rng.standard_normal((n, sc.d))


def step_kappa(sc, P, q, lam):
    """(max L_ii / min L_ii)^2 and kappa_2 of T^-1 (J J^T + lam I) T^-T, T^-1 = [E^T, J_r(w)] per pose block (E = exp(w), w the rotation
    error), the identity elsewhere; dropped rows left out, the two rows of a polygon's edge region (one direction) as one."""
    F, J = P.residual(q), P.jacobian(q)
    out, k2 = np.zeros(len(q)), np.zeros(len(q))
    for i in range(len(q)):
        Ti = np.eye(F.shape[1])
        r = 0
        for b in sc.blocks:
            if b.btype in (S.BLK_POSE, S.BLK_REL):
                w = F[i, r + 3:r + 6]
                t = np.linalg.norm(w)
                W = np.array([[0, -w[2], w[1]], [w[2], 0, -w[0]], [-w[1], w[0], 0]])
                Ti[r:r + 3, r:r + 3] = (np.eye(3) + np.sin(t) / t * W + (1 - np.cos(t)) / t ** 2 * W @ W).T
                Ti[r + 3:r + 6, r + 3:r + 6] = np.eye(3) - (1 - np.cos(t)) / t ** 2 * W + (t - np.sin(t)) / t ** 3 * W @ W
                r += 6
            else:
                if b.btype == S.BLK_HULL:
                    u, sv, _ = np.linalg.svd(J[i, r:r + 2], full_matrices=False)
                    if sv[0] > 0 and sv[1] < 1e-10 * sv[0]:
                        J[i, r:r + 2] = u.T @ J[i, r:r + 2]
                        J[i, r + 1] = 0.0
                r += 2 if b.btype in (S.BLK_COM, S.BLK_HULL, S.BLK_AXIS) else 1
        assert r == F.shape[1]
        A = J[i] if sc.name == "arm7_axis" else Ti @ J[i]
        L = lam * np.eye(r) if sc.name == "arm7_axis" else lam * Ti @ Ti.T
        keep = np.abs(J[i]).max(axis=1) > 0
        B = (A @ A.T + L)[np.ix_(keep, keep)]
        d = np.diag(np.linalg.cholesky(B))
        out[i], k2[i] = (d.max() / d.min()) ** 2, np.linalg.cond(B)
    return out, k2


@pytest.mark.parametrize("lam", [0.0, 1e-2])
@pytest.mark.parametrize("name", sorted(SCENES))
def test_fp64_estimate_matches_oracle_rows(name, lam):
    """Both factorise in FP64 by different operation orders: a pivot, at least the smallest eigenvalue, moves by a few 2^-53
    of the largest, so the estimate's relative error is bounded by 1e-15 kappa_2 of the matrix (and 1e-9)."""
    import paper_2604_13323_amd as M
    sc, q = inputs(name)
    k = from_dev(M.Problem(sc.to_blob()).condition(to_dev(q, torch.float64), lam=lam, step_rows=True))
    ke, k2 = step_kappa(sc, oracle.Problem(sc.to_blob()), q, lam)
    assert (np.abs(k / ke - 1.0) <= 1e-9 + 1e-15 * k2).all(), np.abs(k / ke - 1.0).max()


@pytest.mark.parametrize("name", sorted(SCENES))
def test_fp32_estimate_decides(name):
    """One FP32 step queues for FP64 exactly the configurations whose estimate exceeds the threshold, at thresholds in the
    middle of the widest relative gaps between estimates (wider than the 1e-5 by which another contraction of the same
    FP32 operations moves a small estimate)."""
    import paper_2604_13323_amd as M
    sc, q = inputs(name)
    G = M.Problem(sc.to_blob())
    qd = to_dev(q, torch.float32)
    k = np.sort(from_dev(G.condition(qd, step_rows=True)).astype(float))
    k = k[np.isfinite(k)]
    bad = 600 - len(k)
    lo = len(k) // 10
    mid = np.argsort(-(k[lo + 1:-lo] / k[lo:-lo - 1]))[:8] + lo
    for i in mid:
        thr = float(np.sqrt(k[i] * k[i + 1]))
        assert k[i + 1] / k[i] > 1 + 1e-4
        G.project(qd, tol=1e-13, max_iter=1, cond=thr, check=False)
        torch.cuda.synchronize()
        assert G.queue_counts()[1] == (k > thr).sum() + bad, (thr, bad)
