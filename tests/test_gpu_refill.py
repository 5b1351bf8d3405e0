"""Batches of more configurations than the persistent launch has lanes: those that a lane takes from the queue after its
first one are compared with the oracle, whatever the launch shape."""
from types import SimpleNamespace

import numpy as np
import pytest

import paper_2604_13323_amd as M

from parity import compare, config_inputs, from_dev, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("max_geo,waves", [(None, 0), (1000, 2), (500, 1)])
def test_refilled_configurations_match_oracle(max_geo, waves):
    """The benchmark's differentiation batch (74,059 humanoid configurations) in the library's own launch (one wave per SIMD,
    65,536 lanes) and its first 36,000 and 17,000 in launches of one workgroup per CU. Bounds of the parity tests (1e-4 in FP32
    mode), band at most a quarter."""
    sc, P, q, offs, tol, mi = config_inputs("c4", small=False, max_geo=max_geo)
    lanes = torch.cuda.get_device_properties(0).multi_processor_count * 64 * (waves or 4)
    G = M.Problem(sc.to_blob())
    qd = to_dev(q, torch.float32)
    r = G.project(qd, tol=tol, max_iter=mi, variant="fused", check=False, waves_per_block=waves, blocks_per_cu=1 if waves else 0)
    torch.cuda.synchronize()
    assert len(q) - lanes >= 500
    assert G.queue_counts()[0] >= len(q) - lanes  # (a lane also draws once more to find the queue empty)
    idx = np.sort(np.random.default_rng(1).choice(np.arange(lanes, len(q)), 400, replace=False))
    t = torch.from_numpy(idx).cuda()
    sub = SimpleNamespace(q=r.q[:, t], status=r.status[t], iters=r.iters[t], resid=r.resid[t])
    assert compare(P, from_dev(qd).T[idx], sub, tol, mi, 1e-4)["n"] == 400
