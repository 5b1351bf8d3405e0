"""The queue counters over calls of different kinds, eager and captured, in turn on one problem: every call gives what it
gives on a problem of its own, with the same queue counts."""
import numpy as np
import pytest

import paper_2604_13323_amd as M
from paper_2604_13323_amd import scenes as S

from parity import from_dev, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FIELDS = ("q", "status", "iters", "resid", "verdict")


def make():
    return M.Problem(S.arm7_axis_scene(1, 60).to_blob())


def step(G, kind, q):
    """One call; its outputs and the queue counts it leaves for its own queues."""
    if kind == "project":
        r = G.project(q, tol=1e-6, max_iter=30)
        out = [getattr(r, f) for f in FIELDS]
        own = (0, 1, 3)
    elif kind == "check":
        out, own = [G.check(q)], (3,)
    else:
        st = torch.zeros(q.shape[1], dtype=torch.int8, device="cuda")
        out, own = [G.vjp(q, st, torch.ones_like(q), cond=50.0)], (2,)
    torch.cuda.synchronize()
    counts = G.queue_counts()
    return out, [counts[k] for k in own]


@pytest.mark.parametrize("order", [("project", "project", "check", "vjp"), ("vjp", "vjp", "project", "check", "check", "vjp")])
def test_interleaved_calls_match_fresh_problems(order):
    rng = np.random.default_rng(2)
    G = make()
    qg = to_dev(rng.uniform(-2, 2, (500, 7)), torch.float32)
    outs = M.ProjectResult(**{f: torch.empty_like(getattr(G.project(qg, tol=1e-6, max_iter=30), f)) for f in FIELDS}, geo_ok=None)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        G.project(qg, tol=1e-6, max_iter=30, out=outs)
    want, _ = step(make(), "project", qg)
    for turn, n in enumerate((1, 64, 65, 500, 7)):
        q = to_dev(rng.uniform(-2, 2, (n, 7)), torch.float32)
        for kind in order:
            got, counts = step(G, kind, q)
            ref, rcounts = step(make(), kind, q)
            assert all(torch.equal(a, b) for a, b in zip(got, ref)), (turn, kind)
            assert counts == rcounts, (turn, kind)
            g.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(getattr(outs, f), w) for f, w in zip(FIELDS, want)), (turn, kind)
