"""Performance cases of the batched manifold projection: the calls a planner or a trajectory
optimiser makes, from one extension of a tree to the largest batches of the benchmark.

A case names an operation, a scene and a size:

  project      Problem.project with the fused collision check over geodesics (CSR offsets, per-geodesic flags)
  particles    the same call on a handful of particles around one steer point
  extend       Problem.extend, the batched ConstrainedExtend step
  check        Problem.check, collision verdicts of arbitrary configurations
  train        interpolation, differentiable projection, path length and its gradient (tangent-projector VJP)
  train_exact  the same with the exact derivative of the projection map

Scenes are the package's own (scenes.py), with a fixed robot and obstacles each; a seed gives the
configurations. Geodesic endpoints lie on the constraint manifold, as the nodes of a planner's tree
do: raw samples around the reference configuration, projected here by the plain FP64 Newton
iteration below (`Reference`), which also gives the values of `exact`. No library code prepares an
input.

Outputs are the projected configurations, statuses, collision verdicts, per-geodesic flags, losses
and gradients. Two diagnostics of the solver are returned in FP64 mode only or not at all: the step
counts (in FP32 mode a count changes when the rounding of one step moves a residual across the
tolerance, in a few of 10^5 configurations) and the final residual norm, which below the tolerance
is the rounding left by the last step.
"""
import functools
import math

import numpy as np
import torch

import paper_2604_13323_amd as M
from paper_2604_13323_amd import flops as FL
from paper_2604_13323_amd import scenes as S

TOL = 1e-6
# Scene recipe, spread of the raw geodesic endpoints, and steps allowed, as in the benchmark's configurations. The single
# arms run with the paper's step limit (MaxDistance): without it a path near a singularity wanders over many turns, and
# where it ends says nothing.
ROBOTS = {
    "humanoid": dict(make=lambda: S.humanoid36_scene(3), sigma=S.humanoid_noise_sigma, max_iter=40, max_step=0.0),
    "humanoid_near": dict(make=lambda: S.humanoid36_scene(3, slab_x=(0.42, 0.5), slab_h=(1.0, 1.2)),
                          sigma=S.humanoid_noise_sigma, max_iter=40, max_step=0.0),
    "digit": dict(make=lambda: S.digit36_scene(5), sigma=S.humanoid_noise_sigma, max_iter=40, max_step=0.0),
    "dual": dict(make=lambda: S.dual14_rel_scene(2), sigma=lambda: 0.1, max_iter=30, max_step=0.0),
    "tsr": dict(make=lambda: S.arm7_tsr_scene(6), sigma=lambda: 0.2, max_iter=30, max_step=0.5),
    "axis": dict(make=lambda: S.arm7_axis_scene(1), sigma=None, max_iter=30, max_step=0.5),
}


def listed():
    return [
        # one step of a sampling-based planner: extend the tree by one edge (8 particles, then 8 and
        # 9 interpolated points); the latency of a handful of launches
        dict(name="extend_one", op="extend", robot="humanoid", dtype="f32", n=1),
        # the smallest projection call: the particles of one extension
        dict(name="particles_8", op="particles", robot="humanoid", dtype="f32", n=8),
        # the benchmark's humanoid batch: 2,048 geodesics of 32 interior points
        dict(name="humanoid_65536", op="project", robot="humanoid", dtype="f32", n_geo=2048, lo=32, hi=32),
        # an ordinary batch in FP64 mode, ragged and odd in size
        dict(name="humanoid_f64", op="project", robot="humanoid", dtype="f64", n_geo=251, lo=8, hi=64),
        # the Digit constraint set (support polygon, closed linkages), its benchmark size
        dict(name="digit_65536", op="project", robot="digit", dtype="f32", n_geo=2048, lo=32, hi=32),
        # the dual arm: many geodesics of very uneven length
        dict(name="dual_ragged", op="project", robot="dual", dtype="f32", n_geo=4000, lo=4, hi=128),
        # the arm with a bounded task-space region, its benchmark size
        dict(name="tsr_131072", op="project", robot="tsr", dtype="f32", n_geo=4096, lo=32, hi=32),
        # the arm with an axis constraint and the paper's step limit, an ordinary ragged batch
        dict(name="axis_ragged", op="project", robot="axis", dtype="f32", n_geo=1021, lo=4, hi=64),
        # re-validation of stored configurations against a scene within reach of the hands
        dict(name="check_near", op="check", robot="humanoid_near", dtype="f32", n_geo=2048, lo=32, hi=32),
        # trajectory optimisation, forward and backward: as many configurations as the benchmark's
        # differentiation batch, on trajectories of 4 to 24 waypoints (closer waypoints would leave
        # FP32 differences of neighbours with few significant digits)
        dict(name="train_ragged", op="train", robot="humanoid", dtype="f32", n_geo=5290, lo=4, hi=24),
        # the same with the exact derivative at off-manifold inputs, an ordinary batch
        dict(name="train_exact", op="train_exact", robot="humanoid", dtype="f32", n_geo=1321, lo=4, hi=24),
        # a planner that grows many trees at once, in FP64 mode
        dict(name="extend_many_f64", op="extend", robot="humanoid", dtype="f64", n=509),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["project", "project", "project", "project", "particles", "extend", "check", "train", "train_exact"])
    if op == "particles":
        return dict(op=op, robot=rng.choice(["humanoid", "digit", "dual", "tsr"]), dtype=rng.choice(["f32", "f64"]),
                    n=rng.randint(1, 63))
    if op == "extend":
        # (FP32 batches stay small: which particle converges first may turn on one step's rounding)
        if rng.random() < 0.4:
            return dict(op=op, robot="humanoid", dtype="f32", n=rng.randint(1, 4))
        return dict(op=op, robot="humanoid", dtype="f64", n=log_int(4, 509))
    lo = rng.randint(2, 24)
    hi = lo + rng.randint(0, 96)
    mean = 0.5 * (lo + hi)
    if op == "check":
        return dict(op=op, robot=rng.choice(["humanoid_near", "humanoid", "digit", "dual"]), dtype="f32",
                    n_geo=max(1, int(log_int(64, 65536) / mean)), lo=lo, hi=hi)
    if op in ("train", "train_exact"):
        lo = rng.randint(2, 8)
        hi = lo + rng.randint(0, 16)
        mean = 0.5 * (lo + hi)
        top = 70000 if op == "train" else 18000
        return dict(op=op, robot="humanoid", dtype="f32", n_geo=max(2, int(log_int(256, top) / mean)), lo=lo, hi=hi)
    robot = rng.choice(["humanoid", "humanoid", "digit", "dual", "tsr", "axis"])
    dtype = rng.choice(["f32", "f32", "f64"])
    top = dict(humanoid=60000, digit=60000, dual=250000, tsr=120000, axis=60000)[robot] // (8 if dtype == "f64" else 1)
    return dict(op=op, robot=robot, dtype=dtype, n_geo=max(1, int(log_int(64, top) / mean)), lo=lo, hi=hi)


# ------------------------------------------------------------------ plain FP64 reference
class Reference:
    """A scene's residual, Jacobian and Newton iteration in plain torch, FP64 (batch first: q [n, d])."""

    def __init__(self, sc, device):
        self.sc, self.dev = sc, device
        t = functools.partial(torch.as_tensor, dtype=torch.float64, device=device)
        self.O = [(None if np.allclose(j.R, np.eye(3)) else t(np.asarray(j.R)), t(np.asarray(j.p))) for j in sc.joints]
        self.F = [(None if np.allclose(f.R, np.eye(3)) else t(np.asarray(f.R)), t(np.asarray(f.p))) for f in sc.frames]
        d = sc.d
        anc = np.zeros((d, d))  # anc[j, l]: joint j moves link l
        for link in range(d):
            k = link
            while k >= 0:
                anc[k, link] = 1.0
                k = sc.joints[k].parent
        self.anc = t(anc)
        self.rev = t([1.0 if j.jtype == S.JOINT_REV else 0.0 for j in sc.joints])
        self.mass, self.com = t(np.asarray(sc.masses)), t(np.asarray(sc.coms))
        self.ref = []
        fr = self._frames(t(np.asarray(sc.qref))[None])[2] if sc.qref is not None else None
        for b in sc.blocks:
            R, p, length = t(np.asarray(b.R)), t(np.asarray(b.p)), float(b.target[0])
            if b.ref_from_qref and b.btype == S.BLK_POSE:
                R, p = fr[b.fa][0][0], fr[b.fa][1][0]
            elif b.ref_from_qref and b.btype == S.BLK_REL:
                Ra = fr[b.fa][0][0]
                R, p = Ra.T @ fr[b.fb][0][0], Ra.T @ (fr[b.fb][1][0] - fr[b.fa][1][0])
            elif b.ref_from_qref and b.btype == S.BLK_DIST:
                length = float((fr[b.fb][1] - fr[b.fa][1]).norm())
            self.ref.append((R, p, length))

    def _frames(self, q):
        """World rotations and origins of every joint's frame, and of the end-effector frames."""
        n = q.shape[0]
        L = []
        for j, J in enumerate(self.sc.joints):
            O, p = self.O[j]
            if J.parent < 0:
                R = torch.eye(3, dtype=torch.float64, device=self.dev).expand(n, 3, 3)
                x = p.expand(n, 3)
            else:
                R, x = L[J.parent]
                x = x + R @ p
            if O is not None:
                R = R @ O
            if J.jtype == S.JOINT_PRI:
                x = x + R[:, :, J.axis] * q[:, j, None]
            else:
                c, s = torch.cos(q[:, j, None]), torch.sin(q[:, j, None])
                i, k = (J.axis + 1) % 3, (J.axis + 2) % 3
                cols = [None, None, None]
                cols[J.axis] = R[:, :, J.axis]
                cols[i] = R[:, :, i] * c + R[:, :, k] * s
                cols[k] = R[:, :, k] * c - R[:, :, i] * s
                R = torch.stack(cols, -1)
            L.append((R, x))
        ends = []
        for f, (O, p) in zip(self.sc.frames, self.F):
            R, x = L[f.link]
            ends.append((R if O is None else R @ O, x + R @ p))
        z = torch.stack([L[j][0][:, :, J.axis] for j, J in enumerate(self.sc.joints)], 1)
        o = torch.stack([x for _, x in L], 1)
        return L, (z, o), ends

    @staticmethod
    def _mv(A, v):
        """A [n, 3, 3] applied to v [n, d, 3] (or [n, 3])."""
        return (A[:, None] * v[:, :, None, :]).sum(-1) if v.dim() == 3 else (A * v[:, None, :]).sum(-1)

    @staticmethod
    def _mm(A, B):
        return (A[:, :, :, None] * B[:, None]).sum(2)

    @staticmethod
    def _log(R):
        """Rotation vector w of R and the inverse left Jacobian at w."""
        v = 0.5 * torch.stack([R[:, 2, 1] - R[:, 1, 2], R[:, 0, 2] - R[:, 2, 0], R[:, 1, 0] - R[:, 0, 1]], -1)
        c = 0.5 * (R[:, 0, 0] + R[:, 1, 1] + R[:, 2, 2] - 1.0)
        s2 = (v * v).sum(-1)
        small = (c > 0) & (s2 < 1e-8)
        sn = torch.sqrt(torch.where(small, torch.ones_like(s2), s2))
        th = torch.atan2(sn, c)
        w = torch.where(small, 1.0 + s2 / 6.0, th / sn)[:, None] * v
        t2 = (w * w).sum(-1)
        near = t2 < 1e-2
        ts = torch.where(near, torch.ones_like(t2), t2)
        h = 0.5 * torch.sqrt(ts)
        beta = torch.where(near, 1 / 12 + t2 / 720 + t2 ** 2 / 30240 + t2 ** 3 / 1209600 + t2 ** 4 / 47900160,
                           (1.0 - h * torch.cos(h) / torch.sin(h)) / ts)
        o = torch.zeros_like(t2)
        W = torch.stack([o, -w[:, 2], w[:, 1], w[:, 2], o, -w[:, 0], -w[:, 1], w[:, 0], o], -1).reshape(-1, 3, 3)
        I = torch.eye(3, dtype=R.dtype, device=R.device)
        return w, I - 0.5 * W + beta[:, None, None] * Reference._mm(W, W)

    def rows(self, q):
        """(F [n, m], J [n, m, d], dropped [n, m]): rows that vanish on a region are dropped there."""
        sc = self.sc
        L, (z, o), ends = self._frames(q)
        rev = self.rev[None, :, None]
        Fs, Js, drop = [], [], []

        def moved(x):  # velocity of a point x [n, 3] under each joint
            return torch.where(rev > 0, torch.linalg.cross(z, x[:, None] - o, dim=-1), z)

        com = None
        for b, (R, p, length) in zip(sc.blocks, self.ref):
            if b.btype in (S.BLK_POSE, S.BLK_REL):
                if b.btype == S.BLK_POSE:
                    Rf, x = ends[b.fa]
                    W = R.T.expand(q.shape[0], 3, 3)
                    t = self._mv(W, x - p)
                    sign = self.anc[:, sc.frames[b.fa].link]
                else:
                    (Ra, xa), (Rf, x) = ends[b.fa], ends[b.fb]
                    W = self._mm(R.T.expand_as(Ra), Ra.transpose(1, 2))
                    t = self._mv(W, x - xa) - R.T @ p
                    sign = self.anc[:, sc.frames[b.fb].link] - self.anc[:, sc.frames[b.fa].link]
                w, Jl = self._log(self._mm(W, Rf))
                lin = self._mv(W, moved(x))
                ang = self._mv(self._mm(Jl, W), z * rev)
                F = torch.cat([t, w], -1)
                J = (torch.cat([lin, ang], -1) * sign[None, :, None]).transpose(1, 2)
                D = torch.zeros_like(F, dtype=torch.bool)
                if b.aux & S.POSE_BOUNDED:
                    lo = torch.as_tensor(b.ext[:6], dtype=F.dtype, device=F.device)
                    hi = torch.as_tensor(b.ext[6:12], dtype=F.dtype, device=F.device)
                    D = (F >= lo) & (F <= hi)
                    F = torch.where(F > hi, F - hi, torch.where(F < lo, F - lo, torch.zeros_like(F)))
            elif b.btype == S.BLK_AXIS:
                u = ends[b.fa][0][:, :, 2]
                F = u[:, :2]
                sign = self.anc[:, sc.frames[b.fa].link] * self.rev
                J = (torch.linalg.cross(z, u[:, None].expand_as(z), dim=-1)[:, :, :2] * sign[None, :, None]).transpose(1, 2)
                D = torch.zeros_like(F, dtype=torch.bool)
            elif b.btype == S.BLK_DIST:
                xa, xb = ends[b.fa][1], ends[b.fb][1]
                dv = xb - xa
                r = dv.norm(dim=-1, keepdim=True)
                la, lb = self.anc[:, sc.frames[b.fa].link], self.anc[:, sc.frames[b.fb].link]
                only_b, only_a = (lb * (1 - la))[None, :, None], (la * (1 - lb))[None, :, None]
                J = ((moved(xb) * only_b - moved(xa) * only_a) * (dv / r)[:, None]).sum(-1)[:, None]
                F = r - length
                D = torch.zeros_like(F, dtype=torch.bool)
            else:  # centre of mass: at a point, or within a convex polygon
                if com is None:
                    Mt = self.mass.sum()
                    mc = torch.stack([self.mass[k] * (L[k][1] + L[k][0] @ self.com[k]) for k in range(sc.d)], 1)
                    com = mc.sum(1)[:, :2] / Mt
                    Mj = self.anc @ self.mass
                    sub = torch.einsum("jl,nlc->njc", self.anc, mc)
                    Jc = torch.where(rev > 0, torch.linalg.cross(z, sub - Mj[None, :, None] * o, dim=-1), Mj[None, :, None] * z)
                    Jc = (Jc[:, :, :2] / Mt).transpose(1, 2)
                if b.btype == S.BLK_COM:
                    F, J = com - torch.as_tensor(b.target[:2], dtype=com.dtype, device=com.device), Jc
                    D = torch.zeros_like(F, dtype=torch.bool)
                else:
                    F, J, D = self._polygon(com, Jc, b)
            Fs.append(F)
            Js.append(torch.where(D[:, :, None], torch.zeros_like(J), J))
            drop.append(D)
        return torch.cat(Fs, 1), torch.cat(Js, 1), torch.cat(drop, 1)

    @staticmethod
    def _polygon(x, Jc, b):
        V = torch.as_tensor(b.ext[:2 * b.aux].reshape(-1, 2), dtype=x.dtype, device=x.device)
        E = torch.roll(V, -1, 0) - V
        d = x[:, None] - V
        inside = (E[:, 0] * d[:, :, 1] - E[:, 1] * d[:, :, 0] >= 0).all(1)
        t = (d * E).sum(-1) / (E * E).sum(-1)
        c = V + t.clamp(0, 1)[:, :, None] * E
        k = ((x[:, None] - c) ** 2).sum(-1).argmin(1)
        at = torch.arange(len(x), device=x.device)
        edge = (t[at, k] > 0) & (t[at, k] < 1)
        nrm = torch.stack([E[:, 1], -E[:, 0]], -1) / E.norm(dim=-1, keepdim=True)
        nk, r = nrm[k], x - c[at, k]
        # an edge region has one row, along the edge's normal
        F = torch.where(edge[:, None], torch.stack([(nk * r).sum(-1), torch.zeros_like(r[:, 0])], -1), r)
        Je = torch.stack([(nk[:, :, None] * Jc).sum(1), torch.zeros_like(Jc[:, 0])], 1)
        J = torch.where(edge[:, None, None], Je, Jc)
        D = torch.stack([inside, inside | edge], -1)
        return torch.where(D, torch.zeros_like(F), F), J, D

    @staticmethod
    def solve(J, drop, b):
        """(J J^T)^-1 b over the rows kept (zero where dropped)."""
        G = torch.stack([(J * J[:, k, None]).sum(-1) for k in range(J.shape[1])], -1)
        G = G + torch.diag_embed(drop.to(G.dtype))
        G, y, m = G.clone(), b.clone(), G.shape[-1]
        for k in range(m - 1):
            f = G[:, k + 1:, k] / G[:, k, k, None]
            G[:, k + 1:, k + 1:] -= f[:, :, None] * G[:, k, None, k + 1:]
            y[:, k + 1:] -= f * y[:, k, None]
        for k in range(m - 1, -1, -1):
            y[:, k] = (y[:, k] - (G[:, k, k + 1:] * y[:, k + 1:]).sum(-1)) / G[:, k, k]
        return y

    def newton(self, q, tol, max_iter, max_step=0.0):
        """(q, status, steps) of the min-norm Newton iteration with per-configuration termination."""
        q = q.clone()
        n = len(q)
        st = torch.full((n,), -1, dtype=torch.int64, device=q.device)
        it = torch.zeros(n, dtype=torch.int64, device=q.device)
        for k in range(max_iter + 1):
            run = (st < 0).nonzero().flatten()
            if len(run) == 0:
                break
            F, J, D = self.rows(q[run])
            done = (F * F).sum(-1) < tol * tol
            st[run[done]] = M.CONVERGED
            if k == max_iter:
                st[run[~done]] = M.MAX_ITER
                break
            go = (~done).nonzero().flatten()
            if len(go) == 0:
                break
            y = self.solve(J[go], D[go], F[go])
            dq = (J[go] * y[:, :, None]).sum(1)
            far = (dq.norm(dim=-1) > max_step) if max_step > 0 else torch.zeros(len(go), dtype=torch.bool, device=q.device)
            st[run[go[far]]] = M.DIVERGED
            idx = run[go[~far]]
            q[idx] = q[idx] - dq[~far]
            it[idx] += 1
        return q, st, it

    def project_tangent(self, q, g):
        """(I - J^+ J) g at q."""
        _, J, D = self.rows(q)
        y = self.solve(J, D, (J * g[:, None]).sum(-1))
        return g - (J * y[:, :, None]).sum(1)


# ------------------------------------------------------------------ inputs
@functools.lru_cache(maxsize=None)
def _scene(robot):
    return ROBOTS[robot]["make"]()


@functools.lru_cache(maxsize=None)
def _blob(robot):
    return _scene(robot).to_blob()


@functools.lru_cache(maxsize=None)
def _reference(robot):
    return Reference(_scene(robot), torch.device("cuda"))


def _on_manifold(robot, n, raw):
    """n configurations on the manifold: of the raw samples (some more than n) the first n that converge, again from the
    first where they are too few."""
    q, st, _ = _reference(robot).newton(torch.as_tensor(raw, device="cuda"), 1e-9, 40, ROBOTS[robot]["max_step"])
    good = (st == M.CONVERGED).nonzero().flatten()
    return q[good[torch.arange(n, device="cuda") % len(good)]]


def _around_reference(robot, n, rng):
    """n configurations on the manifold around the scene's reference configuration."""
    sc = _scene(robot)
    raw = sc.qref + rng.standard_normal((n + 64, sc.d)) * np.broadcast_to(ROBOTS[robot]["sigma"](), (sc.d,))
    return _on_manifold(robot, n, raw)


def _endpoints(case, rng):
    """Geodesic endpoints [n_geo, 2, d] on the manifold."""
    robot, n_geo = case["robot"], case["n_geo"]
    sc = _scene(robot)
    if robot == "axis":  # anywhere in the joint range, and a short extension from there
        a = _on_manifold(robot, n_geo, rng.uniform(-math.pi, math.pi, (2 * n_geo + 64, sc.d)))
        step = rng.normal(0.0, 0.1, (n_geo, sc.d))
        b, st, _ = _reference(robot).newton(a + torch.as_tensor(step, device="cuda"), 1e-9, 40, 0.5)
        return torch.stack([a, torch.where((st == M.CONVERGED)[:, None], b, a)], 1)
    return _around_reference(robot, 2 * n_geo, rng).reshape(n_geo, 2, sc.d)


def _offsets(case):
    """CSR offsets of geodesics of lo..hi points; they depend on the case alone, so that another seed has the same sizes."""
    L = np.random.default_rng([case["n_geo"], case["lo"], case["hi"]]).integers(case["lo"], case["hi"] + 1, case["n_geo"])
    return np.concatenate([[0], np.cumsum(L)]).astype(np.int32)


def _interior(ends, offs):
    """Interior points of the chords between endpoints, [n, d]."""
    L = np.diff(offs)
    g = torch.as_tensor(np.repeat(np.arange(len(L)), L), device="cuda")
    t = np.concatenate([np.arange(1, k + 1) / (k + 1.0) for k in L])
    t = torch.as_tensor(t, device="cuda")[:, None]
    return ends[g, 0] + t * (ends[g, 1] - ends[g, 0])


def _dtype(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


def _inputs(case, seed):
    """The case's input tensors in FP64 values already rounded to its type, plus offsets."""
    rng = np.random.default_rng([int(seed), 17])
    robot, op, dt = case["robot"], case["op"], _dtype(case)
    sc = _scene(robot)
    if op == "particles":  # particles spread along one extension direction around a steer point
        a = _around_reference(robot, 2, rng)
        v = (a[1] - a[0]) / (a[1] - a[0]).norm()
        eps = torch.as_tensor(0.3 + rng.normal(0.0, 0.05, case["n"]), device="cuda")
        return dict(q=(a[0] + eps[:, None] * v).T.to(dt).contiguous())
    if op == "extend":
        prm = S.EXTEND_PARAMS["c3"]
        sig = np.broadcast_to(ROBOTS[robot]["sigma"](), (sc.d,))
        a = _around_reference(robot, case["n"], rng)
        b = torch.as_tensor(sc.qref + rng.standard_normal((case["n"], sc.d)) * sig, device="cuda")
        eps = torch.as_tensor(rng.normal(0.0, prm["sigma"], (case["n"], prm["n"])), device="cuda")
        return dict(a=a.T.to(dt).contiguous(), b=b.T.to(dt).contiguous(), eps=eps.to(dt).contiguous())
    offs = _offsets(case)
    ends = _endpoints(case, rng)
    if op in ("train", "train_exact"):
        e = ends.reshape(-1, sc.d).T.to(dt).contiguous()
        return dict(ends=e, offs_host=offs)
    q = _interior(ends, offs)
    if robot == "axis":  # that arm's chords nearly follow the manifold: joint noise on every point, as in its benchmark recipe
        q = q + torch.as_tensor(rng.normal(0.0, 0.1, tuple(q.shape)), device="cuda")
    if op == "check":  # stored configurations: converged ones
        q, _, _ = _reference(robot).newton(q, TOL, ROBOTS[robot]["max_iter"])
    return dict(q=q.T.to(dt).contiguous(), offs_host=offs)


def prepare(case, seed):
    x = _inputs(case, seed)
    x["case"] = case
    x["problem"] = M.Problem(_blob(case["robot"]))
    if "offs_host" in x:
        x["offs"] = torch.from_numpy(x["offs_host"]).cuda()
    return x


def run(x):
    case, P = x["case"], x["problem"]
    mi = ROBOTS[case["robot"]]["max_iter"]
    op = case["op"]
    if op == "extend":
        prm = S.EXTEND_PARAMS["c3"]
        r = P.extend(x["a"], x["b"], x["eps"], prm["r"], prm["delta"], tol=TOL, max_iter=mi)
        # q holds a column only where a particle was selected
        return dict(q=torch.where(r.particle >= 0, r.q, torch.zeros_like(r.q)), result=r.result, particle=r.particle,
                    n_points=r.n_points)
    if op == "check":
        return dict(verdict=P.check(x["q"]))
    if op in ("train", "train_exact"):
        total = int(x["offs_host"][-1])
        q_in = P.interpolate(x["ends"], x["offs"], total).requires_grad_()
        q, status = M.project(q_in, P, tol=TOL, max_iter=mi, check=False, exact=op == "train_exact")
        loss = M.PathLengthFn.apply(q, P, x["offs"])
        loss.backward()
        return dict(q=q.detach(), status=status, loss=loss.detach(), grad=q_in.grad)
    if op == "particles":
        r = P.project(x["q"], tol=TOL, max_iter=mi, max_step=ROBOTS[case["robot"]]["max_step"])
        out = dict(q=r.q, status=r.status, verdict=r.verdict)
    else:
        r = P.project(x["q"], tol=TOL, max_iter=mi, geo_offsets=x["offs"], geo_ok=True,
                      max_step=ROBOTS[case["robot"]]["max_step"])
        out = dict(q=r.q, status=r.status, verdict=r.verdict, geo_ok=r.geo_ok)
    if case["dtype"] == "f64":
        out["iters"] = r.iters
    return out


def _mean_points(case):
    return case["n_geo"] * 0.5 * (case["lo"] + case["hi"])


def work(case):
    sc = _scene(case["robot"])
    f = FL.iteration_flops(sc)
    size = 8 if case["dtype"] == "f64" else 4
    op = case["op"]
    step, last = f["per_iter"], f["final"]
    if op == "extend":  # 8 particles and 17 chain points each, two steps apiece on average
        n = case["n"] * 25
        return dict(bytes=case["n"] * (3 * sc.d * size + 8 * size + 9), flops=n * (2 * step + last))
    n = case["n"] if op == "particles" else _mean_points(case)
    if op == "check":
        fk = f["parts"]["fk"] + f["parts"]["broad_once"]
        return dict(bytes=n * (sc.d * size + 1), flops=n * fk)
    if op == "train":  # two forward steps, one Gram, factorisation and solve backward
        return dict(bytes=n * 3 * sc.d * size, flops=n * (3 * step + last))
    if op == "train_exact":  # every forward step replayed and pulled back once
        return dict(bytes=n * 3 * sc.d * size, flops=n * (2 * step + last + 2 * 3 * step))
    return dict(bytes=n * (2 * sc.d * size + 2), flops=n * (2 * step + last))


# ------------------------------------------------------------------ 64-bit values
def _path_gradient(q, offs):
    """Path length over geodesics and its gradient, q [n, d]."""
    d = q[1:] - q[:-1]
    cut = torch.as_tensor(offs[1:-1].astype(np.int64), device=q.device)
    keep = torch.ones(len(d), dtype=torch.bool, device=q.device)
    keep[cut[(cut > 0) & (cut < len(q))] - 1] = False
    r = d.norm(dim=-1)
    u = torch.where(keep[:, None], d / r.clamp_min(1e-12)[:, None], torch.zeros_like(d))
    g = torch.zeros_like(q)
    g[1:] += u
    g[:-1] -= u
    return (r * keep).sum(), g


def exact(case, seed):
    op = case["op"]
    if op in ("extend", "check"):
        return None
    x = _inputs(case, seed)
    R = _reference(case["robot"])
    mi = ROBOTS[case["robot"]]["max_iter"]
    max_step = ROBOTS[case["robot"]]["max_step"]
    if op in ("project", "particles"):
        q, st, _ = R.newton(x["q"].double().T.contiguous(), TOL, mi, max_step)
        out = dict(q=q.T, status=None, verdict=None)
        if op == "project":
            out["geo_ok"] = None
        if case["dtype"] == "f64":
            out["iters"] = None
        return out
    ends = x["ends"].double().T.reshape(-1, 2, x["ends"].shape[0])
    # the interpolated inputs are the type's: rounded as the call that makes them rounds
    q_in = _interior(ends, x["offs_host"]).to(_dtype(case)).double()
    q, st, it = R.newton(q_in, TOL, mi)
    loss, g = _path_gradient(q, x["offs_host"])
    g = R.project_tangent(q, g)
    if op == "train_exact":
        g = _pull_back(R, q_in, it, g)
    g = torch.where((st == M.CONVERGED)[:, None], g, torch.zeros_like(g))
    return dict(q=q.T, status=None, loss=loss, grad=g.T)


def _pull_back(R, q_in, steps, g):
    """The cotangent g of the last iterate taken back through every Newton step by automatic
    differentiation of the step itself, 2,048 configurations at a time."""
    out = []
    for k0 in range(0, len(q_in), 2048):
        s = slice(k0, k0 + 2048)
        with torch.enable_grad():
            q0 = q_in[s].detach().requires_grad_()
            q, left = q0, steps[s]
            for _ in range(int(left.max()) if len(left) else 0):
                F, J, D = R.rows(q)
                G = (J[:, :, None] * J[:, None]).sum(-1) + torch.diag_embed(D.to(J.dtype))
                y = torch.linalg.solve(G, F)
                q = torch.where((left > 0)[:, None], q - (J * y[:, :, None]).sum(1), q)
                left = left - 1
            out.append(torch.autograd.grad(q, q0, g[s])[0] if q is not q0 else g[s])
    return torch.cat(out)
