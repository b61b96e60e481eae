"""The work that the solver is measured on: its products, solves and per-linearisation calls.

The problems are synthetic bundle-adjustment systems of the three geometries the tests and the
benchmark use (cameras on a ring, along a walk, on a spherical cap with unevenly popular cameras),
drawn here on the GPU from a seed: a camera model with two radial terms, one pixel of noise, and
the Jacobians at a perturbed state.  `exact` recomputes every result from the same Jacobian blocks
with plain FP64 torch operations.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import torch

import paper_2110_04015_amd as ba

F64 = torch.float64

# Observers of a landmark (mean), by geometry.  walk and cap: 2 and 5 plus a geometric count.
_OBSERVERS = {"walk": 7.8, "cap": 9.0}


# ---------------------------------------------------------------------- problems


class _Draw:
    """Seeded random numbers on the device."""

    def __init__(self, seed, device):
        self.device = device
        self.g = torch.Generator(device=device)
        self.g.manual_seed(int(seed) * 7919 + 17)

    def uniform(self, lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(*shape, generator=self.g, device=self.device, dtype=F64)

    def normal(self, sigma, *shape):
        return sigma * torch.randn(*shape, generator=self.g, device=self.device, dtype=F64)

    def integers(self, lo, hi, n):
        return torch.randint(lo, hi, (n,), generator=self.g, device=self.device)

    def geometric(self, p, n):
        """Failures before the first success."""
        u = self.uniform(0.0, 1.0, n).clamp_(min=1e-300)
        return torch.floor(torch.log(u) / math.log1p(-p)).to(torch.int64)


def _cross(a, b):
    return torch.linalg.cross(a, b, dim=-1)


def _rotate(R, x):
    """R x for rows of 3 x 3 matrices and vectors."""
    return (R * x[..., None, :]).sum(-1)


def _matmul3(A, B):
    return (A[..., :, :, None] * B[..., None, :, :]).sum(-2)


def _look_at(C, target):
    z = target - C
    z = z / z.norm(dim=-1, keepdim=True)
    x = _cross(z, torch.tensor([0.0, 0.0, 1.0], dtype=F64, device=C.device).expand_as(z))
    x = x / x.norm(dim=-1, keepdim=True)
    return torch.stack([x, _cross(z, x), z], dim=-2)


def _skew(w):
    o = torch.zeros_like(w[..., 0])
    return torch.stack([torch.stack([o, -w[..., 2], w[..., 1]], -1), torch.stack([w[..., 2], o, -w[..., 0]], -1),
                        torch.stack([-w[..., 1], w[..., 0], o], -1)], -2)


def _exp(w):
    """Rotations exp([w]x) of rotation vectors."""
    t = w.norm(dim=-1)[..., None, None].clamp(min=1e-12)
    K = _skew(w)
    return torch.eye(3, dtype=F64, device=w.device) + torch.sin(t) / t * K + (1 - torch.cos(t)) / t ** 2 * _matmul3(K, K)


def _project(cams, X, cam, lm):
    """Pixels and the two Jacobian blocks of every observation; cams rows are R, t, f, k1, k2."""
    c = cams[cam]
    R, f, k1, k2 = c[:, :9].reshape(-1, 3, 3), c[:, 12], c[:, 13], c[:, 14]
    P = _rotate(R, X[lm]) + c[:, 9:12]
    iz = 1.0 / P[:, 2]
    p = P[:, :2] * iz[:, None]
    q = (p * p).sum(1)
    s = 1.0 + k1 * q + k2 * q * q
    u = (f * s)[:, None] * p
    M = (f * (2.0 * k1 + 4.0 * k2 * q))[:, None, None] * p[:, :, None] * p[:, None, :]
    M[:, 0, 0] += f * s
    M[:, 1, 1] += f * s
    A = torch.cat([M * iz[:, None, None], -(M * p[:, None, :]).sum(2, keepdim=True) * iz[:, None, None]], 2)
    J_p = torch.cat([-_matmul3(A, _skew(P)), A, (s[:, None] * p)[..., None], ((f * q)[:, None] * p)[..., None],
                     ((f * q * q)[:, None] * p)[..., None]], 2)
    return u, J_p, _matmul3(A, R)


def _take(keys, count):
    """The `count[i]` smallest keys of each row, smallest first: (row, column) of every one of them."""
    k = int(count.max())
    order = torch.topk(keys, k, dim=1, largest=False, sorted=True).indices
    keep = torch.arange(k, device=keys.device)[None, :] < count[:, None]
    row = torch.arange(keys.shape[0], device=keys.device)[:, None].expand_as(keep)
    return row[keep], order[keep]


def _ring(d, n, nl, lo, hi):
    """Cameras on a circle facing the centre; a landmark is seen by the nearest ones in azimuth."""
    th = 2.0 * math.pi * torch.arange(n, device=d.device, dtype=F64) / n
    C = torch.stack([20.0 * torch.cos(th), 20.0 * torch.sin(th), torch.zeros_like(th)], -1)
    R = _look_at(C, torch.zeros_like(C))
    X = d.uniform(-5.0, 5.0, nl, 3)
    count = d.integers(lo, min(hi, n) + 1, nl)
    phi = torch.atan2(X[:, 1], X[:, 0])
    w = min(hi + 2, (n - 1) // 2)
    at = (torch.round(phi / (2.0 * math.pi / n)).to(torch.int64)[:, None]
          + torch.arange(-w, w + 1, device=d.device)[None, :]) % n
    away = phi[:, None] - th[at]
    row, col = _take(torch.atan2(torch.sin(away), torch.cos(away)).abs(), torch.clamp(count, max=2 * w + 1))
    return R, C, X, at[row, col], row


def _walk(d, n, nl):
    """Cameras along a path; a landmark's observers lie in a window of cameras around its anchor."""
    window, most = 10, 60
    heading = torch.cumsum(d.normal(0.1, n), 0)
    C = torch.cumsum(torch.stack([torch.cos(heading), torch.sin(heading), d.normal(0.1, n)], -1), 0)
    C = C - C.mean(0)
    k = torch.arange(n, device=d.device)
    head = C[(k + 15).clamp(max=n - 1)] - C[(k - 15).clamp(min=0)]
    head[:, 2] = 0.0
    z = _cross(head, torch.tensor([0.0, 0.0, 1.0], dtype=F64, device=d.device).expand_as(head))
    R = _look_at(C, C + z / z.norm(dim=1, keepdim=True))
    off = torch.arange(-(most // 2), most // 2 + 1, device=d.device)
    Xs, cams, lms, have = [], [], [], 0
    while have < nl:
        m = int(1.02 * (nl - have)) + 64
        a = d.integers(0, n, m)
        depth = d.uniform(5.0, 30.0, m)
        side = d.uniform(-0.4, 0.4, m, 2) * depth[:, None]
        X = C[a] + depth[:, None] * R[a, 2] + side[:, :1] * R[a, 0] + side[:, 1:] * R[a, 1]
        count = (2 + d.geometric(1.0 / 7.0, m)).clamp(max=most)
        at = a[:, None] + off[None, :]
        ok = (off.abs()[None, :] <= torch.clamp(count // 2, min=window)[:, None]) & (at >= 0) & (at < n)
        at = at.clamp(0, n - 1)
        P = _rotate(R[at], X[:, None, :] - C[at])
        ok &= (P[..., 2] > 1.0) & (P[..., 0].abs() < 1.2 * P[..., 2]) & (P[..., 1].abs() < 1.2 * P[..., 2])
        keys = d.uniform(0.0, 1.0, m, off.numel()).masked_fill_(~ok, 2.0)
        keys[:, most // 2] = -1.0   # the anchor sees it
        count = torch.minimum(count, ok.sum(1))
        good = (count >= 2).nonzero()[: nl - have, 0]
        row, col = _take(keys[good], count[good])
        Xs.append(X[good])
        cams.append(at[good][row, col])
        lms.append(row + have)
        have += good.numel()
    return R, C, torch.cat(Xs), torch.cat(cams), torch.cat(lms)


def _cap(d, n, nl):
    """Cameras on a spherical cap over a site; observers drawn by a Zipf popularity of the cameras."""
    ct = d.uniform(math.cos(math.radians(60.0)), math.cos(math.radians(10.0)), n)
    st = torch.sqrt(1.0 - ct * ct)
    az = d.uniform(0.0, 2.0 * math.pi, n)
    C = 30.0 * torch.stack([st * torch.cos(az), st * torch.sin(az), ct], -1)
    R = _look_at(C, d.normal(1.0, n, 3) * torch.tensor([1.0, 1.0, 0.3], dtype=F64, device=d.device))
    X = d.uniform(-1.0, 1.0, nl, 3) * torch.tensor([6.0, 6.0, 2.0], dtype=F64, device=d.device)
    rank = torch.randperm(n, generator=d.g, device=d.device) + 1
    count = (5 + d.geometric(0.2, nl)).clamp(max=min(40, n))
    gumbel = -torch.log(-torch.log(d.uniform(0.0, 1.0, nl, n).clamp_(1e-300, 1.0 - 1e-16)))
    row, col = _take(1.2 * torch.log(rank.to(F64))[None, :] - gumbel, count)
    return R, C, X, col, row


def _scene(case, seed, device="cuda"):
    """One scene: the state, the observations and their Jacobian blocks, on the device."""
    d = _Draw(seed, device)
    n, nl = case["cams"], case["lms"]
    if case["geometry"] == "ring":
        R, C, X, cam, lm = _ring(d, n, nl, case["least"], case["most"])
    else:
        R, C, X, cam, lm = (_walk if case["geometry"] == "walk" else _cap)(d, n, nl)
    t = -_rotate(R, C)
    inner = torch.stack([d.uniform(400.0, 600.0, n), d.normal(1e-3, n), d.normal(1e-3, n)], 1)
    true = torch.cat([R.reshape(n, 9), t, inner], 1)
    u_obs = _project(true, X, cam, lm)[0]
    u_obs = u_obs + d.normal(1.0, *u_obs.shape)
    E = _exp(d.normal(1e-2, n, 3))
    cams = torch.cat([_matmul3(E, R).reshape(n, 9), _rotate(E, t) + d.normal(1e-2, n, 3), inner + d.normal(1e-2, n, 3)], 1)
    X = X + d.normal(1e-2, *X.shape)
    if case.get("shuffled"):   # the observations in no order, as they come from a feature matcher
        o = torch.randperm(cam.numel(), generator=d.g, device=device)
        cam, lm, u_obs = cam[o], lm[o], u_obs[o]
    u, J_p, J_l = _project(cams, X, cam, lm)
    dp = case.get("dp", 9)
    return SimpleNamespace(n_cams=n, n_lms=nl, d_p=dp, draw=d, cams=cams.contiguous(), points=X.contiguous(),
                           obs_cam=cam.to(torch.int32), obs_lm=lm.to(torch.int32), u_obs=u_obs.contiguous(),
                           J_p=J_p[:, :, :dp].contiguous(), J_l=J_l.contiguous(), r=(u - u_obs).contiguous(),
                           lam=float(case.get("lam", 1e-4)))


def _batch_scenes(case, seed, device="cuda"):
    """The uneven ring problems of one batch (200 landmarks per camera)."""
    lo, hi, count = case["least_cams"], case["most_cams"], case["problems"]
    sizes = [lo + (hi - lo) * ((7 * k) % count) // count for k in range(count)]
    return [_scene({"geometry": "ring", "cams": n, "lms": 200 * n, "least": 2, "most": 20, "lam": case["lam"]},
                   100 * seed + k, device) for k, n in enumerate(sizes)]


def _system(p, **kw):
    return ba.System(p.n_cams, p.n_lms, p.obs_cam, p.obs_lm, p.J_p, p.J_l, p.r, p.lam, **kw)


# ---------------------------------------------------------------------- cases

# Sizes of the named workloads: 50 ring cameras with 5,000 landmarks; 1,936 cameras along a walk with
# 650,000 (5.1M observations, a banded S); 571 on a cap with 100,000 (0.9M, a dense S, 47 subsets).
_RING50 = {"geometry": "ring", "cams": 50, "lms": 5000, "least": 2, "most": 8}
_WALK = {"geometry": "walk", "cams": 1936, "lms": 650_000}
_CAP = {"geometry": "cap", "cams": 571, "lms": 100_000}

# Solves: with the first lambda of an LM run, 1e-4, to the usual 1e-6 (the multidirectional solver, which
# keeps its directions conjugate) or stopped after `steps` iterations, an inexact LM step; with a lambda
# after rejected steps to 1e-6 or, through refinement, to 1e-12.


def listed():
    return [
        # one S v of the smallest problem: what a caller with its own Krylov loop pays per call
        dict(name="matvec_ring50", kind="matvec", precision="fp64", **_RING50),
        # one S v of a ragged, shuffled middle-sized scene from FP32 Jacobians
        dict(name="matvec_ring333_fp32", kind="matvec", precision="fp32", geometry="ring", cams=333, lms=61_111, least=2,
             most=20, shuffled=True),
        # one S v of the largest scene: the product that most of a large solve consists of
        dict(name="matvec_walk1936", kind="matvec", precision="fp64", **_WALK),
        # S on the pose subsets of a multidirectional step, banded S
        dict(name="grouped_walk1936", kind="grouped", precision="fp64", N=16, **_WALK),
        # the same on a dense S, with its many subsets
        dict(name="grouped_cap571", kind="grouped", precision="fp64", N=47, **_CAP),
        # a whole small solve: launches and round trips
        dict(name="pcg_ring50", kind="pcg", precision="fp64", lam=1e-2, eps=1e-6, **_RING50),
        # an inexact PCG step of the largest scene
        dict(name="pcg_walk1936", kind="pcg", precision="fp64", steps=24, **_WALK),
        # the multidirectional solver on the largest scene, to the end
        dict(name="mcg_walk1936", kind="mcg", precision="fp64", N=16, tau=3.3, lam=1e-4, eps=1e-6, **_WALK),
        # mixed precision on the dense scene: FP32 products under FP64 refinement
        dict(name="mcg_cap571_fp32", kind="mcg", precision="fp32", N=47, tau=10.0, lam=1e-2, eps=1e-12, **_CAP),
        # the explicit S of the dense scene
        dict(name="mcg_cap571_explicit", kind="mcg", precision="fp64", N=47, tau=10.0, lam=1e-4, eps=1e-6,
             explicit=True, **_CAP),
        # many uneven problems served together
        dict(name="batch_24_rings", kind="batch", precision="fp32", N=16, tau=3.3, lam=1e-2, eps=1e-12, problems=24,
             least_cams=50, most_cams=200),
        # everything of an LM iteration around its solve, on the largest scene
        dict(name="relinearise_walk1936", kind="relinearise", **_WALK),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["matvec", "matvec", "grouped", "pcg", "mcg", "mcg", "batch", "relinearise"])
    if kind == "batch":
        most = rng.randint(60, 200)
        return dict(kind=kind, precision=rng.choice(["fp64", "fp32"]), N=rng.choice([1, 4, 16]), tau=3.3, lam=1e-2, eps=1e-12,
                    problems=rng.randint(2, 24), least_cams=rng.randint(30, 50), most_cams=most)
    geometry = rng.choice(["ring", "walk", "cap"])
    if geometry == "ring":
        cams = _log_uniform(rng, 50, 800)
        c = dict(kind=kind, geometry=geometry, cams=cams, lms=cams * rng.randint(80, 200) + rng.randint(0, 63), least=2,
                 most=rng.randint(6, 20))
    elif geometry == "walk":
        cams = _log_uniform(rng, 60, 1900)
        c = dict(kind=kind, geometry=geometry, cams=cams, lms=cams * rng.randint(150, 335) + rng.randint(0, 63))
    else:
        cams = _log_uniform(rng, 60, 570)
        c = dict(kind=kind, geometry=geometry, cams=cams, lms=cams * rng.randint(120, 175) + rng.randint(0, 63))
    if rng.random() < 0.3:
        c["shuffled"] = True
    if kind == "relinearise":
        return c
    if kind in ("matvec", "grouped"):
        c["precision"] = rng.choice(["fp64", "fp64", "fp32", "bf16"])
        if kind == "grouped":
            c["N"] = rng.choice([2, 4, 8, 16, 29, 47])
    elif kind == "pcg" and rng.random() < 0.5:
        c.update(precision="fp64", steps=rng.randint(6, 24))
    else:
        precision = rng.choice(["fp64", "fp64", "fp32"])
        c.update(precision=precision, lam=1e-2, eps=1e-12 if precision == "fp32" else 1e-6)
        if kind == "mcg":
            c.update(N=rng.choice([2, 4, 8, 16, 29, 47]), tau=rng.choice([3.3, 10.0]))
            c["lam"] = 1e-2 if precision == "fp32" else 1e-4
    if rng.random() < 0.2:   # poses without intrinsics
        c["dp"] = 6
    elif kind in ("pcg", "mcg") and c["precision"] == "fp64" and rng.random() < 0.25:
        c["explicit"] = True
    return c


def _random_vector(p):
    return p.draw.normal(1.0, p.d_p * p.n_cams)


def prepare(case, seed):
    kind = case["kind"]
    s = SimpleNamespace(case=case)
    if kind == "batch":
        host = []
        for p in _batch_scenes(case, seed):
            host.append(SimpleNamespace(n_cams=p.n_cams, n_lms=p.n_lms, lam=p.lam,
                                        **{k: getattr(p, k).cpu().numpy() for k in ("obs_cam", "obs_lm", "J_p", "J_l", "r")}))
        s.batch = ba.Batch(host, store_fp32=case["precision"] == "fp32")
        return s
    p = _scene(case, seed)
    precision = case.get("precision", "fp64")
    s.system = _system(p, store_fp32=precision == "fp32", store_bf16=precision == "bf16",
                       explicit_schur=bool(case.get("explicit")))
    if kind in ("matvec", "grouped"):
        s.v = _random_vector(p)
    if kind in ("grouped", "mcg"):
        s.system.prepare_mcg(case["N"], precision)
    if kind == "relinearise":
        s.scene = ba.Scene(p.n_cams, p.n_lms, p.obs_cam, p.obs_lm, p.u_obs)
        s.cams, s.points, s.lam = p.cams, p.points, p.lam
        s.step = 1e-3 * _random_vector(p)
    return s


def run(s):
    case, kind = s.case, s.case["kind"]
    if kind == "matvec":
        return s.system.matvec(s.v, precision=case["precision"])
    if kind == "grouped":
        return s.system.matmat_grouped(case["N"], s.v, precision=case["precision"])
    if kind == "relinearise":
        r, J_p, J_l, cost = s.scene.project(s.cams, s.points)
        s.system.update(J_p, J_l, r, s.lam)
        rhs = s.system.rhs()
        points_step = s.system.back_substitute(s.step)
        cams, points = s.scene.apply_step(s.cams, s.points, s.step, points_step)
        return {"cost": cost, "rhs": rhs, "blocks": s.system.precond_blocks(), "points_step": points_step, "cams": cams,
                "points": points}
    stop = dict(eps=1e-14, max_iter=case["steps"]) if "steps" in case else dict(eps=case["eps"])
    if kind == "pcg":
        return s.system.pcg(precision=case["precision"], **stop)[0]
    if kind == "mcg":
        return s.system.mcg(case["N"], case["tau"], precision=case["precision"], **stop)[0]
    return s.batch.mcg(case["N"], case["tau"], precision=case["precision"], **stop)[0]


def _observations(case):
    if case["kind"] == "batch":
        return 200 * case["problems"] * (case["least_cams"] + case["most_cams"]) / 2 * 11.0
    return case["lms"] * ((case["least"] + case["most"]) / 2 if case["geometry"] == "ring" else _OBSERVERS[case["geometry"]])


def work(case):
    """One pass over the Jacobian blocks per product: 2 d_p + 6 values and an index per observation,
    the inverse of each landmark's block, the vectors."""
    kind, m = case["kind"], _observations(case)
    dp = case.get("dp", 9)
    if kind == "batch":
        n_cams = case["problems"] * (case["least_cams"] + case["most_cams"]) / 2
        nl = 200 * n_cams
    else:
        n_cams, nl = case["cams"], case["lms"]
    n = dp * n_cams
    if kind == "relinearise":
        per_obs = 24 + 24 * 8 + 16          # indices and pixels read, blocks and residual written
        return {"bytes": m * (per_obs + 2 * 24 * 8 + 16) + nl * 3 * 8 * 4 + n_cams * 15 * 16,
                "flops": m * 2.0 * (9 * 9 + 9 * 3 + 3 * 3 + 60)}
    size = {"fp64": 8, "fp32": 4, "bf16": 2}[case.get("precision", "fp64")]
    product = m * ((2 * dp + 6) * size + 4) + nl * 48 + 2 * n * 8
    flops = m * (8.0 * dp + 24) + nl * 30.0
    if kind == "matvec":
        return {"bytes": product, "flops": flops}
    if kind == "grouped":
        return {"bytes": product + (case["N"] - 1) * n * 8, "flops": flops}
    # iterations that such a solve takes, about: by lambda and by how far S couples the cameras
    products = case.get("steps") or {1e-4: 200, 1e-2: 45}[case["lam"]] * (2 if case["eps"] < 1e-9 else 1)
    if case.get("geometry") == "cap":
        products = min(products, 30)
    if case.get("explicit"):
        pairs = min(n_cams * n_cams, 90.0 * n_cams) if case["geometry"] == "walk" else 0.8 * n_cams * n_cams
        product, flops = pairs * 648 + 2 * n * 8, pairs * 162.0
    return {"bytes": products * (product + 6 * n * 8), "flops": products * flops}


# ---------------------------------------------------------------------- the same results from plain torch in 64 bits


class _Plain:
    """S, the right-hand side and the block-Jacobi preconditioner, factor by factor."""

    def __init__(self, p):
        self.p, dp = p, p.d_p
        self.cam, self.lm = p.obs_cam.long(), p.obs_lm.long()
        self.J_p, self.J_l = p.J_p, p.J_l
        dev = p.J_p.device
        V = torch.zeros(p.n_lms, 3, 3, dtype=F64, device=dev).index_add_(0, self.lm, _gram(p.J_l, p.J_l))
        U = torch.zeros(p.n_cams, dp, dp, dtype=F64, device=dev).index_add_(0, self.cam, _gram(p.J_p, p.J_p))
        V += torch.diag_embed(p.lam * V.diagonal(dim1=1, dim2=2))
        self.damp = p.lam * U.diagonal(dim1=1, dim2=2)
        self.V_inv = torch.linalg.inv(V)
        b_l = self.to_landmarks(p.r)
        h = _rotate(self.V_inv, b_l)
        self.b = self.to_cameras(p.r - _rotate(p.J_l, h[self.lm])).reshape(-1)
        W = _gram(p.J_p, p.J_l)
        D = U + torch.diag_embed(self.damp)
        D -= torch.zeros_like(D).index_add_(0, self.cam, _mm(_mm(W, self.V_inv[self.lm]), W.transpose(1, 2)))
        self.D, self.D_inv = D, torch.linalg.inv(D)

    def to_landmarks(self, e):
        out = torch.zeros(self.p.n_lms, 3, dtype=F64, device=e.device)
        return out.index_add_(0, self.lm, (self.J_l * e[:, :, None]).sum(1))

    def to_cameras(self, e):
        out = torch.zeros(self.p.n_cams, self.p.d_p, dtype=F64, device=e.device)
        return out.index_add_(0, self.cam, (self.J_p * e[:, :, None]).sum(1))

    def times(self, v):
        v = v.reshape(self.p.n_cams, self.p.d_p)
        e = _rotate(self.J_p, v[self.cam])
        h = _rotate(self.V_inv, self.to_landmarks(e))
        return (self.to_cameras(e - _rotate(self.J_l, h[self.lm])) + self.damp * v).reshape(-1)

    def precondition(self, r):
        return _rotate(self.D_inv, r.reshape(self.p.n_cams, self.p.d_p)).reshape(-1)

    def solve(self, eps, most):
        """Block-Jacobi preconditioned conjugate gradients on S x = -b from zero."""
        x = torch.zeros_like(self.b)
        r = -self.b
        z = self.precondition(r)
        q, rho, stop = z.clone(), r @ z, eps * float(r.norm())
        for _ in range(most):
            s = self.times(q)
            a = rho / (q @ s)
            x += a * q
            r -= a * s
            if float(r.norm()) < stop:
                break
            z = self.precondition(r)
            rho, old = r @ z, rho
            q = z + (rho / old) * q
        return x


def _gram(A, B):
    """A^T B of the 2-row blocks of every observation."""
    return A[:, 0, :, None] * B[:, 0, None, :] + A[:, 1, :, None] * B[:, 1, None, :]


def _mm(A, B):
    return sum(A[:, :, k, None] * B[:, k, None, :] for k in range(A.shape[2]))


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return torch.cat([_Plain(p).solve(1e-15, 400) for p in _batch_scenes(case, seed)])
    p = _scene(case, seed)
    if kind == "relinearise":
        step = 1e-3 * _random_vector(p)
        A = _Plain(p)
        s = step.reshape(-1, 9)
        back = _rotate(A.V_inv, A.to_landmarks(-p.r - _rotate(A.J_p, s[A.cam])))
        E = _exp(s[:, :3])
        R = p.cams[:, :9].reshape(-1, 3, 3)
        cams = torch.cat([_matmul3(E, R).reshape(-1, 9), _rotate(E, p.cams[:, 9:12]) + s[:, 3:6], p.cams[:, 12:] + s[:, 6:]], 1)
        return {"cost": float((p.r * p.r).sum()), "rhs": A.b, "blocks": A.D, "points_step": back.reshape(-1), "cams": cams,
                "points": p.points + back}
    A = _Plain(p)
    if kind == "matvec":
        return A.times(_random_vector(p))
    if kind == "grouped":
        v, N = _random_vector(p).reshape(p.n_cams, p.d_p), case["N"]
        group = torch.clamp(torch.arange(p.n_cams, device=v.device) // (p.n_cams // N), max=N - 1)
        return torch.stack([A.times(torch.where((group == g)[:, None], v, 0.0)) for g in range(N)])
    if "steps" in case:
        return A.solve(1e-14, case["steps"])
    if case["eps"] > 1e-9:   # an iterate that is not yet the solution
        return None
    return A.solve(1e-15, 600)
