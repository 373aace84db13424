"""What this library is measured on: solves, batches and requests as a user's program makes them.

A case is a dict of plain values; ``prepare`` makes its inputs (seeded, the scene shapes of
the paper's workloads) and whatever such a program keeps (a problem handle, a server),
``run`` takes one pass through the public entry points, ``exact`` gives the same outputs in
64-bit torch without the library, ``work`` what one pass cannot do without.

The scene generators are written with torch so that a case is made quickly; they hold no
solver arithmetic.  ``exact`` is a plain matrix-free Gauss-Newton / Schur solver.

Results of a solve come back in the precision the caller chose: a program that asks for
the FP64 mode keeps its poses and map in float64, one that asks for an FP32 mode (or one
with 16-bit Jacobians) keeps them in float32.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2510_15271_amd import ba

F = 500.0                  # pinhole of every scene: fx = fy = 500, 640 x 480
CX, CY, W, H = 320.0, 240.0, 640.0, 480.0


# ------------------------------------------------------------------------------ the cases

def listed():
    return [
        # the sliding window of an online system, its oldest frames held: the smallest solve, all latency
        dict(name="window_f32", kind="drive", cams=24, pts=1777, fixed=4, iters=10, pcg=50, tol=1e-6, prec="f32", huber=1.0,
             outliers=0.0, resident=False),
        # the parity build on a handful of views, PCG run to the end (the tiny FP64 scene of bench.py)
        dict(name="tiny_f64", kind="arc", cams=10, pts=1000, iters=20, pcg=200, tol=1e-14, prec="f64", huber=0.0,
             outliers=0.0, resident=True),
        # a submap: a few hundred frames of one drive, 16-bit Jacobian storage, the default launch mode
        dict(name="submap_bf16j", kind="drive", cams=203, pts=40000, fixed=2, iters=10, pcg=50, tol=1e-6, prec="bf16j",
             huber=1.0, outliers=0.0, resident=False),
        # the headline: the 2M-observation sequential drive, alone on the device
        dict(name="drive_f32", kind="drive", cams=500, pts=250000, fixed=1, iters=10, pcg=50, tol=1e-6, prec="f32", huber=0.0,
             outliers=0.0, resident=True),
        # the largest map: two laps with loop closures, 5 % outliers, Huber
        dict(name="loop_f32", kind="loop", cams=3000, pts=1200000, fixed=1, iters=15, pcg=50, tol=1e-6, prec="f32", huber=1.0,
             outliers=0.05, resident=True),
        # dense co-visibility (every camera sees most points) near the top of the serving range, FP16 Jacobians
        dict(name="arc_f16j", kind="arc", cams=197, pts=20011, iters=20, pcg=50, tol=1e-6, prec="f16j", huber=0.0,
             outliers=0.0, resident=False),
        # a mixed-size stream through the server, every request submitted at once
        dict(name="serve_f32", kind="serve", n=16, cams=120, pts=16000, iters=20, pcg=50, tol=1e-6, prec="f32"),
        # extrinsic refinement of a three-camera rig
        dict(name="rig_f32", kind="rig", frames=200, pts=20000, iters=10, pcg=100, tol=1e-6, prec="f32"),
        # a pose graph of two laps with loop closures and absolute (GNSS) priors
        dict(name="graph_f32", kind="graph", frames=1500, iters=10, pcg=50, tol=1e-6, prec="f32", prior=0.1,
             resident=True),
        # one localisation request: the smallest call
        dict(name="pose_one", kind="pose", n=1, lo=400, hi=401, iters=10),
        # a batch of localisation requests
        dict(name="pose_batch", kind="pose", n=4096, lo=100, hi=2000, iters=10),
        # triangulation of every track of a map from scratch, with outliers
        dict(name="ransac_tracks", kind="tri", cams=400, pts=120000, n_hyp=64, outliers=0.05, method="midpoint"),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["drive", "drive", "arc", "arc", "pose", "tri", "graph", "rig", "serve"])
    prec = rng.choice(["f32", "f32", "f64", "f16j", "bf16j"])
    if kind == "drive":
        cams = log(8, 500)
        out = rng.choice([0.0, 0.02, 0.05])
        return dict(kind=kind, cams=cams, pts=cams * log(50, 400) + rng.randrange(97), fixed=max(1, cams // 12), iters=rng.choice([5, 10, 15]),
                    pcg=50, tol=1e-6, prec=prec if prec != "f64" else "f32", huber=1.0 if out else 0.0, outliers=out,
                    resident=rng.random() < 0.5)
    if kind == "arc":
        return dict(kind=kind, cams=log(5, 150), pts=log(1000, 12000), iters=rng.choice([10, 20]),
                    pcg=200 if prec == "f64" else 50, tol=1e-14 if prec == "f64" else 1e-6, prec=prec, huber=0.0,
                    outliers=0.0, resident=rng.random() < 0.5)
    if kind == "pose":
        lo = log(50, 500)
        return dict(kind=kind, n=log(1, 2000), lo=lo, hi=lo + log(1, 1500), iters=rng.choice([5, 10]))
    if kind == "tri":
        return dict(kind=kind, cams=log(20, 400), pts=log(1000, 100000), n_hyp=rng.choice([16, 32, 64]),
                    outliers=rng.choice([0.02, 0.05, 0.1]), method=rng.choice(["midpoint", "dlt"]))
    if kind == "graph":
        return dict(kind=kind, frames=log(40, 1500), iters=rng.choice([5, 10]), pcg=50, tol=1e-6, prec="f32", prior=0.1,
                    resident=rng.random() < 0.5)
    if kind == "rig":
        f = log(30, 200)
        return dict(kind=kind, frames=f, pts=f * log(50, 100), iters=10, pcg=100, tol=1e-6, prec="f32")
    return dict(kind="serve", n=rng.randrange(4, 13), cams=log(20, 100), pts=log(2000, 12000), iters=rng.choice([10, 20]),
                pcg=50, tol=1e-6, prec=prec if prec != "f64" else "f32")


# ------------------------------------------------------------------------------ generators

def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


class _Rng:
    def __init__(self, seed):
        self.d = _dev()
        self.g = torch.Generator(device=self.d)
        self.g.manual_seed(int(seed))

    def u(self, lo, hi, *n):
        return lo + (hi - lo) * torch.rand(*n, generator=self.g, device=self.d, dtype=torch.float64)

    def n(self, s, *n):
        return s * torch.randn(*n, generator=self.g, device=self.d, dtype=torch.float64)

    def i(self, lo, hi, n):
        return torch.randint(lo, hi, (n,), generator=self.g, device=self.d)

    def geom(self, p, n):  # 1, 2, ...
        return torch.ceil(torch.log1p(-self.u(0.0, 1.0, n)) / math.log1p(-p)).clamp(min=1).long()

    def unit(self, n):
        v = self.n(1.0, n, 3)
        return v / v.norm(dim=1, keepdim=True)


def _hat(v):
    z = torch.zeros_like(v[..., 0])
    return torch.stack([z, -v[..., 2], v[..., 1], v[..., 2], z, -v[..., 0], -v[..., 1], v[..., 0], z],
                       -1).reshape(*v.shape[:-1], 3, 3)


def _mm(A, B):
    """Products of small matrices, batched (no library batched product: elementwise and a sum)."""
    return (A.unsqueeze(-1) * B.unsqueeze(-3)).sum(-2)


def _mv(A, v):
    return (A * v.unsqueeze(-2)).sum(-1)


def _se3(xi):
    """Exp of (rho, phi): rotation and translation."""
    rho, phi = xi[..., :3], xi[..., 3:]
    th2 = (phi * phi).sum(-1)[..., None, None]
    th = th2.sqrt().clamp(min=1e-300)
    small = th2 < 1e-8
    A = torch.where(small, 1 - th2 / 6 + th2 * th2 / 120, torch.sin(th) / th)
    h = torch.where(small, 1 - th2 / 24, torch.sin(th / 2) / (th / 2))
    B = torch.where(small, 0.5 - th2 / 24 + th2 * th2 / 720, 0.5 * h * h)
    C = torch.where(small, 1 / 6 - th2 / 120 + th2 * th2 / 5040, (th - torch.sin(th)) / (th2 * th).clamp(min=1e-300))
    K = _hat(phi)
    K2 = _mm(K, K)
    I = torch.eye(3, dtype=xi.dtype, device=xi.device)
    return I + A * K + B * K2, _mv(I + B * K + C * K2, rho)


def _rot(v):
    return _se3(torch.cat([torch.zeros_like(v), v], -1))[0]


def _quat(R):
    """(w, x, y, z), w >= 0, from rotation matrices (rotations of the scenes and results)."""
    m = R.reshape(-1, 9).T
    q2 = torch.stack([1 + m[0] + m[4] + m[8], 1 + m[0] - m[4] - m[8], 1 - m[0] + m[4] - m[8], 1 - m[0] - m[4] + m[8]], 1)
    a, b, c = m[7] - m[5], m[2] - m[6], m[3] - m[1]
    d, e, f = m[3] + m[1], m[2] + m[6], m[7] + m[5]
    rows = torch.stack([torch.stack([q2[:, 0], a, b, c], 1), torch.stack([a, q2[:, 1], d, e], 1),
                        torch.stack([b, d, q2[:, 2], f], 1), torch.stack([c, e, f, q2[:, 3]], 1)], 1)
    q = rows[torch.arange(q2.shape[0], device=R.device), q2.argmax(1)]
    q = q / q.norm(dim=1, keepdim=True)
    return torch.where(q[:, :1] < 0, -q, q)


def _matrix(q):
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).T
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y), 2 * (x * y + w * z),
                        1 - 2 * (x * x + z * z), 2 * (y * z - w * x), 2 * (x * z - w * y), 2 * (y * z + w * x),
                        1 - 2 * (x * x + y * y)], 1).reshape(-1, 3, 3)


def _look(fwd):
    """World -> camera rotations with the optical axis along fwd (x-z plane), y down."""
    y = torch.zeros_like(fwd)
    y[:, 1] = 1.0
    x = torch.linalg.cross(y, fwd)
    x = x / x.norm(dim=1, keepdim=True)
    return torch.stack([x, torch.linalg.cross(fwd, x), fwd], 1)


def _project(R, c, X):
    P = _mv(R, X - c)
    uv = torch.stack([F * P[:, 0] / P[:, 2] + CX, F * P[:, 1] / P[:, 2] + CY], 1)
    seen = (P[:, 2] > 0.5) & (uv[:, 0] >= 0) & (uv[:, 0] < W) & (uv[:, 1] >= 0) & (uv[:, 1] < H)
    return uv, seen


def _curve(n, d):
    """n frames 1 m apart, heading 0.3 sin(2 pi s / 500)."""
    s = torch.arange(n, device=d, dtype=torch.float64)
    h = 0.3 * torch.sin(2 * math.pi * s / 500.0)
    step = torch.stack([torch.sin(h), torch.zeros_like(h), torch.cos(h)], 1)
    return _look(step), torch.cumsum(step, 0) - step


def _back_project(g, R, c, last):
    """A point per track: a uniform pixel at 3 to 40 m of its last frame."""
    n = last.shape[0]
    d = g.u(3.0, 40.0, n)
    ray = torch.stack([(g.u(0, W, n) - CX) / F, (g.u(0, H, n) - CY) / F, torch.ones_like(d)], 1) * d[:, None]
    return c[last] + _mv(R[last].transpose(1, 2), ray)


def _spans(first, length):
    """(index of the span, frame) of every frame of the spans [first, first + length)."""
    idx = torch.repeat_interleave(torch.arange(first.shape[0], device=first.device), length)
    off = torch.arange(idx.shape[0], device=first.device) - (torch.cumsum(length, 0) - length)[idx]
    return idx, first[idx] + off


def _scene(g, R, c, X, cam, pt, first, case):
    """Pixels with noise and outliers, a drifted start (the first frames exact and fixed),
    points carried with the drifted pose of their first frame; points without parallax are
    left out, as a front end does."""
    uv, seen = _project(R[cam], c[cam], X[pt])
    cam, pt, uv = cam[seen], pt[seen], uv[seen]
    keep = _first(_parallax(X, c, cam, pt) > 1.5, case["pts"])
    ok = keep[pt]
    cam, pt, uv = cam[ok], (torch.cumsum(keep, 0) - 1)[pt[ok]], uv[ok]
    X, first = X[keep], first[keep]
    if case.get("obs"):  # a front end loses some of a track's views: so many are left
        o = torch.randperm(cam.shape[0], generator=g.g, device=g.d)[:case["obs"]]
        cam, pt, uv = cam[o], pt[o], uv[o]
    o = torch.argsort(cam, stable=True)  # camera-major, as an image database holds it
    cam, pt, uv = cam[o], pt[o], uv[o] + g.n(0.7, uv.shape[0], 2)
    bad = g.u(0, 1, uv.shape[0]) < case["outliers"]
    uv = torch.where(bad[:, None], torch.stack([g.u(0, W, uv.shape[0]), g.u(0, H, uv.shape[0])], 1), uv)
    n = c.shape[0]
    dr, dt = g.n(0.002, n, 3), g.n(0.01, n, 3)
    dr[:case["fixed"]] = dt[:case["fixed"]] = 0
    R0 = _mm(R, _rot(torch.cumsum(dr, 0)).transpose(1, 2))
    c0 = c + torch.cumsum(dt, 0)
    X0 = c0[first] + _mv(R0[first].transpose(1, 2), _mv(R[first], X - c[first])) + g.n(0.05, X.shape[0], 3)
    return _host(R0, -_mv(R0, c0), X0, cam, pt, uv, case)


def _first(keep, n):
    """The first n of the marked."""
    rank = torch.cumsum(keep, 0)
    if int(rank[-1]) < n:
        raise ValueError("the scene has too few points")
    return keep & (rank <= n)


def _parallax(X, c, cam, pt):
    """Degrees between the rays of each point's first and last cameras (0 with one view)."""
    p = X.shape[0]
    lo = torch.full((p,), 1 << 30, device=X.device).scatter_reduce_(0, pt, cam, "amin")
    hi = torch.full((p,), -1, device=X.device).scatter_reduce_(0, pt, cam, "amax")
    lo = torch.where(hi < 0, 0, lo)
    a, b = X - c[lo], X - c[hi.clamp(min=0)]
    x = (a * b).sum(1) / (a.norm(dim=1) * b.norm(dim=1))
    return torch.where(hi > lo, torch.rad2deg(torch.acos(x.clamp(-1, 1))), 0.0)


def _host(R0, t0, X0, cam, pt, uv, case):
    n = R0.shape[0]
    fixed = np.zeros(n, np.uint8)
    fixed[:case["fixed"]] = 1
    fixed[n - case.get("fixed_last", 0):] = 1
    return SimpleNamespace(K=np.tile([F, F, CX, CY], (n, 1)), q0=_quat(R0).cpu().numpy(), t0=t0.cpu().numpy(),
                           X0=X0.cpu().numpy(), obs_cam=cam.int().cpu().numpy(), obs_pt=pt.int().cpu().numpy(),
                           obs_uv=uv.cpu().numpy(), cam_fixed=fixed, huber_delta=case["huber"])


def _drive(case, seed):
    g = _Rng(seed)
    n, p = case["cams"], 2 * case["pts"] + 200
    R, c = _curve(n, g.d)
    s = g.i(0, n - 1, p)
    L = torch.minimum(1 + g.geom(1 / 7, p), n - s)
    X = _back_project(g, R, c, s + L - 1)
    pt, cam = _spans(s, L)
    return _scene(g, R, c, X, cam, pt, s, case)


def _loop(case, seed):
    """One circle driven twice, the second lap 1 m inside; a quarter of the points on both."""
    g = _Rng(seed)
    n, p = case["cams"] // 2, 3 * case["pts"]
    h = 2 * math.pi * torch.arange(n, device=g.d, dtype=torch.float64) / n
    z, r = torch.zeros_like(h), n / (2 * math.pi)
    R = _look(torch.stack([torch.sin(h), z, torch.cos(h)], 1)).repeat(2, 1, 1)
    c = torch.stack([r * (1 - torch.cos(h)), z, r * torch.sin(h)], 1)
    c = torch.cat([c, c + torch.stack([torch.cos(h), z, -torch.sin(h)], 1)])
    both = torch.arange(p, device=g.d) % 4 == 0
    s = torch.where(both, g.i(0, n - 1, p), g.i(0, 2 * n - 1, p))
    L = torch.minimum(1 + g.geom(1 / 5, p), torch.where(both, n - s, 2 * n - s))
    X = _back_project(g, R, c, s + L - 1)
    pt, cam = _spans(s, L)
    pt2, cam2 = _spans(s[::4] + n, L[::4])
    return _scene(g, R, c, X, torch.cat([cam, cam2]), torch.cat([pt, 4 * pt2]), s, case)


def _arc(case, seed):
    """Cameras on a 2 m arc looking at a box that all of them see; the end cameras are held."""
    g = _Rng(seed)
    n, p = case["cams"], case["pts"] + case["pts"] // 2
    a = torch.linspace(-1 / 6, 1 / 6, n, device=g.d, dtype=torch.float64)
    c = torch.stack([6 * torch.sin(a), torch.zeros_like(a), 6 - 6 * torch.cos(a)], 1)
    R = _look((torch.tensor([0.0, 0.0, 6.0], device=g.d, dtype=torch.float64) - c) / 6)
    X = torch.stack([g.u(-2, 2, p), g.u(-2, 2, p), g.u(2, 10, p)], 1)
    cam = torch.arange(n, device=g.d).repeat_interleave(p)
    pt = torch.arange(p, device=g.d).repeat(n)
    uv, seen = _project(R[cam], c[cam], X[pt])
    keep = _first(torch.bincount(pt[seen], minlength=p) >= max(2, n // 2), case["pts"])
    seen &= keep[pt]
    cam, pt, uv = cam[seen], (torch.cumsum(keep, 0) - 1)[pt[seen]], uv[seen] + g.n(0.5, int(seen.sum()), 2)
    X = X[keep]
    p = X.shape[0]
    dr, dt = 0.01 * g.unit(n), 0.05 * g.unit(n)
    dr[0] = dt[0] = dr[-1] = dt[-1] = 0
    return _host(_mm(_rot(dr), R), -_mv(R, c) + dt, X + 0.05 * g.unit(p), cam, pt, uv,
                 dict(case, fixed=1, fixed_last=1, huber=0.0))


def _mounts(d):
    """Vehicle -> camera of the rig: yaws 0 and +-60 degrees, 0.5 m along the optical axis."""
    out = []
    for yaw in (0.0, 60.0, -60.0):
        Re = _rot(torch.tensor([[0.0, math.radians(yaw), 0.0]], device=d, dtype=torch.float64))[0].T.contiguous()
        out.append((Re, torch.tensor([0.0, 0.0, -0.5], device=d, dtype=torch.float64)))
    return torch.stack([a for a, _ in out]), torch.stack([b for _, b in out])


def _rig(case, seed):
    """Each point is tracked by one camera; the others see it where they can, also in the
    20 frames after the track."""
    g = _Rng(seed)
    n, per = case["frames"], case["pts"]  # three times as many as are kept, from each camera
    Rv, cv = _curve(n, g.d)
    tv = -_mv(Rv, cv)
    Re, te = _mounts(g.d)
    Rc = [_mm(Re[k], Rv) for k in range(3)]
    cc = [-_mv(Rc[k].transpose(1, 2), _mv(Re[k], tv) + te[k]) for k in range(3)]
    Xs, S, own, obs = [], [], [], []
    for k in range(3):
        s = g.i(0, n - 1, per)
        L = torch.minimum(1 + g.geom(1 / 7, per), n - s)
        X = _back_project(g, Rc[k], cc[k], s + L - 1)
        for k2 in range(3):
            i, f = _spans(s, L if k2 == k else torch.minimum(L + 20, n - s))
            uv, seen = _project(Rc[k2][f], cc[k2][f], X[i])
            obs.append((f[seen], torch.full_like(f[seen], k2), i[seen] + k * per, uv[seen]))
        Xs.append(X)
        S.append(s)
        own.append(torch.full_like(s, k))
    f, k, pt, uv = (torch.cat([o[j] for o in obs]) for j in range(4))
    X, s, own = torch.cat(Xs), torch.cat(S), torch.cat(own)
    keep = _parallax(X, cv, f, pt) > 1.5
    keep = torch.cat([_first(keep[own == j], case["pts"] // 3) for j in range(3)])
    ok = keep[pt]
    f, k, pt, uv = f[ok], k[ok], (torch.cumsum(keep, 0) - 1)[pt[ok]], uv[ok] + g.n(0.7, int(ok.sum()), 2)
    X, s, own = X[keep], s[keep], own[keep]
    dr, dt = g.n(0.002, n, 3), g.n(0.01, n, 3)
    dr[0] = dt[0] = 0
    Rv0 = _mm(Rv, _rot(torch.cumsum(dr, 0)).transpose(1, 2))
    tv0 = -_mv(Rv0, cv + torch.cumsum(dt, 0))
    Re0, te0 = _mm(_rot(g.n(0.01, 3, 3)), Re), te + g.n(0.02, 3, 3)
    P = _mv(Re[own], _mv(Rv[s], X) + tv[s]) + te[own]
    V = _mv(Re0[own].transpose(1, 2), P - te0[own])
    X0 = _mv(Rv0[s].transpose(1, 2), V - tv0[s]) + g.n(0.05, X.shape[0], 3)
    fixed = np.zeros(n, np.uint8)
    fixed[0] = 1
    a = lambda v: v.cpu().numpy()  # noqa: E731
    return SimpleNamespace(K=np.tile([F, F, CX, CY], (3, 1)), qv0=a(_quat(Rv0)), tv0=a(tv0), qe0=a(_quat(Re0)), te0=a(te0),
                           X0=a(X0), frame=a(f.int()), rcam=a(k.int()), obs_pt=a(pt.int()), obs_uv=a(uv), fixed_v=fixed,
                           fixed_e=np.zeros(3, np.uint8))


RIG_PRIORS = dict(prior_ext=100.0, prior_rig=100.0, rig_pairs=[[0, 1], [0, 2]])


def _graph(case, seed):
    """Two laps of a circle with a three-camera rig: sequential (k = 1, 2), loop-closure and
    extrinsic edges; the start integrates noisy odometry."""
    g = _Rng(seed)
    n = case["frames"]
    T = 2 * n
    h = 2 * math.pi * (torch.arange(T, device=g.d) % n).double() / n
    z, r = torch.zeros_like(h), n / (2 * math.pi)
    c = torch.stack([r * (1 - torch.cos(h)), z, r * torch.sin(h)], 1)
    c = c + (torch.arange(T, device=g.d) // n).double()[:, None] * torch.stack([torch.cos(h), z, -torch.sin(h)], 1)
    Rv = _look(torch.stack([torch.sin(h), z, torch.cos(h)], 1))
    tv = -_mv(Rv, c)

    def rel(Ra, ta, Rb, tb):
        A = _mm(Ra, Rb.transpose(-1, -2))
        return A, ta - _mv(A, tb)

    D, d = rel(Rv[1:], tv[1:], Rv[:-1], tv[:-1])
    E = _rot(g.n(1e-3, T - 1, 3))
    D, d = _mm(E, D).cpu().numpy(), (_mv(E, d) + g.n(1e-2, T - 1, 3)).cpu().numpy()
    R0, t0 = [Rv[0].cpu().numpy()], [tv[0].cpu().numpy()]
    for k in range(T - 1):
        R0.append(D[k] @ R0[-1])
        t0.append(D[k] @ t0[-1] + d[k])
    R0 = torch.from_numpy(np.stack(R0)).to(g.d)
    t0 = torch.from_numpy(np.stack(t0)).to(g.d)
    Re, te = _mounts(g.d)

    def nodes(Rw, tw):  # node f * 3 + camera
        return (_mm(Re[None], Rw[:, None]).reshape(-1, 3, 3), (_mv(Re[None], tw[:, None]) + te[None]).reshape(-1, 3))

    Rg, tg = nodes(Rv, tv)
    Ri, ti = nodes(R0, t0)
    f = torch.arange(T, device=g.d)
    edges = []
    for k in (1, 2):
        i = (f[:T - k, None] * 3 + torch.arange(3, device=g.d)).reshape(-1)
        j = i + 3 * k
        edges.append((i, j, *rel(Ri[i], ti[i], Ri[j], ti[j]), 100.0, 1.0))
    i = 3 * f[n::2]
    j = i - 3 * n
    A, a = rel(Rg[i], tg[i], Rg[j], tg[j])
    E = _rot(g.n(1e-3, i.shape[0], 3))
    edges.append((i, j, _mm(E, A), _mv(E, a) + g.n(2e-2, i.shape[0], 3), 100.0, 0.25))
    for k in (1, 2):
        i, j = 3 * f, 3 * f + k
        edges.append((i, j, *rel(Rg[i], tg[i], Rg[j], tg[j]), 1e4, 100.0))
    a = lambda v: v.cpu().numpy()  # noqa: E731
    fixed = np.zeros(3 * T, np.uint8)
    fixed[0] = 1
    w = [np.concatenate([np.full(e[0].shape[0], e[k]) for e in edges]) for k in (4, 5)]
    return SimpleNamespace(q0=a(_quat(Ri)), t0=a(ti), edge_i=a(torch.cat([e[0] for e in edges]).int()),
                           edge_j=a(torch.cat([e[1] for e in edges]).int()), meas_q=a(_quat(torch.cat([e[2] for e in edges]))),
                           meas_t=a(torch.cat([e[3] for e in edges])), w_rot=w[0], w_trans=w[1], fixed=fixed, edge_type=None)


def _requests(case, seed):
    """Localisation requests: 1 px noise, 10 % outliers, start off by 0.01 rad and 0.05 m."""
    g = _Rng(seed)
    n = case["n"]
    m = torch.exp(g.u(math.log(case["lo"]), math.log(case["hi"]), n)).long()
    r = torch.repeat_interleave(torch.arange(n, device=g.d), m)
    N = r.shape[0]
    R, c = _rot(g.n(0.5, n, 3)), g.n(10.0, n, 3)
    uv = torch.stack([g.u(0, W, N), g.u(0, H, N)], 1)
    P = torch.cat([(uv - torch.tensor([CX, CY], device=g.d)) / F, torch.ones(N, 1, device=g.d, dtype=torch.float64)], 1)
    X = _mv(R[r].transpose(1, 2), P * g.u(2, 30, N)[:, None]) + c[r]
    uv = uv + g.n(1.0, N, 2)
    bad = g.u(0, 1, N) < 0.1
    uv = torch.where(bad[:, None], torch.stack([g.u(0, W, N), g.u(0, H, N)], 1), uv)
    R0 = _mm(_rot(0.01 * g.unit(n)), R)
    t0 = -_mv(R, c) + 0.05 * g.unit(n)
    q, t, X, uv = (v.cpu().numpy() for v in (_quat(R0), t0, X, uv))
    at = np.concatenate([[0], np.cumsum(m.cpu().numpy())])
    K = np.array([F, F, CX, CY])
    return [SimpleNamespace(K=K, q0=q[i], t0=t[i], X=X[at[i]:at[i + 1]], uv=uv[at[i]:at[i + 1]]) for i in range(n)]


def _serve_cases(case):
    """The sizes of a stream: log-uniform up to the case's, the first request the largest."""
    r = np.random.default_rng(case["n"])
    nc = np.exp(r.uniform(math.log(5), math.log(case["cams"]), case["n"])).astype(int)
    npt = np.exp(r.uniform(math.log(1000), math.log(case["pts"]), case["n"])).astype(int)
    nc[0], npt[0] = case["cams"], case["pts"]
    return [dict(kind="arc", cams=int(a), pts=int(b)) for a, b in zip(nc, npt)]


# ------------------------------------------------------------------------------ prepare, run

_SCENES = dict(drive=_drive, loop=_loop, arc=_arc)


def _lm_opts(case):
    return dict(max_iters=case["iters"], pcg_max_iters=case["pcg"], pcg_rel_tol=case["tol"], precision=case["prec"])


def prepare(case, seed):
    kind = case["kind"]
    flags = ba.FLAG_PCG_RESIDENT if case.get("resident") else 0
    if kind in _SCENES:
        p = ba.Problem.from_scene(_SCENES[kind](case, seed), flags=flags, prior_seq=case.get("seq", 0.0), **_lm_opts(case))
        return dict(case=case, problem=p)
    if kind == "rig":
        return dict(case=case, problem=ba.Problem.from_rig(_rig(case, seed), **RIG_PRIORS, **_lm_opts(case)))
    if kind == "graph":
        p = ba.Problem.from_pose_graph(_graph(case, seed), prior_abs=case["prior"], flags=flags, **_lm_opts(case))
        return dict(case=case, problem=p)
    if kind == "serve":
        descs = [ba.scene_desc(_arc(c, seed * 1000 + i)) for i, c in enumerate(_serve_cases(case))]
        return dict(case=case, descs=descs, opts=ba.options(**_lm_opts(case)),
                    server=ba.Server(8 << 30, 16, case["prec"]))
    if kind == "pose":
        return dict(case=case, requests=_requests(case, seed))
    s = _drive(dict(case, fixed=1, huber=0.0, obs=6 * case["pts"]), seed)
    return dict(case=case, desc=ba.scene_desc(s))


def _kept(case, **arrays):
    """Results in the type of the precision mode."""
    t = np.float64 if case["prec"] == "f64" else np.float32
    return {k: np.asarray(v).astype(t, copy=False) for k, v in arrays.items()}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "rig":
        r = state["problem"].reset().solve().rig_result()
        return dict(_kept(case, q=r["q"], t=r["t"], X=r["X"], qe=r["qe"], te=r["te"], cost=r["iter_cost"]),
                    accepted=r["accepted"])
    if kind in _SCENES or kind == "graph":
        r = state["problem"].reset().solve().result()
        out = dict(_kept(case, q=r["q"], t=r["t"], cost=r["iter_cost"]), accepted=r["accepted"])
        return out if kind == "graph" else dict(out, **_kept(case, X=r["X"]), n_masked=r["n_masked"])
    if kind == "serve":
        sv = state["server"]
        tickets = [sv.submit(d, state["opts"]) for d in state["descs"]]
        rs = [sv.wait(t) for t in tickets]
        return dict(_kept(case, **{k: np.concatenate([r[k] for r in rs]) for k in ("q", "t", "X")},
                          cost=np.concatenate([r["iter_cost"] for r in rs])), accepted=[r["accepted"] for r in rs])
    if kind == "pose":
        r = ba.pose_batch(state["requests"], iters=case["iters"], huber_delta=1.0)
        return dict(_kept(dict(prec="f32"), q=r["q"], t=r["t"], cost=r["cost"]), status=r["status"])
    X, ok, inl, _ = ba.triangulate_ransac(state["desc"], tau_px=3.0, n_hyp=case["n_hyp"], method=case["method"])
    return dict(X=np.where(ok[:, None], X, 0.0), ok=ok, inliers=inl)


# ------------------------------------------------------------------------------ exact

def _gpu(v, t=torch.float64):
    return torch.from_numpy(np.ascontiguousarray(v)).to(_dev(), t)


def _add(n, idx, v):
    """Rows of v summed by index, spread over several copies of a short result."""
    k = min(max(1, 262144 // n), 1024)
    at = idx * k + torch.arange(idx.shape[0], device=idx.device) % k
    return torch.zeros((n * k, *v.shape[1:]), dtype=v.dtype, device=v.device).index_add_(0, at, v).unflatten(0, (n, k)).sum(1)


def _rows(R, t):
    """d [R | t] / d xi of a left increment, 12 x 6 (R row-major, then t)."""
    n = R.shape[0]
    J = torch.zeros(n, 12, 6, dtype=R.dtype, device=R.device)
    for m in range(3):
        e = torch.zeros(3, dtype=R.dtype, device=R.device)
        e[m] = 1.0
        J[:, :9, 3 + m] = _mm(_hat(e).expand(n, 3, 3), R).reshape(n, 9)
        J[:, 9 + m, m] = 1.0
    J[:, 9:, 3:] = -_hat(t)
    return J


def _rows_j(A):
    """d A / d xi_j of A = T_i T_j^-1."""
    n = A.shape[0]
    J = torch.zeros(n, 12, 6, dtype=A.dtype, device=A.device)
    for m in range(3):
        e = torch.zeros(3, dtype=A.dtype, device=A.device)
        e[m] = 1.0
        J[:, :9, 3 + m] = -_mm(A, _hat(e).expand(n, 3, 3)).reshape(n, 9)
    J[:, 9:, :3] = -A
    return J


def _twelve(R, t):
    return torch.cat([R.reshape(-1, 9), t], 1)


def _inv(A):
    return torch.linalg.inv(A)


class _Model:
    """Poses G (n blocks), points X, observations and relative / absolute pose terms.  For a
    rig the blocks are the vehicle poses, then the extrinsics, and an observation moves two."""

    def __init__(s, q, t, fixed, X=None, blocks=None, pt=None, uv=None, delta=0.0, edges=None, absolute=None):
        s.R, s.t = _matrix(_gpu(q)), _gpu(t)
        s.free = torch.from_numpy(np.asarray(fixed) == 0).to(_dev())
        s.X = None if X is None else X if isinstance(X, torch.Tensor) else _gpu(X)
        s.blocks, s.delta = blocks, delta
        if X is not None:
            s.pt, s.uv = _gpu(pt, torch.int64), _gpu(uv)
        s.edges, s.absolute = edges, absolute

    def _camera(s, R, t):
        if len(s.blocks) == 1:
            return R[s.blocks[0]], t[s.blocks[0]]
        v, e = s.blocks
        return _mm(R[e], R[v]), _mv(R[e], t[v]) + t[e]

    def _terms(s, R, t):
        """(blocks, 12-row residual, weights, Jacobians) of the pose terms."""
        out = []
        if s.edges is not None:
            i, j, M, w = s.edges
            A = _mm(R[i], R[j].transpose(1, 2))
            a = t[i] - _mv(A, t[j])
            out.append(((i, j), _twelve(A, a) - M, w, (_rows(A, a), _rows_j(A))))
        if s.absolute is not None:
            i, M, w = s.absolute
            out.append(((i,), _twelve(R[i], t[i]) - M, w, (_rows(R[i], t[i]),)))
        return out

    def cost(s, R, t, X):
        c, masked = torch.zeros((), dtype=torch.float64, device=R.device), 0
        for _, r, w, _ in s._terms(R, t):
            c = c + 0.5 * (w * r * r).sum()
        if X is not None:
            Rc, tc = s._camera(R, t)
            P = _mv(Rc, X[s.pt]) + tc
            on = P[:, 2] > 1e-6
            z = torch.where(on, P[:, 2], 1.0)
            r = torch.stack([F * P[:, 0] / z + CX, F * P[:, 1] / z + CY], 1) - s.uv
            q = (r * r).sum(1)
            if s.delta > 0:
                q = torch.where(q <= s.delta ** 2, q, 2 * s.delta * q.sqrt() - s.delta ** 2)
            c, masked = c + 0.5 * q[on].sum(), int((~on).sum())
        return float(c), masked

    def linearise(s):
        n = s.R.shape[0]
        s.g = torch.zeros(n, 6, dtype=torch.float64, device=s.R.device)
        s.U = torch.zeros(n, 6, 6, dtype=torch.float64, device=s.R.device)
        s.terms = s._terms(s.R, s.t)
        for b, r, w, J in s.terms:
            for i, Ji in zip(b, J):
                s.g += _add(n, i, ((w * r)[:, :, None] * Ji).sum(1))
                s.U += _add(n, i, _mm((w[:, :, None] * Ji).transpose(1, 2), Ji))
        if s.X is None:
            return
        Rc, tc = s._camera(s.R, s.t)
        P = _mv(Rc, s.X[s.pt]) + tc
        on = (P[:, 2] > 1e-6).double()[:, None]
        z = torch.where(P[:, 2] > 1e-6, P[:, 2], 1.0)
        o = torch.zeros_like(z)
        r = (torch.stack([F * P[:, 0] / z + CX, F * P[:, 1] / z + CY], 1) - s.uv) * on
        q = (r * r).sum(1)
        w = torch.ones_like(q) if s.delta <= 0 else torch.where(q <= s.delta ** 2, 1.0, s.delta / q.clamp(min=1e-300).sqrt())
        sw = w.sqrt()[:, None] * on
        Jpi = torch.stack([F / z, o, -F * P[:, 0] / z ** 2, o, F / z, -F * P[:, 1] / z ** 2], 1).reshape(-1, 2, 3)
        Jpi = Jpi * sw[:, :, None]
        Jc = torch.cat([Jpi, -_mm(Jpi, _hat(P))], 2)
        s.Jp = _mm(Jpi, Rc)
        s.r = r * sw
        s.J = [Jc]
        if len(s.blocks) == 2:
            Re, te = s.R[s.blocks[1]], s.t[s.blocks[1]]
            Ad = torch.cat([torch.cat([Re, _mm(_hat(te), Re)], 2), torch.cat([torch.zeros_like(Re), Re], 2)], 1)
            s.J = [_mm(Jc, Ad), Jc]
        p = s.X.shape[0]
        s.V = _add(p, s.pt, _mm(s.Jp.transpose(1, 2), s.Jp))
        s.gp = _add(p, s.pt, (s.Jp * s.r[:, :, None]).sum(1))
        for b, J in zip(s.blocks, s.J):
            s.U += _add(n, b, _mm(J.transpose(1, 2), J))
            s.g += _add(n, b, (J * s.r[:, :, None]).sum(1))

    def damp(s, lam):
        n = s.R.shape[0]
        s.D = torch.diagonal(s.U, dim1=1, dim2=2).clamp(1e-6, 1e32)
        B = s.U + lam * torch.diag_embed(s.D)
        s.b = -s.g
        if s.X is not None:
            p = s.X.shape[0]
            s.Dp = torch.diagonal(s.V, dim1=1, dim2=2).clamp(1e-6, 1e32)
            s.Vi = _inv(s.V + lam * torch.diag_embed(s.Dp))
            y = _mv(s.Vi, s.gp)
            for b, J in zip(s.blocks, s.J):
                W = _mm(J.transpose(1, 2), s.Jp)
                s.b = s.b + _add(n, b, _mv(W, y[s.pt]))
                pt = s.pt
                if len(s.blocks) == 2:  # a block may see a point through several cameras
                    key, idx = torch.unique(b * p + s.pt, return_inverse=True)
                    W, b, pt = _add(key.shape[0], idx, W), key // p, key % p
                B = B - _add(n, b, _mm(_mm(W, s.Vi[pt]), W.transpose(1, 2)))
        s.M = _inv(B)
        s.lam = lam
        s.b = torch.where(s.free[:, None], s.b, 0.0)

    def product(s, x):
        n = x.shape[0]
        y = s.lam * s.D * x
        for b, _, w, J in s.terms:
            e = w * sum(_mv(Ji, x[i]) for i, Ji in zip(b, J))
            for i, Ji in zip(b, J):
                y = y + _add(n, i, (Ji * e[:, :, None]).sum(1))
        if s.X is not None:
            e = sum(_mv(J, x[b]) for b, J in zip(s.blocks, s.J))
            k = _mv(s.Vi, _add(s.X.shape[0], s.pt, (s.Jp * e[:, :, None]).sum(1)))
            e = e - _mv(s.Jp, k[s.pt])
            for b, J in zip(s.blocks, s.J):
                y = y + _add(n, b, (J * e[:, :, None]).sum(1))
        return torch.where(s.free[:, None], y, 0.0)

    def pcg(s, cap, tol):
        x, r = torch.zeros_like(s.b), s.b.clone()
        z = _mv(s.M, r)
        p, rz, stop = z.clone(), (r * z).sum(), tol * r.norm()
        for it in range(cap):
            if it and r.norm() <= stop:
                break
            q = s.product(p)
            pq = (p * q).sum()
            if not pq > 0:
                break
            a = rz / pq
            x, r = x + a * p, r - a * q
            z = torch.where(s.free[:, None], _mv(s.M, r), 0.0)
            rz, old = (r * z).sum(), rz
            p = z + rz / old * p
        return x

    def solve(s, iters, cap, tol):
        """Levenberg-Marquardt with the Nielsen schedule; a step that masks more is refused."""
        c, masked = s.cost(s.R, s.t, s.X)
        lam, nu, costs, accepted = 1e-4, 2.0, [c], 0
        for _ in range(iters):
            s.linearise()
            s.damp(lam)
            x = s.pcg(cap, tol)
            dR, dt = _se3(x)
            R, t = _mm(dR, s.R), _mv(dR, s.t) + dt
            dL = 0.5 * (x * (lam * s.D * x - torch.where(s.free[:, None], s.g, 0.0))).sum()
            X = None
            if s.X is not None:
                e = sum(_mv(J, x[b]) for b, J in zip(s.blocks, s.J))
                dp = _mv(s.Vi, -s.gp - _add(s.X.shape[0], s.pt, (s.Jp * e[:, :, None]).sum(1)))
                X = s.X + dp
                dL = dL + 0.5 * (dp * (lam * s.Dp * dp - s.gp)).sum()
            c1, m1 = s.cost(R, t, X)
            rho = (c - c1) / float(dL) if float(dL) > 0 else -1.0
            if rho > 1e-3 and m1 <= masked:
                s.R, s.t, s.X, c, masked = R, t, X, c1, m1
                lam, nu, accepted = lam * max(1 / 3, 1 - (2 * rho - 1) ** 3), 2.0, accepted + 1
            else:
                lam, nu = lam * nu, nu * 2
            lam = min(max(lam, 1e-12), 1e16)
            costs.append(c)
        return np.array(costs)


def _out(**v):
    return {k: a.cpu().numpy() if isinstance(a, torch.Tensor) else a for k, a in v.items()}


def _exact_ba(case, sc):
    edges = None
    if case.get("seq"):
        R, t = _matrix(_gpu(sc.q0)), _gpu(sc.t0)
        i = torch.arange(R.shape[0] - 1, device=_dev())
        A = _mm(R[i], R[i + 1].transpose(1, 2))
        w = torch.full((i.shape[0], 12), case["seq"], dtype=torch.float64, device=_dev())
        edges = (i, i + 1, _twelve(A, t[i] - _mv(A, t[i + 1])), w)
    m = _Model(sc.q0, sc.t0, sc.cam_fixed, sc.X0, [_gpu(sc.obs_cam, torch.int64)], sc.obs_pt, sc.obs_uv, sc.huber_delta,
               edges)
    cost = m.solve(case["iters"], case["pcg"], case["tol"])
    return _out(q=_quat(m.R), t=m.t, X=m.X, cost=cost)


def _exact_rig(case, sc):
    n = sc.qv0.shape[0]
    q, t = np.concatenate([sc.qv0, sc.qe0]), np.concatenate([sc.tv0, sc.te0])
    R, T = _matrix(_gpu(q)), _gpu(t)
    i, j = (torch.tensor([n + p[k] for p in RIG_PRIORS["rig_pairs"]], device=_dev()) for k in (0, 1))
    A = _mm(R[i], R[j].transpose(1, 2))
    full = lambda k, v: torch.full((k, 12), v, dtype=torch.float64, device=_dev())  # noqa: E731
    edges = (i, j, _twelve(A, T[i] - _mv(A, T[j])), full(2, RIG_PRIORS["prior_rig"]))
    e = torch.arange(n, n + 3, device=_dev())
    m = _Model(q, t, np.concatenate([sc.fixed_v, sc.fixed_e]), sc.X0,
               [_gpu(sc.frame, torch.int64), n + _gpu(sc.rcam, torch.int64)], sc.obs_pt, sc.obs_uv, 0.0, edges,
               (e, _twelve(R[e], T[e]), full(3, RIG_PRIORS["prior_ext"])))
    cost = m.solve(case["iters"], case["pcg"], case["tol"])
    q = _quat(m.R)
    return _out(q=q[:n], t=m.t[:n], X=m.X, qe=q[n:], te=m.t[n:], cost=cost)


def _exact_graph(case, g):
    w = np.concatenate([np.repeat(g.w_rot[:, None], 9, 1), np.repeat(g.w_trans[:, None], 3, 1)], 1)
    i, j = _gpu(g.edge_i, torch.int64), _gpu(g.edge_j, torch.int64)
    R, t = _matrix(_gpu(g.q0)), _gpu(g.t0)
    n = torch.arange(R.shape[0], device=_dev())
    prior = torch.full((R.shape[0], 12), case["prior"], dtype=torch.float64, device=_dev())
    m = _Model(g.q0, g.t0, g.fixed, edges=(i, j, _twelve(_matrix(_gpu(g.meas_q)), _gpu(g.meas_t)), _gpu(w)),
               absolute=(n, _twelve(R, t), prior))
    cost = m.solve(case["iters"], case["pcg"], case["tol"])
    return _out(q=_quat(m.R), t=m.t, cost=cost)


def _exact_pose(case, reqs):
    """Gauss-Newton on every request, Huber 1 px."""
    n = len(reqs)
    r = _gpu(np.repeat(np.arange(n), [q.X.shape[0] for q in reqs]), torch.int64)
    X, uv = _gpu(np.concatenate([q.X for q in reqs])), _gpu(np.concatenate([q.uv for q in reqs]))
    m = _Model(np.stack([q.q0 for q in reqs]), np.stack([q.t0 for q in reqs]), np.zeros(n), X, [r],
               np.arange(r.shape[0]), np.zeros((r.shape[0], 2)), 1.0)
    m.uv = uv
    for _ in range(case["iters"]):
        m.linearise()
        dR, dt = _se3(-_mv(_inv(m.U), m.g))
        m.R, m.t = _mm(dR, m.R), _mv(dR, m.t) + dt
    P = _mv(m.R[r], X) + m.t[r]
    q = ((torch.stack([F * P[:, 0] / P[:, 2] + CX, F * P[:, 1] / P[:, 2] + CY], 1) - uv) ** 2).sum(1)
    q = torch.where(P[:, 2] > 1e-6, torch.where(q <= 1, q, 2 * q.sqrt() - 1), 0.0)
    return _out(q=_quat(m.R), t=m.t, cost=0.5 * _add(n, r, q))


def _exact_tri(case, sc):
    """RANSAC per track over the fixed schedule of observation pairs, two-ray midpoints, then
    the midpoint or the homogeneous solution of the inliers."""
    R, t = _matrix(_gpu(sc.q0)), _gpu(sc.t0)
    pt = _gpu(sc.obs_pt, torch.int64)
    o = torch.argsort(pt, stable=True)  # a track's observations in the caller's order
    cam, uv, pt = _gpu(sc.obs_cam, torch.int64)[o], _gpu(sc.obs_uv)[o], pt[o]
    p = sc.X0.shape[0]
    n = torch.bincount(pt, minlength=p)
    at = torch.cumsum(n, 0) - n
    d = torch.cat([(uv - torch.tensor([CX, CY], device=uv.device)) / F, torch.ones_like(uv[:, :1])], 1)
    d = _mv(R[cam].transpose(1, 2), d)
    d = d / d.norm(dim=1, keepdim=True)
    c = -_mv(R[cam].transpose(1, 2), t[cam])
    I = torch.eye(3, dtype=torch.float64, device=uv.device)
    A = I - d[:, :, None] * d[:, None, :]
    b = _mv(A, c)

    def solve3(M, v):
        """M^-1 v by the adjugate, and whether the determinant is over 1e-12."""
        r0, r1, r2 = M[:, 0], M[:, 1], M[:, 2]
        cr = torch.stack([torch.linalg.cross(r1, r2), torch.linalg.cross(r2, r0), torch.linalg.cross(r0, r1)], 2)
        det = (r0 * cr[:, :, 0]).sum(1)
        ok = det > 1e-12
        return _mv(cr, v) / torch.where(ok, det, 1.0)[:, None], ok

    def inliers(X):
        P = _mv(R[cam], X[pt]) + t[cam]
        e = torch.stack([F * P[:, 0] / P[:, 2] + CX, F * P[:, 1] / P[:, 2] + CY], 1) - uv
        return (P[:, 2] > 1e-6) & ((e * e).sum(1) <= 9.0)

    best = torch.zeros(p, dtype=torch.int64, device=uv.device)
    keep = torch.zeros(pt.shape[0], dtype=torch.bool, device=uv.device)
    m = n.clamp(min=2)
    for h in range(case["n_hyp"]):
        i = h % m
        j = (i + 1 + (h // m) % (m - 1)) % m
        i, j = (at + torch.minimum(i, n - 1)).clamp(min=0), (at + torch.minimum(j, n - 1)).clamp(min=0)
        X, ok = solve3(A[i] + A[j], b[i] + b[j])
        for k in (i, j):  # the point lies in front of both cameras of the pair
            ok = ok & ((R[cam[k], 2] * X).sum(1) + t[cam[k], 2] > 1e-6)
        ok = ok & (n >= 2)
        inl = inliers(X) & ok[pt]
        cnt = _add(p, pt, inl.long())
        better = cnt > best
        best = torch.where(better, cnt, best)
        keep = torch.where(better[pt], inl, keep)
    k = keep.double()[:, None, None]
    if case["method"] == "midpoint":
        X, ok = solve3(_add(p, pt, A * k), _add(p, pt, b * k[:, :, 0]))
    else:
        P = torch.cat([R[cam], t[cam][:, :, None]], 2)
        x = (uv - torch.tensor([CX, CY], device=uv.device)) / F
        rows = x[:, :, None] * P[:, 2:3] - P[:, :2]
        _, V = torch.linalg.eigh(_add(p, pt, _mm(rows.transpose(1, 2), rows) * k))
        w = V[:, 3, 0]
        ok = w.abs() > 1e-12
        X = V[:, :3, 0] / torch.where(ok, w, 1.0)[:, None]
    z = (_mv(R[cam], X[pt]) + t[cam])[:, 2]
    behind = _add(p, pt, (keep & ~(z > 1e-6)).long())
    ok = ok & (best >= 2) & (behind == 0)
    return dict(X=torch.where(ok[:, None], X, 0.0).cpu().numpy(), ok=None, inliers=None)


def exact(case, seed):
    kind = case["kind"]
    if kind in _SCENES:
        return dict(_exact_ba(case, _SCENES[kind](case, seed)), accepted=None, n_masked=None)
    if kind == "rig":
        return dict(_exact_rig(case, _rig(case, seed)), accepted=None)
    if kind == "graph":
        return dict(_exact_graph(case, _graph(case, seed)), accepted=None)
    if kind == "serve":
        rs = [_exact_ba(case, _arc(c, seed * 1000 + i)) for i, c in enumerate(_serve_cases(case))]
        return dict({k: np.concatenate([r[k] for r in rs]) for k in ("q", "t", "X", "cost")}, accepted=None)
    if kind == "pose":
        return dict(_exact_pose(case, _requests(case, seed)), status=None)
    return _exact_tri(case, _drive(dict(case, fixed=1, huber=0.0, obs=6 * case["pts"]), seed))


# ------------------------------------------------------------------------------ work

def _ba_work(obs, pts, pairs, blocks, iters, pcg, word):
    """Per LM iteration: every observation (indices and pixel) once to linearise and once at
    the trial state, every point read and written, the upper triangle of S written once and
    read once per PCG iteration; the products of the observation pairs (6 x 3 by 3 x 6), 300
    operations per observation of linearisation and trial, the products with S."""
    b = 2 * obs * (8 + 2 * word) + pts * 72 + blocks * 36 * word * (1 + pcg)
    f = 300 * obs + pairs * 216 + pcg * blocks * 144
    return dict(bytes=float(b * iters), flops=float(f * iters))


def work(case):
    kind = case["kind"]
    word = 8 if case.get("prec") == "f64" else 4
    if kind == "drive":  # 9 views a point (58 pairs), a band of about 55 upper columns
        n, p = case["cams"], case["pts"]
        return _ba_work(9.1 * p, p, 58 * p, n * min(55, n / 2), case["iters"], 40, word)
    if kind == "loop":
        p = case["pts"]
        return _ba_work(8.6 * p, p, 54 * p, case["cams"] * 74, case["iters"], 17, word)
    if kind == "arc":
        n, p = case["cams"], case["pts"]
        return _ba_work(0.98 * n * p, p, 0.48 * n * n * p, n * n / 2, case["iters"], 20, word)
    if kind == "serve":
        n, p = case["cams"] / 2.5, case["pts"] / 2.5
        one = _ba_work(0.98 * n * p, p, 0.48 * n * n * p, n * n / 2, case["iters"], 20, word)
        return {k: v * case["n"] for k, v in one.items()}
    if kind == "rig":
        p, n = case["pts"], case["frames"]
        return _ba_work(12.0 * p, p, 90 * p, n * 30, case["iters"], 60, word)
    if kind == "graph":  # 9000 nodes, 24741 edges at 1500 frames
        n = 6 * case["frames"]
        blocks = 3.75 * n
        return dict(bytes=float(case["iters"] * (2.75 * n * 240 + n * 192 + blocks * 36 * word * 51)),
                    flops=float(case["iters"] * (2.75 * n * 4000 + 50 * blocks * 144)))
    if kind == "pose":
        corr = case["n"] * (case["hi"] + case["lo"]) / 2
        return dict(bytes=corr * 40.0 + case["n"] * 160.0, flops=corr * 120.0 * case["iters"])
    obs = 6 * case["pts"]
    return dict(bytes=obs * 25.0 + case["pts"] * 25.0 + case["cams"] * 88.0,
                flops=float(case["n_hyp"]) * (obs * 35.0 + case["pts"] * 150.0))
