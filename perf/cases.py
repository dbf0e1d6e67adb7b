"""The work that programs have this library do, as cases to time and compare.

Each case is one call (or one forward and backward) of the public entry points
at one size. `listed` holds the sizes that are followed over time, `draw`
gives others of the same ranges, `prepare` makes a case's inputs on the GPU
from a seed, `run` is the pass itself, `work` the bytes and operations it
cannot do without, and `exact` its result in plain 64-bit torch.

Inputs follow the shapes and distributions of the library's own workloads:
frames with a 518-pixel long side unprojected from smooth depth maps, 1 cm
target noise, 10 % outliers, log-normal confidences (about 88 % of a frame
passes the threshold), random-walk pose graphs with loop closures.
"""

import math
import random

import numpy as np
import torch

import paper_2510_02080_amd as s3a

DEV = "cuda:0"
F8 = torch.float64
DELTA = 0.05  # Huber threshold in metres


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest registration: one pair of thumbnail pointmaps (64 x 48); latency and launches
        dict(name="align_1x3072", kind="align", pairs=1, lo=3072, hi=3072, dtype="f32", iters=10, holes=False),
        # one shared keyframe of two submaps, the call a mapping back end makes for each new submap
        dict(name="align_1x203056", kind="align", pairs=1, lo=203056, hi=203056, dtype="f32", iters=10, holes=False),
        # a new submap against the dozen it overlaps: ragged counts, some pixels without a depth (NaN)
        dict(name="align_12_ragged", kind="align", pairs=12, lo=20000, hi=400000, dtype="f32", iters=10, holes=True),
        # offline or serving: many pairs in one call, the largest batch
        dict(name="align_256_f32", kind="align", pairs=256, lo=20000, hi=400000, dtype="f32", iters=10, holes=False),
        # the same from bf16 storage
        dict(name="align_256_bf16", kind="align", pairs=256, lo=20000, hi=400000, dtype="bf16", iters=10, holes=False),
        # submaps kept as depth maps and cameras: a few pairs of a running session
        dict(name="depth_4", kind="depth", pairs=4, width=518, height=392, frames=2, dtype="f32", iters=10),
        # and a large batch of them
        dict(name="depth_256", kind="depth", pairs=256, width=518, height=392, frames=2, dtype="f32", iters=10),
        # a training step through the alignment cost: forward, then every gradient
        dict(name="cost_grad_64x203056", kind="cost_grad", pairs=64, lo=203056, hi=203056, dtype="f32", holes=False),
        # a training step through the solved poses (implicit derivative)
        dict(name="solve_grad_64x203056", kind="solve_grad", pairs=64, lo=203056, hi=203056, iters=10, holes=False),
        # after a pose-graph solve: every submap's points to the world frame, the sparse map's points replaced
        dict(name="points_200x160000", kind="points", submaps=200, rows=32000000, corr=1000000, dtype="f32"),
        # the pose graph of one room-size sequence, Levenberg-Marquardt
        dict(name="pgo_52", kind="pgo", nodes=52, loops=10, lm=True, iters=20),
        # the pose graph of a long session with many loop closures, Gauss-Newton
        dict(name="pgo_1000", kind="pgo", nodes=1000, loops=200, lm=False, iters=20),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["align", "align", "align", "depth", "cost_grad", "solve_grad", "points", "pgo"])
    if kind in ("align", "cost_grad", "solve_grad"):
        most = 32000000 if kind == "align" else 12000000
        pairs = _log(rng, 1, 256 if kind == "align" else 64)
        hi = min(_log(rng, 3000, 400000), most // pairs)
        c = dict(kind=kind, pairs=pairs, lo=max(1000, int(hi * rng.choice([1.0, 0.5, 0.05]))), hi=hi, holes=rng.random() < 0.25)
        if kind != "solve_grad":
            c["dtype"] = rng.choice(["f32", "f32", "bf16"])
        if kind != "cost_grad":
            c["iters"] = rng.choice([3, 5, 10])
        return c
    if kind == "depth":
        return dict(kind=kind, pairs=_log(rng, 1, 200), width=rng.randint(160, 518), height=rng.randint(120, 392),
                    frames=rng.randint(1, 3), dtype=rng.choice(["f32", "f32", "bf16"]), iters=rng.choice([5, 10]))
    if kind == "points":
        rows = _log(rng, 20000, 30000000)
        return dict(kind=kind, submaps=min(_log(rng, 1, 400), rows // 100), rows=rows, corr=_log(rng, 100, max(200, rows // 30)),
                    dtype=rng.choice(["f32", "f32", "bf16"]))
    nodes = _log(rng, 8, 1000)
    return dict(kind=kind, nodes=nodes, loops=max(1, int(nodes * rng.uniform(0.02, 0.2))), lm=rng.random() < 0.4, iters=rng.choice([10, 20]))


def _counts(case):
    """Points per pair: log-uniform in [lo, hi], the same for every seed."""
    rng = random.Random(case["pairs"] * 1000003 + case["hi"])
    return [case["hi"] if case["lo"] >= case["hi"] else _log(rng, case["lo"], case["hi"]) for _ in range(case["pairs"])]


def _tau(case):
    return 0.0 if case["hi"] <= 3072 else 1.5


def _frames(case):
    """Shared frames per depth pair: mostly one."""
    rng = random.Random(case["pairs"] * 7919 + case["width"])
    return [1 if rng.random() < 0.7 else rng.randint(1, case["frames"]) for _ in range(case["pairs"])]


# ---------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _rotation(r, most):
    ax = r.normal(size=3)
    ax /= np.linalg.norm(ax)
    th = np.deg2rad(r.uniform(0.0, most))
    K = np.array([[0, -ax[2], ax[1]], [ax[2], 0, -ax[0]], [-ax[1], ax[0], 0]])
    return np.eye(3) + np.sin(th) * K + (1 - np.cos(th)) * K @ K


def _similarity(r, most=30.0):
    return r.uniform(0.5, 2.0), _rotation(r, most), r.normal(size=3)


def _surface(r, h, w):
    """A smooth depth map in [1, 10] m, (h * w,) float32."""
    v = torch.arange(h, device=DEV, dtype=torch.float32).view(h, 1) / h
    u = torch.arange(w, device=DEV, dtype=torch.float32).view(1, w) / w
    z = torch.zeros(h, w, device=DEV)
    for _ in range(8):
        a, f, th, ph = r.uniform(0.2, 1.0), 2 * np.pi * r.uniform(0.5, 4.0), r.uniform(0, 2 * np.pi), r.uniform(0, 2 * np.pi)
        z += a * torch.sin((f * np.cos(th)) * u + (f * np.sin(th)) * v + ph)
    z -= z.min()
    return (1.0 + 9.0 * z / z.max()).reshape(-1)


def _pair(r, g, n):
    """One pair's planes (7, n) float32: a frame of about n pixels and its image under a similarity."""
    w = min(518, max(32, int(math.sqrt(n * 518 / 392))))
    h = -(-n // w)
    z = _surface(r, h, w)[:n]
    i = torch.arange(n, device=DEV)
    p = torch.stack([z * ((i % w).float() - (w - 1) / 2) / w, z * ((i // w).float() - (h - 1) / 2) / w, z])
    s, R, t = _similarity(r)
    M = torch.tensor(s * R, dtype=torch.float32, device=DEV)
    q = M @ p + torch.tensor(t, dtype=torch.float32, device=DEV).view(3, 1) + 0.01 * torch.randn(3, n, generator=g, device=DEV)
    out = torch.rand(n, generator=g, device=DEV) < 0.1
    q = torch.where(out, 10.0 * torch.rand(3, n, generator=g, device=DEV) - 5.0, q)
    c = torch.exp(1.0 + 0.5 * torch.randn(1, n, generator=g, device=DEV))
    return torch.cat([p, q, c]), (s, R, t)


def _planes(case, seed):
    """Seven plane tensors, the offsets, and the similarities the targets were made with."""
    counts = _counts(case)
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    r, g = np.random.default_rng(int(seed)), _gen(seed)
    N = int(off[-1])
    X = torch.empty(7, (N + 3) // 4 * 4, device=DEV)
    gt = []
    for k, n in enumerate(counts):
        x, T = _pair(r, g, n)
        X[:, off[k]:off[k + 1]] = x
        gt.append(T)
    if case["holes"]:  # pixels without a depth
        hole = torch.rand(N, generator=g, device=DEV) < 0.002
        X[:3, :N][:, hole] = float("nan")
    if case.get("dtype") == "bf16":
        return [X[j, :N].to(torch.bfloat16) for j in range(7)], torch.from_numpy(off).to(DEV), gt
    return [X[j, :N] for j in range(7)], torch.from_numpy(off).to(DEV), gt


def _sim3_rows(items):
    rows = np.zeros((len(items), 16))
    for k, (s, R, t) in enumerate(items):
        rows[k, :9], rows[k, 9:12], rows[k, 12] = np.asarray(R).ravel(), t, s
    return torch.from_numpy(rows).to(DEV)


def _pointmaps(planes, offsets, case):
    if case.get("dtype") == "bf16":
        return s3a.Pointmaps([p.view(torch.int16) for p in planes], offsets, s3a.BF16, covers_all=True)
    return s3a.Pointmaps(planes, offsets, s3a.F32, covers_all=True)


def _near(gt, r):
    """Poses near the true ones: where a training step stands."""
    return [(s * math.exp(0.01 * r.normal()), _rotation(r, 0.5) @ R, t + 0.01 * r.normal(size=3)) for s, R, t in gt]


CAM = np.dtype([("fx", "<f4"), ("fy", "<f4"), ("cx", "<f4"), ("cy", "<f4"), ("R", "<f4", 9), ("t", "<f4", 3)])
DEPTH_PAIR = np.dtype([("width", "<i4"), ("frame_pixels", "<i4"), ("n_frames", "<i4"), ("reserved", "<i4"), ("p", CAM, 4), ("q", CAM, 4)])


def _depth_inputs(case, seed):
    w, h, frames = case["width"], case["height"], _frames(case)
    r, g = np.random.default_rng(int(seed)), _gen(seed)
    off = np.concatenate([[0], np.cumsum([f * w * h for f in frames])]).astype(np.int64)
    N = int(off[-1])
    rec = np.zeros(len(frames), dtype=DEPTH_PAIR)
    dp, dq = torch.empty(N, device=DEV), torch.empty(N, device=DEV)
    at = 0
    for k, nf in enumerate(frames):
        rec[k]["width"], rec[k]["frame_pixels"], rec[k]["n_frames"] = w, w * h, nf
        (sj, Rj, tj), (si, Ri, ti) = _similarity(r), _similarity(r)
        for f in range(nf):
            Rf, tf = _rotation(r, 10.0), r.normal(0, 0.3, 3)
            for side, (s, R, t) in (("p", (sj, Rj, tj)), ("q", (si, Ri, ti))):
                cam = rec[k][side][f]
                cam["fx"] = cam["fy"] = w
                cam["cx"], cam["cy"] = w / 2.0, h / 2.0
                cam["R"], cam["t"] = (R @ Rf).ravel(), s * R @ tf + t
            d = _surface(r, h, w)
            dp[at:at + w * h], dq[at:at + w * h] = sj * d, si * d
            at += w * h
        a, b = int(off[k]), int(off[k + 1])
        out = torch.rand(b - a, generator=g, device=DEV) < 0.1
        dq[a:b] = torch.where(out, si * (1.0 + 9.0 * torch.rand(b - a, generator=g, device=DEV)),
                              dq[a:b] * (1.0 + 0.005 * torch.randn(b - a, generator=g, device=DEV)))
    c = torch.exp(1.0 + 0.5 * torch.randn(N, generator=g, device=DEV))
    planes = [dp, dq, c]
    if case["dtype"] == "bf16":
        planes = [x.to(torch.bfloat16) for x in planes]
    return planes, torch.from_numpy(off).to(DEV), rec


def _points_inputs(case, seed):
    r, g = np.random.default_rng(int(seed)), _gen(seed)
    N, n, m = case["rows"], case["submaps"], case["corr"]
    cut = np.sort(random.Random(N + n).sample(range(1, N), n - 1)) if n > 1 else []
    off = np.concatenate([[0], cut, [N]]).astype(np.int64)
    xyz = torch.empty(3, (N + 7) // 8 * 8, device=DEV).normal_(0.0, 3.0, generator=g)
    if case["dtype"] == "bf16":
        xyz = xyz.to(torch.bfloat16)
    T = _sim3_rows([_similarity(r) for _ in range(n)])
    src = torch.randperm(N, generator=g, device=DEV)[:m]
    dst = torch.randperm(2 * m, generator=g, device=DEV)[:m]
    sparse = torch.empty(3, (2 * m + 3) // 4 * 4, device=DEV).normal_(0.0, 3.0, generator=g)
    return xyz[:, :N], torch.from_numpy(off).to(DEV), T, src, dst, sparse[:, :2 * m]


def _pgo_inputs(case, seed):
    """A random-walk trajectory, sequential and loop edges, measurements with 1e-3 noise and their information."""
    n = case["nodes"]
    shape = random.Random(n * 31 + case["loops"])
    edges = [(k, k + 1) for k in range(n - 1)]
    gap = min(20, max(2, n // 3))
    seen = set()
    while len(seen) < case["loops"]:
        i, j = sorted(shape.sample(range(n), 2))
        if j - i >= gap:
            if (i, j) not in seen:
                edges.append((i, j))
            seen.add((i, j))
    edges = np.array(edges, dtype=np.int32)
    r = np.random.default_rng(int(seed))
    T = [np.eye(4)]
    for _ in range(n - 1):
        step = np.eye(4)
        yaw = np.deg2rad(r.uniform(-10.0, 10.0))
        step[:3, :3] = math.exp(r.normal(0.0, 0.01)) * np.array([[np.cos(yaw), -np.sin(yaw), 0], [np.sin(yaw), np.cos(yaw), 0], [0, 0, 1]])
        step[:3, 3] = r.normal(0.0, 0.3, 3)
        T.append(T[-1] @ step)
    meas, sd = [], np.array([1e-3] * 6 + [1e-4])
    for i, j in edges:
        x = r.normal(size=7) * sd
        D = np.eye(4)
        th = np.linalg.norm(x[3:6])
        K = np.array([[0, -x[5], x[4]], [x[5], 0, -x[3]], [-x[4], x[3], 0]]) / max(th, 1e-300)
        D[:3, :3] = math.exp(x[6]) * (np.eye(3) + np.sin(th) * K + (1 - np.cos(th)) * K @ K)
        D[:3, 3] = x[:3]
        Z = D @ np.linalg.inv(T[i]) @ T[j]
        s = np.cbrt(np.linalg.det(Z[:3, :3]))
        meas.append((s, Z[:3, :3] / s, Z[:3, 3]))
    B = np.eye(7) + 0.2 * r.normal(size=(len(edges), 7, 7))
    B /= sd
    omega = np.matmul(B.transpose(0, 2, 1), B)
    return edges, _sim3_rows(meas), torch.from_numpy(omega.reshape(-1, 49)).to(DEV)


HUBER_PG = 3.75  # on the whitened residual


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case, handle=s3a.handle(0))
    if kind in ("align", "cost_grad", "solve_grad"):
        planes, off, gt = _planes(case, seed)
        r = np.random.default_rng(int(seed) + 77)
        if kind == "align":
            st["pm"] = _pointmaps(planes, off, case)
        else:
            st["off"] = off
            st["gL"] = torch.from_numpy(r.uniform(0.5, 1.5, case["pairs"])).to(DEV)
            if kind == "cost_grad":
                st["S"] = _sim3_rows(_near(gt, r))
                xi = torch.from_numpy(0.005 * r.normal(size=(case["pairs"], 7))).to(DEV)
                st["xi"] = xi if case["dtype"] == "bf16" else xi.requires_grad_()
                st["pm"] = _pointmaps(planes, off, case)
            else:
                gS = r.normal(size=(case["pairs"], 16))
                gS[:, 13:] = 0.0
                st["gS"] = torch.from_numpy(gS).to(DEV)
            if case.get("dtype") != "bf16":
                st["planes"] = [p.detach().requires_grad_() for p in planes]
    elif kind == "depth":
        planes, off, rec = _depth_inputs(case, seed)
        table = torch.from_numpy(rec.view(np.uint8).copy()).to(DEV)
        bf = case["dtype"] == "bf16"
        st["dm"] = s3a.DepthPointmaps([p.view(torch.int16) for p in planes] if bf else planes, off, table, s3a.BF16 if bf else s3a.F32)
    elif kind == "points":
        st["xyz"], st["off"], st["T"], st["src"], st["dst"], st["sparse"] = _points_inputs(case, seed)
    else:
        st["edges"], st["meas"], st["omega"] = _pgo_inputs(case, seed)
    return st


# ---------------------------------------------------------------- one pass

def run(st):
    case, h = st["case"], st["handle"]
    kind = case["kind"]
    if kind == "align":
        return s3a.align_pairs(st["pm"], _tau(case), DELTA, case["iters"], info=False)[0]
    if kind == "depth":
        return h.align_depth_pairs(st["dm"], 1.5, DELTA, case["iters"], info=False)[0]
    if kind == "cost_grad":
        if case["dtype"] == "bf16":  # bf16 storage goes through the plain calls
            pm, S, xi = st["pm"], st["S"], st["xi"]
            L, C = s3a.align_cost(pm, S, xi, _tau(case), DELTA)
            gp, gq, gc, gxi = s3a.align_pairs_backward(pm, S, xi, L, C, st["gL"], _tau(case), DELTA)
            return L, gp, gq, gc, gxi
        L = s3a.align_cost_autograd(st["planes"], st["off"], st["S"], st["xi"], _tau(case), DELTA, h)
        return (L,) + torch.autograd.grad(L, st["planes"] + [st["xi"]], st["gL"])
    if kind == "solve_grad":
        S = s3a.align_solve(st["planes"], st["off"], _tau(case), DELTA, case["iters"], h)
        return (S,) + torch.autograd.grad(S, st["planes"], st["gS"])
    if kind == "points":
        world = h.transform_points(st["xyz"], st["off"], st["T"])
        return world, h.correct_points(world, st["src"], st["dst"], st["sparse"])
    T, rep = s3a.pose_graph_solve(st["edges"], st["meas"], omega=st["omega"], iters=case["iters"], huber_delta=HUBER_PG, lm=case["lm"])
    return T, rep.final_chi2


def work(case):
    """Inputs read once, outputs written once, and the arithmetic of every pass: about 60 operations a point (90 a
    pixel from depth, with both rays) for each Gauss-Newton pass, 40 for the closed form."""
    kind = case["kind"]
    b = 2 if case.get("dtype") == "bf16" else 4
    if kind in ("align", "solve_grad"):
        N = sum(_counts(case))
        k = case["iters"]
        if kind == "align":
            return {"bytes": 7 * b * N + 128 * case["pairs"], "flops": N * (60 * k + 40)}
        return {"bytes": 56 * N + 256 * case["pairs"], "flops": N * (60 * k + 40 + 300)}
    if kind == "depth":
        N = sum(_frames(case)) * case["width"] * case["height"]
        return {"bytes": 3 * b * N + (528 + 128) * case["pairs"], "flops": N * (90 * case["iters"] + 70)}
    if kind == "cost_grad":
        N = sum(_counts(case))
        return {"bytes": (7 * b + 28) * N + 400 * case["pairs"], "flops": N * 130}
    if kind == "points":
        return {"bytes": (3 * b + 12) * case["rows"] + 40 * case["corr"] + 136 * case["submaps"], "flops": 18 * case["rows"]}
    n, e = case["nodes"], case["nodes"] - 1 + case["loops"]
    # per iteration: edges linearised (about 4000 operations each), a sparse factor of about 343 operations for each
    # pair of blocks of a column (order of 10 blocks a column), the solves
    return {"bytes": 128 * n + (128 + 392 + 8) * e, "flops": case["iters"] * (4000 * e + n * (100 * 343 + 2 * 10 * 98))}


# ---------------------------------------------------------------- the same in 64 bits

def _segments(planes, off):
    o = off.cpu().numpy()
    X = [p.detach() for p in planes]
    for k in range(len(o) - 1):
        a, b = int(o[k]), int(o[k + 1])
        yield k, a, b, torch.stack([p[a:b].to(F8) for p in X])


def _valid(x, tau):
    return torch.isfinite(x).all(0) & (x[6] >= float(np.float32(tau)))


def _gram(A, B):
    """A B^T of (a, n) and (b, n) for a long n: a product by sums, which spread over the chip."""
    return torch.stack([(x * B).sum(-1) for x in A])


def _umeyama(p, q, w):
    W = w.sum()
    mp, mq = (p * w).sum(1) / W, (q * w).sum(1) / W
    P, Q = p - mp[:, None], q - mq[:, None]
    U, D, Vt = np.linalg.svd((_gram(Q * w, P) / W).cpu().numpy())
    sg = np.array([1.0, 1.0, np.sign(np.linalg.det(U) * np.linalg.det(Vt))])
    R = U @ np.diag(sg) @ Vt
    s = float((D * sg).sum()) / float(((P * P).sum(0) * w).sum() / W)
    mp, mq = mp.cpu().numpy(), mq.cpu().numpy()
    return s, R, mq - s * R @ mp


def _hat(v):
    """(..., 3) -> (..., 3, 3)"""
    o = torch.zeros_like(v[..., 0])
    return torch.stack([torch.stack([o, -v[..., 2], v[..., 1]], -1), torch.stack([v[..., 2], o, -v[..., 0]], -1),
                        torch.stack([-v[..., 1], v[..., 0], o], -1)], -2)


def _gen4(x):
    """(..., 7) tangent (rho, omega, sigma) -> (..., 4, 4) generator"""
    G = torch.zeros(x.shape[:-1] + (4, 4), dtype=F8, device=x.device)
    G[..., :3, :3] = _hat(x[..., 3:6]) + x[..., 6, None, None] * torch.eye(3, dtype=F8, device=x.device)
    G[..., :3, 3] = x[..., :3]
    return G


def _mat4(s, R, t):
    T = torch.eye(4, dtype=F8)
    T[:3, :3] = torch.as_tensor(s * np.asarray(R))
    T[:3, 3] = torch.as_tensor(np.asarray(t))
    return T


def _row(T):
    """(..., 4, 4) -> (..., 16) in the library's layout"""
    s = torch.linalg.det(T[..., :3, :3]) ** (1.0 / 3.0)
    out = torch.zeros(T.shape[:-2] + (16,), dtype=F8, device=T.device)
    out[..., :9] = (T[..., :3, :3] / s[..., None, None]).reshape(T.shape[:-2] + (9,))
    out[..., 9:12], out[..., 12] = T[..., :3, 3], s
    return out


def _residual(T, p, q):
    y = T[:3, :3] @ p + T[:3, 3:4]
    r = y - q
    e = torch.sqrt((r * r).sum(0))
    psi = torch.where(e <= DELTA, torch.ones_like(e), DELTA / torch.clamp(e, min=1e-300))
    return y, r, e, psi


def _jacobian(y):
    """(7, 3, n): columns of d(Exp(xi) y)/dxi"""
    n = y.shape[1]
    J = torch.zeros(7, 3, n, dtype=F8, device=y.device)
    for i in range(3):
        J[i, i] = 1.0
    J[3, 1], J[3, 2] = -y[2], y[1]
    J[4, 0], J[4, 2] = y[2], -y[0]
    J[5, 0], J[5, 1] = -y[1], y[0]
    J[6] = y
    return J


def _irls(p, q, w, iters):
    T = _mat4(*_umeyama(p, q, w)).to(p.device)
    for _ in range(iters):
        y, r, _, psi = _residual(T, p, q)
        mid = (y * w).sum(1) / w.sum()  # the step is solved about the points' middle, then moved back
        J = _jacobian(y - mid[:, None]).reshape(7, -1)
        Jw = J * (w * psi).repeat(3)
        Hg = _gram(Jw, torch.cat([J, r.reshape(1, -1)])).cpu()
        x = torch.linalg.solve(Hg[:, :7], -Hg[:, 7])
        c, om = mid.cpu(), x[3:6]
        x = torch.cat([x[:3] + torch.linalg.cross(c, om) - x[6] * c, x[3:]])
        T = torch.matrix_exp(_gen4(x)).to(p.device) @ T
    return T


def _exact_align(segments, tau, iters):
    rows = []
    for _, _, _, x in segments:
        x = x[:, _valid(x, tau)]
        rows.append(_row(_irls(x[:3], x[3:6], x[6], iters).cpu()))
    return torch.stack(rows).to(DEV)


def _depth_segments(planes, off, rec):
    for k, a, b, d in _segments(planes, off):
        w, hw = int(rec[k]["width"]), int(rec[k]["frame_pixels"])
        j = torch.arange(b - a, device=DEV)
        f, pin = j // hw, j % hw
        col, line = (pin % w).to(F8), (pin // w).to(F8)
        x = torch.empty(7, b - a, dtype=F8, device=DEV)
        for side, at, depth in (("p", 0, d[0]), ("q", 3, d[1])):
            for g in range(int(rec[k]["n_frames"])):
                cam, here = rec[k][side][g], f == g
                ray = torch.stack([(col - float(cam["cx"])) / float(cam["fx"]), (line - float(cam["cy"])) / float(cam["fy"]), torch.ones_like(col)])
                R = torch.from_numpy(cam["R"].astype(np.float64).reshape(3, 3)).to(DEV)
                t = torch.from_numpy(cam["t"].astype(np.float64)).to(DEV)
                x[at:at + 3] = torch.where(here, R @ (depth * ray) + t[:, None], x[at:at + 3])
        x[6] = d[2]
        yield k, a, b, x


def _exact_cost_grad(case, seed):
    planes, off, gt = _planes(case, seed)
    r = np.random.default_rng(int(seed) + 77)
    gL = torch.from_numpy(r.uniform(0.5, 1.5, case["pairs"])).to(DEV)
    S = _near(gt, r)
    xi = torch.from_numpy(0.005 * r.normal(size=(case["pairs"], 7)))
    N = planes[0].numel()
    g = torch.zeros(7, N, dtype=F8, device=DEV)
    L, gxi = torch.zeros(case["pairs"], dtype=F8), torch.zeros(case["pairs"], 7, dtype=F8)
    for k, a, b, x in _segments(planes, off):
        m = _valid(x, _tau(case))
        x = x[:, m].requires_grad_()
        z = xi[k].clone().requires_grad_()
        T = (torch.matrix_exp(_gen4_diff(z)) @ _mat4(*S[k])).to(DEV)
        res = T[:3, :3] @ x[:3] + T[:3, 3:4] - x[3:6]
        e2 = (res * res).sum(0)
        e = torch.sqrt(torch.clamp(e2, min=1e-300))
        rho = torch.where(e <= DELTA, 0.5 * e2, DELTA * (e - 0.5 * DELTA))
        Lk = (x[6] * rho).sum() / x[6].sum()
        gx, gz = torch.autograd.grad(gL[k] * Lk, [x, z])
        L[k], gxi[k] = Lk.item(), gz
        g[:, a:b][:, m] = gx
    if case["dtype"] == "bf16":
        return L, g[:3], g[3:6], g[6], gxi
    return (L,) + tuple(g) + (gxi,)


def _gen4_diff(x):
    """_gen4 without in-place writes, for autograd."""
    o = torch.zeros((), dtype=F8)
    return torch.stack([torch.stack([x[6], -x[5], x[4], x[0]]), torch.stack([x[5], x[6], -x[3], x[1]]),
                        torch.stack([-x[4], x[3], x[6], x[2]]), torch.stack([o, o, o, o])])


def _exact_solve_grad(case, seed):
    planes, off, _ = _planes(case, seed)
    r = np.random.default_rng(int(seed) + 77)
    r.uniform(0.5, 1.5, case["pairs"])
    gS = torch.from_numpy(r.normal(size=(case["pairs"], 16)))
    g = torch.zeros(7, planes[0].numel(), dtype=F8, device=DEV)
    rows = []
    E = _gen4(torch.eye(7, dtype=F8))
    for k, a, b, x in _segments(planes, off):
        m = _valid(x, _tau(case))
        x = x[:, m]
        T = _irls(x[:3], x[3:6], x[6], case["iters"])
        Tc = T.cpu()
        row = _row(Tc)
        rows.append(row)
        # the exact Hessian of the Huber cost in a left perturbation, about T
        y, res, e, psi = _residual(T, x[:3], x[3:6])
        w = x[6] / x[6].sum()
        J = _jacobian(y)
        flat = J.reshape(7, -1)
        H = _gram(flat * (w * psi).repeat(3), flat)
        Jr = (J * res).sum(1)
        far = torch.where(e > DELTA, w * psi / torch.clamp(e * e, min=1e-300), torch.zeros_like(e))
        H = (H - _gram(Jr * far, Jr)).cpu()
        yh = torch.cat([y, torch.ones(1, y.shape[1], dtype=F8, device=DEV)])
        K = _gram(res * (w * psi), yh).cpu()
        GG = torch.matmul(E[:, None], E[None])[..., :3, :]
        H = H + 0.5 * ((GG + GG.transpose(0, 1)) * K).sum((-1, -2))
        # dl/dxi from dl/dS: S -> Exp(xi) S moves R, t and s
        R, t, s = row[:9].reshape(3, 3), row[9:12], row[12]
        gR, gt_, gs = gS[k, :9].reshape(3, 3), gS[k, 9:12], gS[k, 12]
        u = torch.empty(7, dtype=F8)
        u[:3] = gt_
        for i in range(3):
            G = E[3 + i, :3, :3]
            u[3 + i] = (gR * (G @ R)).sum() + (gt_ * (G @ t)).sum()
        u[6] = gs * s + (gt_ * t).sum()
        v = torch.linalg.solve(H, u).to(DEV)
        z = x.clone().requires_grad_()
        y2 = T[:3, :3] @ z[:3] + T[:3, 3:4]
        r2 = y2 - z[3:6]
        e2 = torch.sqrt(torch.clamp((r2 * r2).sum(0), min=1e-300))
        om = z[6] * torch.where(e2 <= DELTA, torch.ones_like(e2), DELTA / e2)
        Jv = v[:3, None] + torch.linalg.cross(v[3:6, None].expand_as(y2), y2, dim=0) + v[6] * y2
        Fv = (om * (Jv * r2).sum(0)).sum() / z[6].sum()
        g[:, a:b][:, m] = -torch.autograd.grad(Fv, z)[0]
    return (torch.stack(rows),) + tuple(g)


def _log4(Z):
    """(..., 4, 4) similarities -> (..., 7)"""
    s = torch.linalg.det(Z[..., :3, :3]) ** (1.0 / 3.0)
    R = Z[..., :3, :3] / s[..., None, None]
    a = 0.5 * torch.stack([R[..., 2, 1] - R[..., 1, 2], R[..., 0, 2] - R[..., 2, 0], R[..., 1, 0] - R[..., 0, 1]], -1)
    sn = torch.linalg.norm(a, dim=-1)
    th = torch.atan2(sn, 0.5 * (R[..., 0, 0] + R[..., 1, 1] + R[..., 2, 2] - 1.0))
    om = a * torch.where(sn > 1e-12, th / torch.clamp(sn, min=1e-300), torch.ones_like(sn))[..., None]
    sg = torch.log(s)
    A = _hat(om) + sg[..., None, None] * torch.eye(3, dtype=F8, device=Z.device)
    B = torch.zeros(Z.shape[:-2] + (6, 6), dtype=F8, device=Z.device)
    B[..., :3, :3], B[..., :3, 3:] = A, torch.eye(3, dtype=F8, device=Z.device)
    V = torch.matrix_exp(B)[..., :3, 3:]
    return torch.cat([torch.linalg.solve(V, Z[..., :3, 3]), om, sg[..., None]], -1)


def _ad(x):
    """(..., 7) -> (..., 7, 7) of the bracket, order (rho, omega, sigma)"""
    A = torch.zeros(x.shape[:-1] + (7, 7), dtype=F8, device=x.device)
    W = _hat(x[..., 3:6])
    A[..., :3, :3] = W + x[..., 6, None, None] * torch.eye(3, dtype=F8, device=x.device)
    A[..., :3, 3:6] = _hat(x[..., :3])
    A[..., :3, 6] = -x[..., :3]
    A[..., 3:6, 3:6] = W
    return A


def _Ad(T):
    """(..., 4, 4) -> (..., 7, 7)"""
    s = torch.linalg.det(T[..., :3, :3]) ** (1.0 / 3.0)
    R, t = T[..., :3, :3] / s[..., None, None], T[..., :3, 3]
    A = torch.zeros(T.shape[:-2] + (7, 7), dtype=F8, device=T.device)
    A[..., :3, :3] = T[..., :3, :3]
    A[..., :3, 3:6] = torch.matmul(_hat(t), R)
    A[..., :3, 6] = -t
    A[..., 3:6, 3:6] = R
    A[..., 6, 6] = 1.0
    return A


def _exact_pgo(case, seed):
    edges, meas, omega = _pgo_inputs(case, seed)
    n, m = case["nodes"], len(edges)
    i, j = (torch.from_numpy(edges[:, k].astype(np.int64)).to(DEV) for k in (0, 1))
    Om = omega.reshape(m, 7, 7)
    M = torch.eye(4, dtype=F8, device=DEV).repeat(m, 1, 1)
    M[:, :3, :3], M[:, :3, 3] = meas[:, 12, None, None] * meas[:, :9].reshape(m, 3, 3), meas[:, 9:12]
    Mi = torch.linalg.inv(M)
    # the start: poses chained breadth first from node 0
    T, Mh, Mih = [None] * n, M.cpu(), Mi.cpu()
    T[0] = torch.eye(4, dtype=F8)
    at = [[] for _ in range(n)]
    for k, (a, b) in enumerate(edges):
        at[a].append(k)
        at[b].append(k)
    todo = [0]
    for a in todo:
        for k in at[a]:
            u, v = int(edges[k][0]), int(edges[k][1])
            if u == a and T[v] is None:
                T[v] = T[a] @ Mh[k]
                todo.append(v)
            elif v == a and T[u] is None:
                T[u] = T[a] @ Mih[k]
                todo.append(u)
    T = torch.stack(T).to(DEV)

    def residual(T):
        e = _log4(torch.matmul(torch.matmul(Mi, torch.linalg.inv(T[i])), T[j]))
        q = (e * torch.matmul(Om, e[..., None])[..., 0]).sum(-1)
        return e, q

    def system(T, e, q):
        B = torch.zeros(m, 14, 14, dtype=F8, device=DEV)
        B[:, :7, :7], B[:, :7, 7:] = -_ad(e), torch.eye(7, dtype=F8, device=DEV)
        A = torch.linalg.solve(torch.matrix_exp(B)[:, :7, 7:], _Ad(torch.linalg.inv(T[j])))
        r = torch.sqrt(q)
        psi = torch.where(r <= HUBER_PG, torch.ones_like(r), HUBER_PG / torch.clamp(r, min=1e-300))
        AtO = torch.matmul(A.transpose(1, 2), Om) * psi[:, None, None]
        D, v = torch.matmul(AtO, A), torch.matmul(AtO, e[..., None])[..., 0]
        H = torch.zeros(n * n, 7, 7, dtype=F8, device=DEV)
        for a, b, s in ((i, i, 1.0), (j, j, 1.0), (i, j, -1.0), (j, i, -1.0)):
            H.index_add_(0, a * n + b, s * D)
        H = H.reshape(n, n, 7, 7).permute(0, 2, 1, 3).reshape(7 * n, 7 * n)[7:, 7:].contiguous()
        g = torch.zeros(n, 7, dtype=F8, device=DEV).index_add_(0, j, v).index_add_(0, i, -v)
        return H, g.reshape(-1)[7:]

    def step(H, g, lam):
        d = torch.diagonal(H).clone()
        A = H.clone()
        A.diagonal().add_(lam * d)
        L = torch.linalg.cholesky(A)
        x = -torch.cholesky_solve(g[:, None], L)[:, 0]
        full = torch.zeros(n, 7, dtype=F8, device=DEV)
        full[1:] = x.reshape(-1, 7)
        return full, float(0.5 * (x * (lam * d * x - g)).sum())

    def energy(q):
        r = torch.sqrt(q)
        return float(torch.where(r <= HUBER_PG, 0.5 * q, HUBER_PG * (r - 0.5 * HUBER_PG)).sum())

    e, q = residual(T)
    if not case["lm"]:
        for _ in range(case["iters"]):
            x, _ = step(*system(T, e, q), 0.0)
            T = torch.matmul(torch.matrix_exp(_gen4(x)), T)
            e, q = residual(T)
    else:
        lam, F, kept = 1e-4, energy(q), 0
        while kept < case["iters"]:
            H, g = system(T, e, q)
            nu, good = 2.0, False
            for _ in range(10):
                x, pred = step(H, g, lam)
                if pred <= 1e-15 * F:
                    break
                Tt = torch.matmul(torch.matrix_exp(_gen4(x)), T)
                et, qt = residual(Tt)
                Ft = energy(qt)
                if Ft < F:
                    lam *= max(1.0 / 3.0, 1.0 - (2.0 * (F - Ft) / pred - 1.0) ** 3)
                    T, e, q, F, good = Tt, et, qt, Ft, True
                    break
                lam, nu = lam * nu, nu * 2.0
            if not good:
                break
            kept += 1
    return _row(T), float(q.sum())


def exact(case, seed):
    kind = case["kind"]
    if kind == "align":
        planes, off, _ = _planes(case, seed)
        return _exact_align(_segments(planes, off), _tau(case), case["iters"])
    if kind == "depth":
        planes, off, rec = _depth_inputs(case, seed)
        return _exact_align(_depth_segments(planes, off, rec), 1.5, case["iters"])
    if kind == "cost_grad":
        return _exact_cost_grad(case, seed)
    if kind == "solve_grad":
        return _exact_solve_grad(case, seed)
    if kind == "points":
        xyz, off, T, src, dst, sparse = _points_inputs(case, seed)
        o = off.cpu().numpy()
        world = torch.empty(3, case["rows"], dtype=F8, device=DEV)
        for k in range(case["submaps"]):
            a, b = int(o[k]), int(o[k + 1])
            world[:, a:b] = (T[k, 12] * T[k, :9].reshape(3, 3)) @ xyz[:, a:b].to(F8) + T[k, 9:12, None]
        out = sparse.to(F8)
        out[:, dst] = world[:, src]
        return world, out
    return _exact_pgo(case, seed)
