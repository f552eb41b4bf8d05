"""Performance cases of the pose solver: the calls its users make, with their inputs.

A case names one call form ("kind") and its sizes:

  solve      Context.solve of one frame (the multi-hypothesis LM registration)
  static     Context.solve_static of one frame (no device allocation)
  batch      Context.solve of several uneven frames in one call
  serve      admit / step / poll of concurrently served frames until all are done
  linearize  Context.linearize of one level (normal equations at given poses)
  lift       Context.lift of a frame's anchors and their descriptors, all levels

"tiles" says which context the program holds: one that reads the shipped tile
database (as the benchmark and the serving loop do) or a default Context(0).
Contexts live as long as the program; frames are new from call to call.

The inputs are synthetic registration frames of the kind the package's
benchmark draws: a DSM crop with hills and buildings, an oblique camera 150 m
above it, smooth unit-norm descriptor fields, reference descriptors sampled at
the true projections with noise, noisy gravity and laser-range readings, and
hypotheses within 20 m / 10 degrees of a prior 5 m / 3 degrees off the truth.
"""
import math
import os
import random
from types import SimpleNamespace

import numpy as np
import torch

import paper_2606_31098_amd as package
from paper_2606_31098_amd.pilot import Context, DeviceFrame, DeviceResult

TILES = os.path.join(os.path.dirname(os.path.abspath(package.__file__)), "tiles_gfx950.txt")

# the pyramid of the benchmark and the channel counts per level, coarse to fine
FINEST = {"S": (120, 160), "M": (240, 320), "L": (360, 480), "XL": (480, 640)}


def _case(name, kind, **kw):
    c = dict(name=name, kind=kind, N=8192, M=256, fine="XL", levels=3, channels="32-64-128", iters="15-15-15",
             bf16=False, tiles=True, weights=False, adaptive=False, grid=False, frames=1)
    c.update(kw)
    return c


def listed():
    return [
        # tracking a single prior pose: one small level, latency of one call
        _case("single", "solve", N=1024, M=1, levels=1, fine="S", channels="32", iters="20"),
        # a first program on a default context: small odd sizes, every option on
        _case("small_default", "solve", N=777, M=13, fine="S", channels="16-32-64", iters="8-8-8", tiles=False,
              weights=True, adaptive=True),
        # the method's online form: 500 anchors, the 1210-pose grid pruned to 128, few iterations
        _case("paper_grid", "solve", N=500, M=1210, channels="32-32-32", iters="2-3-4", grid=True),
        # the plain FP32 pyramid solve, with the tile database and as the README's example runs it
        _case("pyramid_f32", "solve"),
        _case("pyramid_default", "solve", tiles=False),
        # a tight loop that may not allocate: odd sizes, bf16
        _case("static_bf16", "static", N=5003, M=97, bf16=True),
        # the benchmark's workload (precision form) and the FP32 solver on the same sizes
        _case("large_bf16", "solve", N=16384, M=1024, bf16=True),
        _case("large_f32", "solve", N=16384, M=1024),
        # offline registration: uneven frames in one call
        _case("batch_bf16", "batch", frames=10, bf16=True),
        # four video streams served together, few iterations each
        _case("serve_bf16", "serve", frames=4, bf16=True, iters="2-3-4"),
        # covariance / diagnostics: the normal equations of the finest level at every hypothesis
        _case("linearize", "linearize", N=8192, M=256, tiles=False),
        # building a frame's anchors from the DSM and the reference pyramid
        _case("lift", "lift", N=16384, bf16=True),
    ]


def draw(rng):
    kind = rng.choice(["solve"] * 6 + ["static", "linearize", "linearize", "lift", "serve"])
    bf16 = rng.random() < 0.5
    tiles = rng.random() < 0.6

    def log_uniform(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    N = log_uniform(300, 16384)
    M = log_uniform(1, 1024)
    most = (1 << 21) if (not tiles or kind == "static") else (1 << 23)
    while N * M > most:
        M = max(1, M // 2)
    fine = rng.choice(["S", "M", "L", "XL"])
    levels = rng.choice([1, 2, 3, 3])
    channels = rng.choice(["32-64-128", "32-64-128", "32-32-32", "16-32-64"])
    channels = "-".join(channels.split("-")[-levels:])
    iters = "-".join(rng.choice(["15-15-15", "2-3-4", "8-8-8"]).split("-")[:levels])
    c = _case("", kind, N=N, M=M, fine=fine, levels=levels, channels=channels, iters=iters, bf16=bf16, tiles=tiles,
              weights=rng.random() < 0.25, adaptive=rng.random() < 0.25)
    if kind == "serve":
        c.update(frames=rng.randint(1, 6), iters="-".join("2-3-4".split("-")[:levels]))
    del c["name"]
    return c


# ----------------------------------------------------------------- inputs
def _rz(a):
    c, s = math.cos(a), math.sin(a)
    return np.array([[c, -s, 0.0], [s, c, 0.0], [0.0, 0.0, 1.0]])


def _pose(R_wc, C):
    return np.concatenate([R_wc.T.reshape(-1), -R_wc.T @ C])


def _axis_angle(axis, angle):
    k = axis / np.linalg.norm(axis)
    K = np.array([[0.0, -k[2], k[1]], [k[2], 0.0, -k[0]], [-k[1], k[0], 0.0]])
    return np.eye(3) + math.sin(angle) * K + (1.0 - math.cos(angle)) * (K @ K)


def _dsm(rng, side, gsd=0.5):
    """Eight hills over 50 m and four buildings, (side, side) heights, centred."""
    ext = (side - 1) * gsd
    ax = np.arange(side) * gsd - 0.5 * ext
    h = np.zeros((side, side))
    for _ in range(8):
        cx, cy = rng.uniform(-0.75 * ext, 0.75 * ext, 2)
        s = rng.uniform(0.1, 0.4) * ext
        h += rng.uniform(0.5, 1.0) * np.exp(-((ax[None] - cx) ** 2 + (ax[:, None] - cy) ** 2) / (2 * s * s))
    h = (h - h.min()) / (h.max() - h.min()) * 50.0
    for _ in range(4):
        w, l = rng.uniform(0.1, 0.25, 2) * side
        i, j = rng.uniform(0, side, 2)
        h[int(max(0, i - l / 2)):int(i + l / 2), int(max(0, j - w / 2)):int(j + w / 2)] += rng.uniform(10.0, 40.0)
    return SimpleNamespace(heights=h.astype(np.float32), x0=-0.5 * ext, y0=-0.5 * ext, gsd=gsd)


def _blur_matrix(n, sigma=8.0):
    """Dense Gaussian blur with reflected borders along an axis of n samples."""
    r = int(math.ceil(4 * sigma))
    k = np.exp(-np.arange(-r, r + 1) ** 2 / (2 * sigma ** 2))
    k /= k.sum()
    B = np.zeros((n, n))
    for d, w in zip(range(-r, r + 1), k):
        j = np.abs(np.arange(n) + d)
        j = np.where(j > n - 1, 2 * (n - 1) - j, j)
        B[np.arange(n), np.clip(j, 0, n - 1)] += w
    return torch.as_tensor(B, dtype=torch.float32, device="cuda")


def _field(gen, H, W, C):
    """Smooth random descriptor field, unit norm per pixel, (H, W, C) on the device."""
    x = torch.randn((H, W * C), generator=gen, device="cuda")
    x = (_blur_matrix(H) @ x).view(H, W, C)
    x = torch.matmul(_blur_matrix(W), x)
    return x / x.norm(dim=2, keepdim=True)


def _sample(F, u, v):
    """Bilinear samples of a device field at float64 pixel coordinates."""
    H, W, _ = F.shape
    u, v = torch.as_tensor(u, device="cuda"), torch.as_tensor(v, device="cuda")
    x0, y0 = u.floor().long().clamp(0, W - 2), v.floor().long().clamp(0, H - 2)
    a, b = (u - x0).float()[:, None], (v - y0).float()[:, None]
    return (1 - b) * ((1 - a) * F[y0, x0] + a * F[y0, x0 + 1]) + b * ((1 - a) * F[y0 + 1, x0] + a * F[y0 + 1, x0 + 1])


def _shapes(case):
    H, W = FINEST[case["fine"]]
    C = [int(c) for c in case["channels"].split("-")]
    n = case["levels"]
    return [(max(H >> (n - 1 - l), 2), max(W >> (n - 1 - l), 2), C[l]) for l in range(n)]


def _intrinsics(H, W):
    s = 140.0 * H / 120.0
    return (s, s, (W - 1) / 2.0, (H - 1) / 2.0)


def _frame(case, seed):
    """One registration frame of host arrays, as a program hands it to DeviceFrame."""
    rng = np.random.default_rng([seed, 31098])
    gen = torch.Generator(device="cuda").manual_seed(seed * 7919 + 17)
    N, shapes = case["N"], _shapes(case)
    dsm = _dsm(rng, 128 if N <= 4096 else 256)
    side = dsm.heights.shape[0]
    pitch, roll = math.radians(45.0), math.radians(rng.uniform(-3.0, 3.0))
    c, s = math.cos(-pitch), math.sin(-pitch)
    rx = np.array([[1.0, 0.0, 0.0], [0.0, c, -s], [0.0, s, c]])
    R_wc = _rz(rng.uniform(0, 2 * math.pi)) @ np.array([[1.0, 0, 0], [0, 0, 1.0], [0, -1.0, 0]]) @ rx @ _rz(roll)
    axis = R_wc[:, 2]
    C = axis * (150.0 / axis[2])
    gt = _pose(R_wc, C)

    jj, ii = np.meshgrid(np.arange(side), np.arange(side))
    P = np.stack([(dsm.x0 + jj * dsm.gsd).ravel(), (dsm.y0 + ii * dsm.gsd).ravel(), dsm.heights.ravel()], 1)
    P = P.astype(np.float32).astype(np.float64)
    X = P @ gt[:9].reshape(3, 3).T + gt[9:]
    ok = X[:, 2] > 1.0
    for H, W, _ in shapes:
        fx, fy, cx, cy = _intrinsics(H, W)
        u, v = fx * X[:, 0] / X[:, 2] + cx, fy * X[:, 1] / X[:, 2] + cy
        ok &= (u >= 1) & (u <= W - 2) & (v >= 1) & (v <= H - 2)
    seen = np.flatnonzero(ok)
    at = np.sort(rng.choice(seen, N, replace=N > seen.size))
    P, X = P[at], X[at]

    levels = []
    for (H, W, Cl), it in zip(shapes, case["iters"].split("-")):
        fx, fy, cx, cy = _intrinsics(H, W)
        F = _field(gen, H, W, Cl)
        ref = _sample(F, fx * X[:, 0] / X[:, 2] + cx, fy * X[:, 1] / X[:, 2] + cy)
        ref = ref + 0.05 * torch.randn(ref.shape, generator=gen, device="cuda")
        x, y, z = (np.ascontiguousarray(P[:, k], dtype=np.float32) for k in range(3))
        levels.append(SimpleNamespace(
            H=H, W=W, C=Cl, feat=F.cpu().numpy(), K=(fx, fy, cx, cy), x=x, y=y, z=z, ref=ref.cpu().numpy(),
            iters=int(it), loss=(0, 0.1 * Cl / 32.0),
            ref_w=rng.uniform(0.2, 1.0, N).astype(np.float32) if case["weights"] else None,
            qconf=rng.uniform(0.2, 1.0, (H, W)).astype(np.float32) if case["weights"] else None))

    def unit():
        d = rng.normal(size=3)
        return d / np.linalg.norm(d)

    prior_C = C + 5.0 * unit()
    prior_R = R_wc @ _axis_angle(unit(), math.radians(3.0))
    if case["grid"]:
        steps = np.arange(-10.0, 10.1, 2.0)
        yaws = [math.radians(k * a) for a in (1, 3, 5, 7, 9) for k in (1, -1)]
        offsets = np.array([(x, y, a) for x in steps for y in steps for a in yaws])
    else:
        M = case["M"]
        offsets = np.stack([rng.uniform(-20, 20, M), rng.uniform(-20, 20, M), np.radians(rng.uniform(-10, 10, M))], 1)
        offsets[0] = 0.0
    poses = np.stack([_pose(_rz(a) @ prior_R, prior_C + np.array([x, y, 0.0])) for x, y, a in offsets])

    # noisy gravity (0.5 degrees) and laser range (0.5 m) along the optical axis
    p, r = pitch + math.radians(rng.normal(0, 0.5)), roll + math.radians(rng.normal(0, 0.5))
    g_imu = np.array([math.cos(p) * math.sin(r), math.cos(p) * math.cos(r), math.sin(p)])
    t = np.arange(0.0, 400.0, 0.25)
    ray = C[None] + t[:, None] * axis[None]
    j = np.clip(np.rint((ray[:, 0] - dsm.x0) / dsm.gsd).astype(int), 0, side - 1)
    i = np.clip(np.rint((ray[:, 1] - dsm.y0) / dsm.gsd).astype(int), 0, side - 1)
    d_range = float(t[np.argmax(ray[:, 2] <= dsm.heights[i, j])] + rng.normal(0, 0.5))
    H, W, _ = shapes[-1]
    return SimpleNamespace(
        levels=levels, poses=poses, dsm=dsm, g_imu=g_imu, d_range=max(d_range, 1.0), pc=((W - 1) / 2.0, (H - 1) / 2.0),
        use_gravity=1, use_range=1, g_world=(0.0, 0.0, -1.0), lambda_imu=0.05 ** 2 / math.radians(0.5) ** 2,
        lambda_range=0.05 ** 2 / 0.5 ** 2, gravity_loss=(1, math.radians(1.5) ** 2), range_loss=(1, 1.5 ** 2),
        lm=dict(tau=1e-6, up=10.0, down=10.0, lambda_min_rel=1e-12, lambda_max_rel=1e8, step_tol_t=1e-5,
                step_tol_r=1e-7, z_min=0.1, min_valid=8, cost_tol=1e-6),
        keep_top=128 if case["grid"] else 0, prune_level=0, adaptive_priors=int(case["adaptive"]), alpha_ratio=1.0,
        gravity_gate=5 * math.radians(0.5), range_gate=2.5, uv=at)


def _cases_of(case):
    """The frames of a case: one, or several uneven ones (batch, serve)."""
    if case["kind"] not in ("batch", "serve"):
        return [case]
    out = []
    r = random.Random(4 + 131 * case["N"] + case["M"])
    for _ in range(case["frames"]):
        if case["kind"] == "batch":
            c = dict(case, N=int(math.exp(r.uniform(math.log(2048), math.log(32768)))),
                     M=r.choice([32, 64, 128, 256, 512]), fine=r.choice(["M", "L", "XL"]))
        else:
            c = dict(case, N=max(64, int(case["N"] * r.uniform(0.25, 1.0))), M=r.choice([64, 128, 256]))
        out.append(c)
    return out


_contexts = {}


def _context(case):
    key = (case["tiles"], case["kind"] == "serve")
    if key not in _contexts:
        _contexts[key] = Context(0, tune_cache=TILES if case["tiles"] else None, max_slots=8 if key[1] else 0)
    return _contexts[key]


def prepare(case, seed):
    ctx = _context(case)
    host = [_frame(c, seed * 64 + k) for k, c in enumerate(_cases_of(case))]
    state = SimpleNamespace(kind=case["kind"], ctx=ctx)
    if case["kind"] == "lift":
        f, dt = host[0], torch.bfloat16 if case["bf16"] else torch.float32
        gen = np.random.default_rng([seed, 5])
        side = f.dsm.heights.shape[0]
        state.dsm = torch.as_tensor(f.dsm.heights, device="cuda")
        state.at = (f.dsm.x0, f.dsm.y0, f.dsm.gsd)
        # anchors anywhere on the crop, not only on its samples
        state.uv = torch.as_tensor(gen.uniform(0, side - 1, (case["N"], 2)).astype(np.float32), device="cuda")
        state.maps = [(torch.as_tensor(L.feat, device="cuda").to(dt), L.H / side) for L in f.levels]
        return state
    state.frames = [DeviceFrame(f, dtype="bf16" if case["bf16"] else "f32") for f in host]
    if case["kind"] == "linearize":
        state.level = case["levels"] - 1
    else:
        state.results = [DeviceResult(d.M) for d in state.frames]
    return state


def run(state):
    ctx = state.ctx
    if state.kind == "lift":
        out = []
        for k, (F, scale) in enumerate(state.maps):
            x, y, z, ref = ctx.lift(state.dsm, *state.at, state.uv, F, scale, points=k == 0)
            out.append(dict(x=x, y=y, z=z, ref=ref) if k == 0 else dict(ref=ref))
        return out
    if state.kind == "linearize":
        f = state.frames[0]
        H, g, cost, n = ctx.linearize(f, state.level, f.poses)
        return dict(H=H, g=g, cost=cost, n=n)
    if state.kind == "static":
        ctx.solve_static(state.frames, state.results)
    elif state.kind == "serve":
        live = [ctx.admit(f, r) for f, r in zip(state.frames, state.results)]
        while live:
            ctx.step()
            live = [s for s in live if not ctx.poll(s)]
    else:
        ctx.solve(state.frames, state.results)
    return [dict(poses=r.poses, cost=r.cost, alpha=r.alpha, iterations=r.iterations, status=r.status, best=r.best)
            for r in state.results]


def work(case):
    """Every input read once and every output written once; the operations of
    the evaluations no solve does without: at each level the start pose and up
    to three steps of every hypothesis (a tenth of them where the grid has been
    pruned), four tap products per channel and about 250 operations a pair."""
    es = 2 if case["bf16"] else 4
    nbytes = flops = 0.0
    for c in _cases_of(case):
        shapes = _shapes(c)
        M = 1210 if c["grid"] else c["M"]
        if c["kind"] == "lift":
            side = 128 if c["N"] <= 4096 else 256
            nbytes += side * side * 4 + c["N"] * 20
            for H, W, C in shapes:
                nbytes += min(H * W, 4 * c["N"]) * C * es + c["N"] * C * es
                flops += 10.0 * c["N"] * C
            continue
        if c["kind"] == "linearize":
            shapes = shapes[-1:]
        for l, ((H, W, C), it) in enumerate(zip(shapes, c["iters"].split("-"))):
            m = 128 if c["grid"] and l > 0 else M
            nbytes += H * W * C * es + c["N"] * (C * es + 12) + (c["N"] * 4 + H * W * 4 if c["weights"] else 0)
            evals = 1 if c["kind"] == "linearize" else 1 + min(int(it), 3)
            flops += evals * float(c["N"]) * m * (8.0 * C + 250.0)
        nbytes += M * (96 + (232 if c["kind"] == "linearize" else 128))
    return {"bytes": nbytes, "flops": flops}


# ----------------------------------------------------- the same in 64 bits
def _rho(kind, b, s):
    if kind == 0:
        return b * torch.log1p(s / b), 1.0 / (1.0 + s / b)
    r = (b * s).clamp_min(1e-300).sqrt()
    return torch.where(s <= b, s, 2 * r - b), torch.where(s <= b, torch.ones_like(s), b / r)


def _f64(a, bf16=False):
    t = torch.as_tensor(a, device="cuda")
    return (t.to(torch.bfloat16) if bf16 else t).to(torch.float64)


class _Exact:
    """A frame's objective in FP64 torch: photometric sums and priors."""

    def __init__(self, f, bf16):
        self.f = f
        self.lv = [SimpleNamespace(
            F=_f64(L.feat, bf16).reshape(-1, L.C), ref=_f64(L.ref, bf16), P=torch.stack([_f64(L.x), _f64(L.y), _f64(L.z)], 1),
            w=_f64(L.ref_w) if L.ref_w is not None else torch.ones(len(L.x), dtype=torch.float64, device="cuda"),
            q=_f64(L.qconf).reshape(-1) if L.qconf is not None else None, L=L) for L in f.levels]
        self.dsm = _f64(f.dsm.heights)

    def photo(self, l, T):
        """J^T W J, J^T W r, cost and visible count of poses T (M, 12) at level l."""
        v = self.lv[l]
        N, C = v.ref.shape
        step = max(1, (1 << 24) // max(1, N * C))
        parts = [self._photo(v, T[i:i + step]) for i in range(0, len(T), step)]
        return [torch.cat(p) for p in zip(*parts)]

    def _photo(self, v, T):
        L, (fx, fy, cx, cy) = v.L, v.L.K
        R, t = T[:, :9].view(-1, 3, 3), T[:, 9:]
        X = torch.matmul(v.P[None].expand(len(T), -1, -1).contiguous(), R.transpose(1, 2).contiguous()) + t[:, None]
        x, y, Z = X[..., 0] / X[..., 2], X[..., 1] / X[..., 2], X[..., 2]
        u, w = fx * x + cx, fy * y + cy
        ok = (Z > self.f.lm["z_min"]) & (u >= 0) & (u <= L.W - 1) & (w >= 0) & (w <= L.H - 1)
        u, w = torch.where(ok, u, 0.0), torch.where(ok, w, 0.0)
        x, y, Z = torch.where(ok, x, 0.0), torch.where(ok, y, 0.0), torch.where(ok, Z, 1.0)
        x0, y0 = u.long().clamp_max(L.W - 2), w.long().clamp_max(L.H - 2)
        a, b = (u - x0)[..., None], (w - y0)[..., None]
        c = y0 * L.W + x0
        f00, f10, f01, f11 = v.F[c], v.F[c + 1], v.F[c + L.W], v.F[c + L.W + 1]
        Fu, Fv = (1 - b) * (f10 - f00) + b * (f11 - f01), (1 - a) * (f01 - f00) + a * (f11 - f10)
        r = (1 - b) * ((1 - a) * f00 + a * f10) + b * ((1 - a) * f01 + a * f11) - v.ref[None]
        del f00, f10, f01, f11
        m = [(p * q).sum(-1) for p, q in ((Fu, Fu), (Fu, Fv), (Fv, Fv), (Fu, r), (Fv, r), (r, r))]
        wt = v.w[None].expand_as(u)
        if v.q is not None:
            a, b = a[..., 0], b[..., 0]
            wq = (1 - b) * ((1 - a) * v.q[c] + a * v.q[c + 1]) + b * ((1 - a) * v.q[c + L.W] + a * v.q[c + L.W + 1])
            wt = torch.where(ok, wt * wq, wt)
        rho, d = _rho(L.loss[0], L.loss[1], torch.where(ok, wt * m[5], 2 * wt))
        W = torch.where(ok, d * wt, 0.0)
        o, z = torch.zeros_like(x), 1 / Z
        Ju = fx * torch.stack([z, o, -x * z, -x * y, 1 + x * x, -y], -1)
        Jv = fy * torch.stack([o, z, -y * z, -1 - y * y, x * y, x], -1)
        Qu = (W * m[0])[..., None] * Ju + (W * m[1])[..., None] * Jv
        Qv = (W * m[1])[..., None] * Ju + (W * m[2])[..., None] * Jv
        H = torch.matmul(Ju.transpose(1, 2).contiguous(), Qu) + torch.matmul(Jv.transpose(1, 2).contiguous(), Qv)
        g = (Ju * (W * m[3])[..., None] + Jv * (W * m[4])[..., None]).sum(1)
        return H, g, rho.sum(1), ok.sum(1)

    def priors(self, T):
        """Per prior: J^T J and J^T r with the loss weight, the loss, |r|, |weight J^T r|."""
        f, D = self.f, self.dsm
        R, t = T[:, :9].view(-1, 3, 3), T[:, 9:]
        gc = R @ torch.tensor(f.g_world, dtype=torch.float64, device="cuda")
        r = gc - _f64(f.g_imu)
        rho, d = _rho(*f.gravity_loss, (r * r).sum(1))
        J = torch.zeros((len(T), 3, 6), dtype=torch.float64, device="cuda")
        J[:, 0, 4], J[:, 0, 5], J[:, 1, 3] = gc[:, 2], -gc[:, 1], -gc[:, 2]
        J[:, 1, 5], J[:, 2, 3], J[:, 2, 4] = gc[:, 0], gc[:, 1], -gc[:, 0]
        out = [(J, r, rho, d)]
        fx, fy, cx, cy = f.levels[-1].K
        q = np.array([(f.pc[0] - cx) / fx, (f.pc[1] - cy) / fy, 1.0])
        q = _f64(f.d_range * q / np.linalg.norm(q))
        P = ((q - t)[:, None] @ R)[:, 0]
        fj, fi = (P[:, 0] - f.dsm.x0) / f.dsm.gsd, (P[:, 1] - f.dsm.y0) / f.dsm.gsd
        Hd, Wd = D.shape
        cj, ci = (fj >= 0) & (fj <= Wd - 1), (fi >= 0) & (fi <= Hd - 1)
        fj, fi = fj.clamp(0, Wd - 1), fi.clamp(0, Hd - 1)
        j, i = fj.long().clamp_max(Wd - 2), fi.long().clamp_max(Hd - 2)
        a, b = fj - j, fi - i
        top, bot = D[i, j] * (1 - a) + D[i, j + 1] * a, D[i + 1, j] * (1 - a) + D[i + 1, j + 1] * a
        hx = ((1 - b) * (D[i, j + 1] - D[i, j]) + b * (D[i + 1, j + 1] - D[i + 1, j])) / f.dsm.gsd * cj
        hy = (bot - top) / f.dsm.gsd * ci
        n = torch.stack([-hx, -hy, torch.ones_like(hx)], 1)
        Rn = (R @ n[..., None])[..., 0]
        J = torch.cat([-Rn, torch.linalg.cross(Rn, q.expand_as(Rn))], 1)[:, None]
        r = (P[:, 2] - (1 - b) * top - b * bot)[:, None]
        rho, d = _rho(*f.range_loss, (r * r).sum(1))
        return out + [(J, r, rho, d)]

    def scales(self, T, gv):
        f = self.f
        al = torch.tensor([[f.lambda_imu, f.lambda_range]], dtype=torch.float64, device="cuda").repeat(len(T), 1)
        if f.adaptive_priors:
            nv = gv.norm(dim=1)
            for k, ((J, r, _, d), gate) in enumerate(zip(self.priors(T), (f.gravity_gate, f.range_gate))):
                gn = (d[:, None] * (J * r[..., None]).sum(1)).norm(dim=1) * al[:, k]
                rn, base = r.norm(dim=1), al[:, k].clone()
                base = torch.where(gn > f.alpha_ratio * nv, base * f.alpha_ratio * nv / gn.clamp_min(1e-300), base)
                al[:, k] = torch.where(rn > gate, base * (gate / rn.clamp_min(1e-300)) ** 2, base)
        return al

    def total(self, l, T, al=None):
        H, g, cost, n = self.photo(l, T)
        if al is None:
            al = self.scales(T, g)
        for k, (J, r, rho, d) in enumerate(self.priors(T)):
            W = al[:, k] * d
            H = H + W[:, None, None] * torch.matmul(J.transpose(1, 2).contiguous(), J)
            g = g + W[:, None] * (J * r[..., None]).sum(1)
            cost = cost + al[:, k] * rho
        return H, g, cost, n, al


def _exp(xi):
    w = xi[:, 3:]
    t2 = (w * w).sum(1)[:, None, None]
    t = t2.sqrt().clamp_min(1e-150)
    small = t2 < 1e-8
    A = torch.where(small, 1 - t2 / 6, torch.sin(t) / t)
    B = torch.where(small, 0.5 - t2 / 24, (1 - torch.cos(t)) / t2.clamp_min(1e-300))
    G = torch.where(small, 1 / 6 - t2 / 120, (t - torch.sin(t)) / (t2 * t).clamp_min(1e-300))
    o = torch.zeros_like(w[:, 0])
    K = torch.stack([o, -w[:, 2], w[:, 1], w[:, 2], o, -w[:, 0], -w[:, 1], w[:, 0], o], 1).view(-1, 3, 3)
    I, KK = torch.eye(3, dtype=torch.float64, device="cuda"), K @ K
    return I + A * K + B * KK, ((I + B * K + G * KK) @ xi[:, :3, None])[..., 0]


def _solve_exact(f, bf16):
    """The coarse-to-fine LM of every hypothesis at once, in FP64."""
    E, lm = _Exact(f, bf16), f.lm
    T = _f64(f.poses)
    M = len(T)
    cost = torch.full((M,), math.nan, dtype=torch.float64, device="cuda")
    alpha = torch.tensor([[f.lambda_imu, f.lambda_range]], dtype=torch.float64, device="cuda").repeat(M, 1)
    live = torch.arange(M, device="cuda")
    for l, L in enumerate(f.levels):
        H, g, c, n, al = E.total(l, T[live])
        cost[live], alpha[live] = c, al
        D = H.diagonal(dim1=1, dim2=2).amax(1)
        good = (n >= lm["min_valid"]) & torch.isfinite(c) & (D > 0)
        live, H, g, D = live[good], H[good], g[good], D[good]
        lam, lo, hi = lm["tau"] * D, lm["lambda_min_rel"] * D, lm["lambda_max_rel"] * D
        on = torch.ones(len(live), dtype=torch.bool, device="cuda")
        it = torch.zeros(len(live), dtype=torch.long, device="cuda")
        dx = torch.zeros_like(g)
        Tc = T[live].clone()
        while True:
            todo = on.clone()                       # propose: failed factorisations use up iterations
            while todo.any():
                on &= ~(todo & (it >= L.iters))
                todo &= on
                it += todo
                A = H + lam[:, None, None] * torch.eye(6, dtype=torch.float64, device="cuda")
                c6, info = torch.linalg.cholesky_ex(A)
                ok = todo & (info == 0)
                step = torch.cholesky_solve(-g[..., None], c6)[..., 0]
                dx = torch.where(ok[:, None], step, dx)
                bad = todo & ~ok
                lam = torch.where(bad, lam * lm["up"], lam)
                on &= ~(bad & (lam >= hi))
                todo = bad & on
            k = on.nonzero()[:, 0]
            if not len(k):
                break
            h = live[k]
            Re, te = _exp(dx[k])
            R, t = T[h, :9].view(-1, 3, 3), T[h, 9:]
            Tc[k] = torch.cat([(Re @ R).reshape(-1, 9), (Re @ t[..., None])[..., 0] + te], 1)
            Hc, gc, cc, _, _ = E.total(l, Tc[k], alpha[h])
            old = cost[h]
            flat = (cc - old).abs() <= lm["cost_tol"] * old
            take = cc < old
            tiny = (dx[k, :3].norm(dim=1) < lm["step_tol_t"]) & (dx[k, 3:].norm(dim=1) < lm["step_tol_r"])
            a = k[take]
            T[live[a]], H[a], g[a], cost[live[a]] = Tc[a], Hc[take], gc[take], cc[take]
            lam[k] = torch.where(take, torch.maximum(lam[k] / lm["down"], lo[k]), lam[k] * lm["up"])
            on[k] = ~(flat | (take & tiny) | (~take & (lam[k] >= hi[k])))
        if f.keep_top and l == f.prune_level:
            order = torch.sort(cost[live], stable=True).indices[: f.keep_top]
            live = live[order.sort().values]
    return dict(poses=T, cost=cost, alpha=alpha, iterations=None, status=None, best=None)


def _lift_exact(case, seed):
    s = prepare(case, seed)

    def sample(F, u, v):
        H, W = F.shape[:2]
        u, v = u.clamp(0, W - 1), v.clamp(0, H - 1)
        i, j = u.long().clamp_max(W - 2), v.long().clamp_max(H - 2)
        a, b = (u - i)[:, None], (v - j)[:, None]
        F = F.to(torch.float64)
        return (1 - b) * ((1 - a) * F[j, i] + a * F[j, i + 1]) + b * ((1 - a) * F[j + 1, i] + a * F[j + 1, i + 1])

    u, v = s.uv[:, 0].double(), s.uv[:, 1].double()
    out = []
    for k, (F, scale) in enumerate(s.maps):
        ref = sample(F, scale * (u + 0.5) - 0.5, scale * (v + 0.5) - 0.5)
        out.append(dict(ref=ref) if k else dict(
            ref=ref, x=s.at[0] + u * s.at[2], y=s.at[1] + v * s.at[2], z=sample(s.dsm[..., None], u, v)[:, 0]))
    return out


def exact(case, seed):
    if case["kind"] == "lift":
        return _lift_exact(case, seed)
    if case["kind"] == "batch":                     # over half a minute
        return None
    frames = [_frame(c, seed * 64 + k) for k, c in enumerate(_cases_of(case))]
    if case["kind"] == "linearize":
        f = frames[0]
        H, g, cost, _, _ = _Exact(f, case["bf16"]).total(case["levels"] - 1, _f64(f.poses), _f64(
            np.array([[f.lambda_imu, f.lambda_range]])).repeat(len(f.poses), 1))
        i = torch.triu_indices(6, 6)
        return dict(H=H[:, i[0], i[1]], g=g, cost=cost, n=None)
    return [_solve_exact(f, case["bf16"]) for f in frames]
