"""Performance cases of the keyframe depth update: what a program that uses this library has it do.

A case names a kind of work and its settings:

- "life":   one keyframe's life as a camera stream runs it: a new prior, the following frames fused one by
            one, the depth map read out at the end (kf_set_prior, kf_fuse_frame x frames, kf_read_depth);
- "solve":  the optimisation alone from a semi-dense state that the caller brings (kf_import_state, kf_solve);
- "batch":  many keyframes of mixed sizes, each fused with one new frame per call (kf_batch_fuse);
- "subset": the call a serving loop makes, a frame for whichever members have one (kf_batch_fuse_subset);
- "init":   a new keyframe from the network's outputs at the network's resolution, and its read-out
            (kf_set_prior_network, kf_read_depth).

Inputs are rendered here on the GPU: three slanted planes before a background, value-noise texture, a
small camera walk, and noisy priors around the true log-depth, as in the repository's synthetic scenes.
`exact` repeats a case in 64 bits with plain torch.
"""
import math

import numpy as np
import torch

from paper_2207_12244_amd import autotune
from paper_2207_12244_amd.kf import Batch, Keyframe

D_NEAR, D_FAR, GATE, SIGMA_PHOTO, R_FLOOR, DELTA = 0.4, 10.0, 6.0, 1.0, 1e-6, 1.345
MIX64 = "160x120:14,320x240:22,512x384:16,640x480:12"     # the 64-keyframe batched workload
MIX32 = "320x240:11,512x384:8,640x480:13"                  # the 32-stream serving workload
TEXTURED = 0.31                                            # share of pixels with enough texture to be searched


def listed():
    return [
        # the smallest call: a thumbnail keyframe and one frame, all latency
        dict(name="life-64x48-f32", kind="life", W=64, H=48, frames=1, precision="f32", pattern="line5", ns=32),
        # the plain FP64 form, solved to a tolerance
        dict(name="life-160x120-f64-rtol", kind="life", W=160, H=120, frames=1, precision="f64", pattern="line5",
             ns=32, rtol=1e-12),
        # a small camera with an odd image size; Tukey's cost
        dict(name="life-333x251-f32-tukey", kind="life", W=333, H=251, frames=5, precision="f32", pattern="line5",
             ns=64, robust="tukey"),
        # quarter VGA, a keyframe of ten frames
        dict(name="life-320x240-f32", kind="life", W=320, H=240, frames=10, precision="f32", pattern="sq5x5", ns=64),
        # VGA in the precision form, thirty frames, the next frame's search beside the solve
        dict(name="life-640x480-bf16-piped", kind="life", W=640, H=480, frames=30, precision="bf16",
             pattern="sq5x5", ns=128, pipeline=True),
        # VGA one frame at a time, as a tracker does that reads every depth map
        dict(name="life-640x480-f32-one", kind="life", W=640, H=480, frames=1, precision="f32", pattern="sq5x5",
             ns=64),
        # a large camera
        dict(name="life-1280x960-f32", kind="life", W=1280, H=960, frames=2, precision="f32", pattern="line5", ns=64),
        # the optimisation alone: an application with its own depth measurements, many or few iterations
        dict(name="solve-640x480-f32", kind="solve", W=640, H=480, precision="f32"),
        dict(name="solve-97x61-f32-3x15", kind="solve", W=97, H=61, precision="f32", n_gn=3, n_cg=15),
        # many keyframes at once
        dict(name="batch-64-mixed-bf16", kind="batch", mix=MIX64, frames=4, precision="bf16", pattern="line5", ns=32),
        # a serving loop at moderate load
        dict(name="subset-6-of-32-f32", kind="subset", mix=MIX32, frames=8, active=6, precision="f32",
             pattern="sq5x5", ns=64),
        # a new keyframe
        dict(name="init-640x480-f32", kind="init", W=640, H=480, precision="f32", net_W=256, net_H=192),
    ]


def _size(rng, lo, hi):
    """Width log-uniform in [lo, hi], any aspect from 1:1 to 16:9, odd sizes among them, at most 1280 x 960 pixels."""
    W = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return W, min(max(16, int(round(W / rng.uniform(1.0, 1.78)))), 1280 * 960 // W)


def draw(rng):
    kind = rng.choice(["life", "life", "life", "solve", "solve", "batch", "subset", "init"])
    precision = rng.choice(["f32", "f32", "bf16"])
    pattern = rng.choice(["line5", "sq5x5"])
    ns = rng.choice([16, 32, 64, 128])
    if kind == "life":
        if rng.random() < 0.15:
            W, H = _size(rng, 48, 240)
            return dict(kind=kind, W=W, H=H, frames=1, precision="f64", pattern="line5", ns=32, rtol=1e-12)
        W, H = _size(rng, 48, 1280)
        c = dict(kind=kind, W=W, H=H, frames=rng.choice([1, 2, 4, 8]), precision=precision, pattern=pattern, ns=ns)
        if rng.random() < 0.2:
            c["pipeline"] = True
        if rng.random() < 0.2:
            c["robust"] = "tukey"
        return c
    if kind == "solve":
        W, H = _size(rng, 48, 1280)
        return dict(kind=kind, W=W, H=H, precision="f32", n_gn=rng.randint(3, 12), n_cg=rng.randint(10, 30))
    if kind == "init":
        W, H = _size(rng, 160, 1280)
        return dict(kind=kind, W=W, H=H, precision=precision, net_W=256, net_H=192)
    parts = []
    for W, H in rng.sample([(160, 120), (200, 130), (320, 240), (424, 240), (512, 384), (640, 480)], 3):
        parts.append("%dx%d:%d" % (W, H, rng.randint(2, 8)))
    c = dict(kind=kind, mix=",".join(parts), frames=rng.choice([2, 4]), precision=precision, pattern=pattern, ns=ns)
    if kind == "subset":
        c["active"] = rng.randint(1, 6)
    return c


# ---------------------------------------------------------------- scenes

class Scene:
    """Three slanted planes before a fronto-parallel background, value-noise texture."""

    def __init__(self, seed):
        self.rng = np.random.default_rng(seed)
        g = torch.Generator(device="cuda")
        g.manual_seed(int(self.rng.integers(1 << 40)))
        self.gen = g
        self.lattice = torch.rand((4, 4, 256, 256), generator=g, device="cuda", dtype=torch.float64)
        self.planes = []
        for _ in range(3):
            th, ph, d = self.rng.uniform(0, math.radians(40)), self.rng.uniform(0, 2 * math.pi), self.rng.uniform(1.2, 3.0)
            R = rotation(th * np.array([math.cos(ph), math.sin(ph), 0.0]))
            self.planes.append((R, np.array([0.0, 0.0, d])))
        self.planes.append((np.eye(3), np.array([0.0, 0.0, 4.0])))

    def cast(self, K, T, u, v):
        rays = torch.stack([(u - K[0, 2]) / K[0, 0], (v - K[1, 2]) / K[1, 1], torch.ones_like(u)], -1)
        R, c = torch.as_tensor(T[:3, :3], device="cuda"), torch.as_tensor(T[:3, 3], device="cuda")
        rw = rays @ R.T
        best = torch.full_like(u, 1e9)
        val = torch.zeros_like(u)
        s = torch.zeros_like(u)
        t = torch.zeros_like(u)
        idx = torch.zeros_like(u, dtype=torch.long)
        for j, (P, p0) in enumerate(self.planes):
            P, p0 = torch.as_tensor(P, device="cuda"), torch.as_tensor(p0, device="cuda")
            lam = ((p0 - c) @ P[:, 2]) / (rw @ P[:, 2])
            hit = (lam > 0.5) & (lam < best)
            best = torch.where(hit, lam, best)
            X = (c + lam[..., None] * rw - p0) @ P
            s, t, idx = torch.where(hit, X[..., 0], s), torch.where(hit, X[..., 1], t), torch.where(hit, j, idx)
        norm = 0.0
        for o in range(4):
            a, b = s * (2.0 ** o / 0.25), t * (2.0 ** o / 0.25)
            i, j = torch.floor(a), torch.floor(b)
            f, g = a - i, b - j
            f, g = f * f * (3 - 2 * f), g * g * (3 - 2 * g)
            i, j = i.long(), j.long()
            L = self.lattice[o]
            at = lambda x, y: L[idx, y % 256, x % 256]  # noqa: E731
            val += 0.5 ** o * ((1 - g) * ((1 - f) * at(i, j) + f * at(i + 1, j)) + g * ((1 - f) * at(i, j + 1) + f * at(i + 1, j + 1)))
            norm += 0.5 ** o
        return best, val / norm

    def view(self, K, T, W, H):
        """(uint8 image, depth), the image 2 x 2 supersampled."""
        v, u = torch.meshgrid(torch.arange(H, device="cuda", dtype=torch.float64),
                              torch.arange(W, device="cuda", dtype=torch.float64), indexing="ij")
        depth, _ = self.cast(K, T, u, v)
        acc = sum(self.cast(K, T, u + du, v + dv)[1] for du in (-0.25, 0.25) for dv in (-0.25, 0.25)) / 4
        return torch.clamp(torch.round(127.5 + 510.0 * (acc - 0.5)), 0, 255).to(torch.uint8), depth

    def walk(self, frames):
        poses = []
        unit = lambda x: x / np.linalg.norm(x)  # noqa: E731
        u, a, t, R = unit(self.rng.standard_normal(3)), unit(self.rng.standard_normal(3)), np.zeros(3), np.eye(3)
        step, turn = (0.05, 1.0) if frames == 1 else (0.02, 0.5)
        for _ in range(frames):
            u, a = unit(u + 0.3 * self.rng.standard_normal(3)), unit(a + 0.3 * self.rng.standard_normal(3))
            t, R = t + step * u, R @ rotation(math.radians(turn) * a)
            T = np.eye(4)
            T[:3, :3], T[:3, 3] = R, t
            poses.append(T)
        return poses

    def priors(self, depth, dtype):
        """The network's stand-in: log-depth and forward-difference gradients with noise of known variance."""
        def noisy(x, lo, hi):
            sg = torch.exp(torch.rand(x.shape, generator=self.gen, device="cuda", dtype=torch.float64) * math.log(hi / lo) + math.log(lo))
            n = torch.randn(x.shape, generator=self.gen, device="cuda", dtype=torch.float64)
            return [(x + sg * n).to(dtype), (sg * sg).to(dtype)]
        x = torch.log(depth)
        gx, gy = torch.zeros_like(x), torch.zeros_like(x)
        gx[:, :-1], gy[:-1] = x[:, 1:] - x[:, :-1], x[1:] - x[:-1]
        return noisy(x, 0.02, 0.3) + noisy(gx, 0.01, 0.2) + noisy(gy, 0.01, 0.2)


def rotation(w):
    th = float(np.linalg.norm(w))
    if th < 1e-15:
        return np.eye(3)
    k = np.asarray(w) / th
    X = np.array([[0, -k[2], k[1]], [k[2], 0, -k[0]], [-k[1], k[0], 0]])
    return np.eye(3) + math.sin(th) * X + (1 - math.cos(th)) * (X @ X)


def camera(W, H):
    return np.array([[0.8 * W, 0.0, W / 2.0], [0.0, 0.8 * W, H / 2.0], [0.0, 0.0, 1.0]])


def _map_type(case):
    return torch.float64 if case["precision"] == "f64" else torch.float32


def _stream(case, W, H, seed):
    """One keyframe's inputs: image, priors, and the frames that follow with their poses."""
    sc = Scene(seed)
    K = camera(W, H)
    image0, depth = sc.view(K, np.eye(4), W, H)
    poses = sc.walk(case["frames"])
    return dict(W=W, H=H, K=K, image0=image0, priors=sc.priors(depth, _map_type(case)), poses=poses,
                images=[sc.view(K, T, W, H)[0] for T in poses])


def _semi_dense(case, seed):
    """A solver's inputs: image, priors, and inverse depths with variances on the textured third of the pixels."""
    W, H, dt = case["W"], case["H"], _map_type(case)
    sc = Scene(seed)
    K = camera(W, H)
    image0, depth = sc.view(K, np.eye(4), W, H)
    pri = sc.priors(depth, dt)
    r = lambda: torch.rand((H, W), generator=sc.gen, device="cuda", dtype=torch.float64)  # noqa: E731
    sd = torch.exp(r() * math.log(20.0) + math.log(0.005))
    noise = torch.randn((H, W), generator=sc.gen, device="cuda", dtype=torch.float64)
    has = r() < TEXTURED
    rho = (1.0 / (0.97 * depth)) * (1.0 + sd * noise).clamp(0.5, 2.0)
    zero = torch.zeros_like(rho)
    return dict(W=W, H=H, K=K, image0=image0, priors=pri, rho=torch.where(has, rho, zero).to(dt),
                var=torch.where(has, (sd * rho) ** 2, zero).to(dt))


def _mix(case):
    out = []
    for part in case["mix"].split(","):
        size, n = part.split(":")
        out += [tuple(int(x) for x in size.split("x"))] * int(n)
    return out


# ---------------------------------------------------------------- one pass

def _keyframe(case, W, H, K, **kw):
    robust = case.get("robust", "huber")
    return Keyframe(W, H, precision=case["precision"], pattern=case.get("pattern", "line5"),
                    n_samples=case.get("ns", 32), n_gn=case.get("n_gn", 10), n_cg=case.get("n_cg", 20),
                    cg_rtol=case.get("rtol", 0.0), K=K, robust=robust,
                    huber_delta=4.685 if robust == "tukey" else DELTA,
                    pipeline_frames=case.get("pipeline", False), **kw)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("life", "solve"):
        s = _stream(case, case["W"], case["H"], seed) if kind == "life" else _semi_dense(case, seed)
        return dict(case=case, kf=_keyframe(case, s["W"], s["H"], s["K"]), s=s)
    if kind == "init":
        W, H, nW, nH = case["W"], case["H"], case["net_W"], case["net_H"]
        sc = Scene(seed)
        _, depth = sc.view(camera(nW, nH), np.eye(4), nW, nH)
        image0, _ = sc.view(camera(W, H), np.eye(4), W, H)
        return dict(case=case, kf=_keyframe(case, W, H, camera(W, H)), image0=image0,
                    priors=sc.priors(depth, _map_type(case)))
    # the tile policy of a batch is tuned once per device and mix; these are the tuner's choices for the listed mixes
    members, streams = [], []
    for i, (W, H) in enumerate(_mix(case)):
        s = _stream(case, W, H, 1000 * seed + i)
        tiles = autotune.tiles_for(W, H, 512, 10) if kind == "batch" else (0, 0)
        members.append(_keyframe(case, W, H, s["K"], tiles=tiles, solver_threads=512))
        streams.append(s)
    st = dict(case=case, members=members, streams=streams, batch=Batch(members))
    if kind == "subset":
        rng = np.random.default_rng(seed)
        st["plan"] = [sorted(rng.choice(len(members), case["active"], replace=False).tolist())
                      for _ in range(case["frames"])]
    return st


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "life":
        kf, s = state["kf"], state["s"]
        kf.set_prior(s["image0"], *s["priors"], np.eye(4))
        for image, T in zip(s["images"], s["poses"]):
            kf.fuse_frame(image, T)
        depth, scale, var = kf.read_depth(with_var=True)
        return [depth, scale, var]
    if kind == "solve":
        kf, s = state["kf"], state["s"]
        kf.set_prior(s["image0"], *s["priors"], np.eye(4))
        kf.import_state(rho=s["rho"], var=s["var"])
        kf.solve()
        depth, scale = kf.read_depth()
        return [depth, scale]
    if kind == "init":
        kf = state["kf"]
        kf.set_prior_network(state["image0"], *state["priors"], np.eye(4), focal_ref=0.75 * case["net_W"])
        depth, scale = kf.read_depth()
        return [depth, scale]
    for kf, s in zip(state["members"], state["streams"]):
        kf.set_prior(s["image0"], *s["priors"], np.eye(4))
    for f in range(case["frames"]):
        if kind == "batch":
            state["batch"].fuse([s["images"][f] for s in state["streams"]], [s["poses"][f] for s in state["streams"]])
        else:
            act = state["plan"][f]
            state["batch"].fuse_subset(act, [state["streams"][i]["images"][f] for i in act],
                                       [state["streams"][i]["poses"][f] for i in act])
    maps = [kf.read_depth() for kf in state["members"]]
    return [torch.cat([d.flatten() for d, _ in maps]), np.array([s for _, s in maps])]


def work(case):
    """Bytes: every image, prior and state word read once and every result written once per frame. Flops: the
    searches' bilinear points and squared differences, the assembly, and the CG iterations' stencil, updates and dots."""
    kind = case["kind"]
    word = 8 if case["precision"] == "f64" else 4
    if kind == "init":
        n, m = case["W"] * case["H"], case["net_W"] * case["net_H"]
        return dict(bytes=n * (1 + 9 * word) + 6 * m * word, flops=n * 90)
    points = {"line5": 5, "sq5x5": 25}[case.get("pattern", "line5")]
    per_sample = points * 10 + 20
    cg = 82 * 10 if case.get("rtol") else case.get("n_gn", 10) * case.get("n_cg", 20)
    per_solve = cg * 22 + case.get("n_gn", 10) * 120
    if kind == "solve":
        n = case["W"] * case["H"]
        return dict(bytes=n * (1 + 6 * word + 2 * word + 2 * word), flops=n * per_solve)
    sizes = [(case["W"], case["H"])] if kind == "life" else _mix(case)
    px = sum(W * H for W, H in sizes)
    fused = px * case["frames"]
    if kind == "subset":
        fused *= case["active"] / len(sizes)
    return dict(bytes=px * (1 + 6 * word + word) + fused * (1 + 2 * word + 4 * word * TEXTURED),
                flops=fused * (TEXTURED * case["ns"] * per_sample + per_solve))


# ---------------------------------------------------------------- the same in 64 bits, plain torch

def _bilinear(img, u, v):
    H, W = img.shape
    i, j = torch.clamp(torch.floor(u), 0, W - 2), torch.clamp(torch.floor(v), 0, H - 2)
    f, g = u - i, v - j
    at = (j * W + i).long()
    flat = img.reshape(-1)
    return (1 - g) * ((1 - f) * flat[at] + f * flat[at + 1]) + g * ((1 - f) * flat[at + W] + f * flat[at + W + 1])


def _search(s, rho, var, pix, image, T, ns, pattern):
    """One frame's epipolar search of the textured pixels `pix`: (inverse depth, variance, measured)."""
    H, W = rho.shape
    rel = np.linalg.inv(T)
    K = s["K"]
    KR = K @ rel[:3, :3]
    Hm, b, e0 = KR @ np.linalg.inv(K), K @ rel[:3, 3], K @ (-rel[:3, :3].T @ rel[:3, 3])
    I0, I1 = s["image0"].double(), image.double()
    u, v = (pix % W).double(), (pix // W).double()
    r, w = rho.reshape(-1)[pix], var.reshape(-1)[pix]
    has, sd = w > 0, torch.sqrt(w)
    lo_all, hi_all = torch.full_like(r, 1 / D_FAR), torch.full_like(r, 1 / D_NEAR)
    lo = torch.where(has, torch.maximum(r - 2 * sd, lo_all), lo_all)
    hi = torch.where(has, torch.minimum(r + 2 * sd, hi_all), hi_all)
    A = [Hm[k, 0] * u + Hm[k, 1] * v + Hm[k, 2] for k in range(3)]
    proj = lambda q: ((A[0] + q * b[0]) / (A[2] + q * b[2]), (A[1] + q * b[1]) / (A[2] + q * b[2]))  # noqa: E731
    ok = (hi > lo) & (A[2] + lo * b[2] > 0) & (A[2] + hi * b[2] > 0)
    (ax, ay), (cx, cy) = proj(lo), proj(hi)
    L = torch.hypot(cx - ax, cy - ay)
    ok &= torch.isfinite(L) & (L >= 1e-6)
    lx, ly = torch.where(ok, (cx - ax) / L, 1.0), torch.where(ok, (cy - ay) / L, 0.0)
    step = torch.where(ok, torch.clamp(L / (ns - 1), min=1.0), 1.0)
    mx, my = torch.where(ok, (ax + cx) / 2, u), torch.where(ok, (ay + cy) / 2, v)
    if pattern == "line5":
        dx, dy = e0[2] * u - e0[0], e0[2] * v - e0[1]
        n0 = torch.hypot(dx, dy)
        l0x, l0y = dx / n0, dy / n0
        mid = (lo + hi) / 2
        q0 = proj(mid)
        B = [A[k] + Hm[k, 0] * l0x + Hm[k, 1] * l0y + mid * b[k] for k in range(3)]
        flip = ((B[0] / B[2] - q0[0]) * lx + (B[1] / B[2] - q0[1]) * ly) < 0
        sg = torch.where(flip, -1.0, 1.0)
        good = torch.isfinite(l0x) & torch.isfinite(l0y)
        ok &= good
        l0x, l0y = torch.where(good, sg * l0x, 0.0), torch.where(good, sg * l0y, 0.0)
        pts = [(j * lx, j * ly) for j in range(-2, 3)]
        pat = [_bilinear(I0, u + j * l0x, v + j * l0y) for j in range(-2, 3)]
    else:
        pts = [(torch.full_like(u, m), torch.full_like(u, n)) for n in range(-2, 3) for m in range(-2, 3)]
        pat = [I0.reshape(-1)[((v + n) * W + u + m).long()] for n in range(-2, 3) for m in range(-2, 3)]
    use_x = lx.abs() >= ly.abs()
    Am, bm = torch.where(use_x, A[0], A[1]), torch.where(use_x, b[0], b[1])

    def sample(k):
        px, py = mx + (k - (ns - 1) / 2) * step * lx, my + (k - (ns - 1) / 2) * step * ly
        pm = torch.where(use_x, px, py)
        return px, py, (pm * A[2] - Am) / (bm - pm * b[2])

    def residuals(px, py):
        return [_bilinear(I1, torch.clamp(px + ox, 0, W - 1), torch.clamp(py + oy, 0, H - 1)) - p for (ox, oy), p in zip(pts, pat)]

    ssd = torch.full((ns, pix.numel()), math.inf, device="cuda", dtype=torch.float64)
    for k in range(ns):
        px, py, rk = sample(k)
        fine = ok & torch.isfinite(rk) & (rk >= 1 / D_FAR) & (rk <= 1 / D_NEAR)
        for ox, oy in (pts[0], pts[4], pts[-5], pts[-1]):
            fine &= (px + ox >= 0) & (px + ox <= W - 1) & (py + oy >= 0) & (py + oy <= H - 1)
        px, py = torch.where(fine, px, u), torch.where(fine, py, v)
        ssd[k] = torch.where(fine, sum(e * e for e in residuals(px, py)), math.inf)
    best, kb = ssd.min(0)
    sm = torch.where(kb > 0, ssd.gather(0, (kb - 1).clamp(min=0)[None])[0], math.inf)
    sp = torch.where(kb < ns - 1, ssd.gather(0, (kb + 1).clamp(max=ns - 1)[None])[0], math.inf)
    nb = torch.where(sm <= sp, kb - 1, kb + 1)
    ok &= torch.isfinite(best) & (torch.isfinite(sm) | torch.isfinite(sp))
    xk, yk, rk = sample(kb.double())
    xn, yn, rn = sample(nb.double())
    ek, en = residuals(xk, yk), residuals(xn, yn)
    dd = sum((q - p) ** 2 for p, q in zip(ek, en))
    lam = torch.clamp(-sum(p * (q - p) for p, q in zip(ek, en)) / dd, 0, 1)
    da, db = 1 / rk, 1 / rn
    d = da + lam * (db - da)
    vd = SIGMA_PHOTO ** 2 * (db - da) ** 2 / dd
    vo = vd / d ** 4
    ok &= (dd > 0) & torch.isfinite(vd) & (vd > 0) & torch.isfinite(d) & (d > 0) & torch.isfinite(vo) & (vo > 0)
    ro = 1 / d
    fr, fv = torch.where(has, (vo * r + w * ro) / (w + vo), ro), torch.where(has, w * vo / (w + vo), vo)
    rho, var = rho.clone(), var.clone()
    rho.view(-1)[pix[ok]], var.view(-1)[pix[ok]] = fr[ok], fv[ok]
    return rho, var


def _textured(image0):
    I = image0.double()
    a, b = torch.zeros_like(I), torch.zeros_like(I)
    a[:, 1:-1], b[1:-1] = (I[:, 2:] - I[:, :-2]) / 2, (I[2:] - I[:-2]) / 2
    m = a * a + b * b >= GATE * GATE
    m[:2], m[-2:], m[:, :2], m[:, -2:] = False, False, False, False
    return torch.nonzero(m.reshape(-1))[:, 0]


def _solve(case, x, tau, priors, rho, var):
    """n_gn Gauss-Newton iterations, the depth step by Jacobi-preconditioned CG, then the scale."""
    mu, vn, gx, vx, gy, vy = priors
    tukey = case.get("robust") == "tukey"
    c = 4.685 if tukey else DELTA

    def weight(r, v):
        a = r.abs() / torch.sqrt(v)
        return (torch.where(a <= c, (1 - (a / c) ** 2) ** 2, 0.0) if tukey else torch.where(a <= c, 1.0, c / a)) / v

    has = var > 0
    q = torch.where(has, rho, 1.0)
    z, R = -torch.log(q), torch.where(has, torch.clamp(var / (q * q), min=R_FLOOR), 1.0)
    gx, vx, gy, vy = gx[:, :-1], vx[:, :-1], gy[:-1], vy[:-1]

    def spread(ex, ey, keep=1.0):
        """Adds an edge quantity to its two pixels (the second one times `keep`)."""
        o = torch.zeros_like(mu)
        o[:, :-1] += ex
        o[:, 1:] += keep * ex
        o[:-1] += ey
        o[1:] += keep * ey
        return o

    for _ in range(case.get("n_gn", 10)):
        wn, ws = weight(x - mu, vn), torch.where(has, weight(x - tau - z, R), 0.0)
        cx, cy = weight(x[:, 1:] - x[:, :-1] - gx, vx), weight(x[1:] - x[:-1] - gy, vy)
        diag = wn + ws + spread(cx, cy)
        rhs = wn * mu + ws * (tau + z) - spread(cx * gx, cy * gy, -1.0)

        def mul(p):
            o = diag * p
            o[:, :-1] -= cx * p[:, 1:]
            o[:, 1:] -= cx * p[:, :-1]
            o[:-1] -= cy * p[1:]
            o[1:] -= cy * p[:-1]
            return o

        inv = torch.where(diag > 0, 1 / diag, 0.0)
        r = rhs - mul(x)
        p = inv * r
        rz = (r * p).sum()
        tol = case.get("rtol", 0.0) * rhs.norm()
        for _ in range(4000 if case.get("rtol") else case.get("n_cg", 20)):
            if case.get("rtol") and r.norm() <= tol:
                break
            ap = mul(p)
            al = rz / (p * ap).sum()
            x = x + al * p
            r = r - al * ap
            y = inv * r
            rn = (r * y).sum()
            p = y + (rn / rz) * p
            rz = rn
        w = torch.where(has, weight(x - tau - z, R), 0.0)
        total = w.sum()
        tau = torch.where(total > 0, (w * (x - z)).sum() / torch.where(total > 0, total, 1.0), tau)
    return x, tau


def _life(case, s):
    pri = [m.double() for m in s["priors"]]
    x, tau = pri[0].clone(), torch.zeros((), device="cuda", dtype=torch.float64)
    rho, var = torch.zeros_like(x), torch.zeros_like(x)
    pix = _textured(s["image0"])
    for image, T in zip(s["images"], s["poses"]):
        rho, var = _search(s, rho, var, pix, image, T, case["ns"], case["pattern"])
        x, tau = _solve(case, x, tau, pri, rho, var)
    return torch.exp(x), math.exp(float(tau))


def exact(case, seed):
    kind = case["kind"]
    if kind in ("batch", "subset"):
        return None          # minutes in 64 bits
    if kind == "life":
        if case["W"] * case["H"] * case["frames"] * case["ns"] > 1e9:
            return None
        depth, scale = _life(case, _stream(case, case["W"], case["H"], seed))
        return [depth, scale, None]
    if kind == "solve":
        s = _semi_dense(case, seed)
        pri = [m.double() for m in s["priors"]]
        x, tau = _solve(case, pri[0].clone(), torch.zeros((), device="cuda", dtype=torch.float64), pri,
                        s["rho"].double(), s["var"].double())
        return [torch.exp(x), math.exp(float(tau))]
    W, H, nW, nH = case["W"], case["H"], case["net_W"], case["net_H"]
    sc = Scene(seed)
    _, depth = sc.view(camera(nW, nH), np.eye(4), nW, nH)
    sc.view(camera(W, H), np.eye(4), W, H)
    mu = sc.priors(depth, _map_type(case))[0].double()
    v, u = torch.meshgrid(torch.arange(H, device="cuda", dtype=torch.float64),
                          torch.arange(W, device="cuda", dtype=torch.float64), indexing="ij")
    x = _bilinear(mu, torch.clamp((u + 0.5) * nW / W - 0.5, 0, nW - 1), torch.clamp((v + 0.5) * nH / H - 0.5, 0, nH - 1))
    return [torch.exp(x + math.log(0.8 * W * (nW / W) / (0.75 * nW))), 1.0]
