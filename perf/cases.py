"""The work that users of the framework have it do, as cases that can be timed and compared.

Each case is one pass through the public entry points of ``paper_2002_00250_amd``:

* ``camera``      one model, device frames: push a frame, copy the mask into the caller's tensor;
* ``host``        one model, frames in host memory: push a frame, read the mask back to the host;
* ``fleet``       many models on one stream: one frame to each (``fgs.push_frames``);
* ``serve``       the multi-stream server: one frame of every stream in, every mask out;
* ``score``       a short sequence: push, mask out, median filter, evaluation and static counters;
* ``checkpoint``  push a frame, copy the whole state out, load it into a standby model;
* ``window``      the GMM adjoint over a window of frames: scores, loss, gradients.

Frames follow the repository's synthetic recipe (textured background, two depth planes, moving
rectangles, noise, depth holes), drawn on the GPU.  A state holds a ring of frames that is
walked one frame a pass (objects move to and fro, so the ring closes), and its models have seen
enough frames before the first pass to be past their initial transient, as a running camera is.
"""
import math
import random

import numpy as np
import torch

from paper_2002_00250_amd import fgs
from paper_2002_00250_amd.adjoint import GmmWindow, GmmWindowFunction, window_bce_loss
from paper_2002_00250_amd.serving import Server

GMM_FIELDS = ("alpha", "rho_mode", "decision", "var_mode")


# ---------------------------------------------------------------------------- the cases
def listed():
    return [
        # The smallest real camera: the 320x240 parity workload, K = 3.  Latency and launches count.
        dict(name="gmm_k3_240p", kind="camera", model="gmm3", H=240, W=320),
        # The paper's own system and largest resolution: Kc = 7, Kd = 3, alpha = 0.001,
        # 1920x1080 RGB with a 1280x720 depth map upscaled in the kernel.
        dict(name="gmm_7_3_1080p", kind="camera", model="gmm7/3", H=1080, W=1920, dH=720, dW=1280, alpha=0.001),
        # The method's variants (per-channel variances, rate alpha / w) at a ragged size.
        dict(name="gmm_k3_variants_ragged", kind="camera", model="gmm3", H=487, W=853, var_mode=1, rho_mode=1),
        # PBAS with the base method's gradient feature (opt-in) at its usual resolution.
        dict(name="pbas_gradient_480p", kind="camera", model="pbasg20", H=480, W=640),
        # A camera program that holds its frames in host memory and wants the mask there.
        dict(name="pbas_n20_480p_host", kind="host", model="pbas20", H=480, W=640),
        # The throughput workload, one launch per kind: 8 GMM K = 5 cameras at 1280x720 ...
        dict(name="gmm_k5_720p_x8", kind="fleet", models="8*gmm5@720x1280"),
        # ... and 4 PBAS N = 35 cameras at 1280x720.
        dict(name="pbas_n35_720p_x4", kind="fleet", models="4*pbas35@720x1280"),
        # The serving workload: 32 streams of three resolutions, half GMM K = 5, half PBAS N = 20.
        dict(name="serve_32_streams", kind="serve",
             models="6*gmm5@240x424,6*pbas20@240x424,6*gmm5@480x640,6*pbas20@480x640,"
                    "4*gmm5@720x1280,4*pbas20@720x1280"),
        # Scoring a sequence: mask, 9x9 median, evaluation and static-object counters per frame.
        dict(name="score_pbas_480p", kind="score", model="pbas20", H=480, W=640, frames=8, radius=4),
        # Checkpoint of a running camera and restore into a standby one, on the device.
        dict(name="checkpoint_pbas_480p", kind="checkpoint", model="pbas20", H=480, W=640),
        # A training step of the adjoint workload: 64 frames of 640x480, K = 3, forward, loss, backward.
        dict(name="window_k3_480p_t64", kind="window", K=3, H=480, W=640, T=64, every=16),
        # A short window on a small ragged crop with more Gaussians, where the chip is not full.
        dict(name="window_k5_crop_t24", kind="window", K=5, H=93, W=131, T=24, every=10),
    ]


def draw(rng):
    def size(lo, hi):  # rows log-uniform, sides odd as often as even
        H = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return H, max(8, int(H * rng.uniform(1.1, 1.8)))

    def gmm():
        return "gmm" + rng.choice(["1", "2", "3", "3", "4", "5", "5", "6", "7", "7/3"])

    def pbas():
        return "pbas%d" % rng.randint(2, 64)

    kind = rng.choice(["camera"] * 5 + ["host", "fleet", "fleet", "serve", "score", "checkpoint", "window", "window"])
    if kind == "camera":
        H, W = size(60, 1080)
        c = dict(kind=kind, model=rng.choice([gmm(), pbas(), "pbasg%d" % rng.randint(4, 40)]), H=H, W=W)
        if c["model"].startswith("gmm"):
            if rng.random() < 0.3:
                c.update(var_mode=rng.randint(0, 1), rho_mode=rng.randint(0, 1))
            if rng.random() < 0.3:
                c.update(dH=max(1, int(H * rng.uniform(0.4, 1.0))), dW=max(1, int(W * rng.uniform(0.4, 1.0))))
        return c
    if kind == "host":
        H, W = size(60, 720)
        return dict(kind=kind, model=rng.choice([gmm(), pbas()]), H=H, W=W)
    if kind == "fleet":
        H, W = size(120, 720)
        if rng.random() < 0.5:
            n, model = rng.randint(2, 8), rng.choice(["gmm3", "gmm5", "gmm7/3"])
            return dict(kind=kind, models="%d*%s@%dx%d" % (n, model, H, min(W, 1280)))
        return dict(kind=kind, models="%d*pbas%d@%dx%d" % (rng.randint(2, 5), rng.choice([20, 35]), H, min(W, 1280)))
    if kind == "serve":
        parts = []
        for model in ("gmm5", "pbas20"):
            H, W = size(120, 480)
            parts.append("%d*%s@%dx%d" % (rng.randint(2, 8), model, H, W))
        return dict(kind=kind, models=",".join(parts))
    if kind == "score":
        H, W = size(120, 720)
        return dict(kind=kind, model=rng.choice(["gmm3", "gmm5", "pbas20"]), H=H, W=W, frames=rng.randint(4, 8),
                    radius=rng.randint(1, 7))
    if kind == "checkpoint":
        H, W = size(120, 480)
        return dict(kind=kind, model=rng.choice(["gmm3", "gmm5", "pbas20", "pbasg20"]), H=H, W=W)
    H, W = size(48, 480)
    return dict(kind=kind, K=rng.randint(1, 5), H=H, W=min(W, 640), T=rng.randint(12, 64), every=rng.randint(4, 24))


# ---------------------------------------------------------------------------- the scene
RING = 32  # frames a state holds


def _scene(H, W, n, seed, dH=0, dW=0, n_objects=5):
    """n frames: rgb uint8 [n, H, W, 3], depth int16 [n, dH or H, dW or W] (bits of a uint16),
    ground truth uint8 [n, H, W]; on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = random.Random(seed)
    dev = "cuda"
    yy = torch.arange(H, device=dev, dtype=torch.float32)[:, None]
    xx = torch.arange(W, device=dev, dtype=torch.float32)[None, :]
    bg = torch.full((H, W, 3), 128.0, device=dev)
    for _ in range(3):
        period, ang = r.uniform(8, 64), r.uniform(0, math.pi)
        arg = (2 * math.pi / period) * (math.cos(ang) * xx + math.sin(ang) * yy)
        for c in range(3):
            bg[..., c] += 20.0 * torch.sin(arg + r.uniform(0, 2 * math.pi))
    bg = (bg + torch.rand((H, W, 3), device=dev, generator=g) * 40.0 - 20.0).clamp(0, 255)
    plane = torch.where(xx < W / 2, 1500.0, 3000.0).expand(H, W).contiguous()
    s = W / 320.0
    objects = []
    for _ in range(n_objects):
        w, h = max(1, min(W, int(r.randint(40, 80) * s))), max(1, min(H, int(r.randint(40, 80) * s)))
        tex = torch.rand((h, w, 3), device=dev, generator=g) * 20.0 - 10.0
        colour = torch.tensor([float(r.randint(0, 255)) for _ in range(3)], device=dev)
        v, ang = r.uniform(1, 4) * s, r.uniform(0, 2 * math.pi)
        objects.append((w, h, (colour + tex).clamp(0, 255), r.uniform(0, W - w), r.uniform(0, H - h),
                        v * math.cos(ang), v * math.sin(ang)))
    rgb = torch.empty((n, H, W, 3), device=dev, dtype=torch.uint8)
    depth = torch.empty((n, dH or H, dW or W), device=dev, dtype=torch.int16)
    gt = torch.empty((n, H, W), device=dev, dtype=torch.uint8)
    if dH:
        sy = ((2 * torch.arange(dH, device=dev) + 1) * H) // (2 * dH)
        sx = ((2 * torch.arange(dW, device=dev) + 1) * W) // (2 * dW)
    for i in range(n):
        t = min(i, n - i)  # to and fro: frame n would be frame 0 again
        f, d, m = bg.clone(), plane.clone(), torch.zeros((H, W), device=dev, dtype=torch.uint8)
        at = []
        for w, h, tex, x0, y0, vx, vy in objects:
            x = int(min(max(0, x0 + vx * t), W - w))
            y = int(min(max(0, y0 + vy * t), H - h))
            at.append((x, y))
            a, b = y + int(0.1 * h), x + int(0.15 * w)  # its shadow
            f[a:a + h, b:b + w] = bg[a:a + h, b:b + w] * 0.6
        for (w, h, tex, *_), (x, y) in zip(objects, at):
            f[y:y + h, x:x + w] = tex
            d[y:y + h, x:x + w] = 900.0
            m[y:y + h, x:x + w] = 255
        f += torch.randn((H, W, 3), device=dev, generator=g).mul_(3.0).round_()
        if dH:
            d = d[sy][:, sx]
        d = (d + torch.randn(d.shape, device=dev, generator=g).mul_(10.0).round_()).clamp(1, 32767)
        d[torch.rand(d.shape, device=dev, generator=g) < 0.02] = 0.0
        rgb[i] = f.clamp(0, 255).to(torch.uint8)
        depth[i] = d.to(torch.int16)
        gt[i] = m
    return rgb, depth, gt


# ---------------------------------------------------------------------------- models
def _params(model, c):
    """("gmm5", "gmm7/3", "pbas20", "pbasg20") -> algo, parameters."""
    if model.startswith("gmm"):
        p = fgs.fgs_gmm_params_default()
        k = model[3:].split("/")
        p.Kc, p.Kd = int(k[0]), int(k[-1])
        for f in GMM_FIELDS:
            if f in c:
                setattr(p, f, c[f])
        return fgs.FGS_GMM, p
    p = fgs.fgs_pbas_params_default()
    p.gradient = 1 if model.startswith("pbasg") else 0
    p.N = int(model[5:] if p.gradient else model[4:])
    p.min_matches = min(p.min_matches, p.N)
    return fgs.FGS_PBAS, p


def _warm_frames(model):
    """Frames a model sees before the first pass: past its transient (PBAS: its N fill frames,
    then the adaptation of R and T)."""
    if model.startswith("gmm"):
        return 40
    return int(model[5:] if model.startswith("pbasg") else model[4:]) + 120


def _fleet(spec):
    out = []
    for part in spec.split(","):
        n, rest = part.split("*")
        model, hw = rest.split("@")
        H, W = (int(v) for v in hw.split("x"))
        out += [(model, H, W)] * int(n)
    return out


class _Borrowed:
    """Device memory of a model as torch sees it (the tensor keeps this object, and so the model)."""

    def __init__(self, owner, ptr, shape, strides, typestr):
        self.owner = owner
        self.__cuda_array_interface__ = dict(shape=shape, strides=strides, typestr=typestr, data=(ptr, False), version=3)


def _mask_view(m):
    return torch.as_tensor(_Borrowed(m, m.mask_ptr, (m.H, m.W), None, "|u1"), device="cuda")


def _gmm_views(m):
    """The model's mixtures, in place: one tensor per state field."""
    out = {}
    for f in fgs.fgs_get_state(m.handle):
        key = "%s.%d.%d" % (f["name"], f["index"], f["sub"])
        out[key] = torch.as_tensor(_Borrowed(m, f["base"], (m.H * m.W,), (f["pixel_stride"],), "<f4"), device="cuda")
    return out


# ---------------------------------------------------------------------------- prepare / run
def prepare(case, seed):
    kind = case["kind"]
    if kind == "window":
        return _prepare_window(case, seed)
    if kind == "fleet":
        return _prepare_fleet(case, seed)
    if kind == "serve":
        return _prepare_serve(case, seed)
    model, H, W = case["model"], case["H"], case["W"]
    dH, dW = case.get("dH", 0), case.get("dW", 0)
    rgb, depth, gt = _scene(H, W, RING, seed, dH, dW)
    algo, p = _params(model, case)
    m = fgs.Model(algo, H, W, p)
    s = dict(kind=kind, m=m, rgb=rgb, depth=depth, gt=gt, i=_warm_frames(model))
    for i in range(s["i"]):
        m.push(rgb[i % RING], depth[i % RING])
    m.sync()
    if kind == "camera":
        s["mask"] = torch.empty((H, W), dtype=torch.uint8, device="cuda")
        s["state"] = _gmm_views(m) if algo == fgs.FGS_GMM else {}
    elif kind == "host":
        s["rgb"] = rgb.cpu().numpy()
        s["depth"] = depth.cpu().numpy().view(np.uint16)
    elif kind == "score":
        n = case["frames"]
        m.static_enable(6)
        s.update(n=n, radius=case["radius"], mask=torch.empty((H, W), dtype=torch.uint8, device="cuda"),
                 smooth=torch.empty((n, H, W), dtype=torch.uint8, device="cuda"),
                 static=torch.empty((n, H, W), dtype=torch.uint8, device="cuda"))
    else:
        s["standby"] = fgs.Model(algo, H, W, p)
        s["blob"] = torch.empty(fgs.fgs_state_size(m.handle), dtype=torch.uint8, device="cuda")
        s["float"] = algo == fgs.FGS_GMM
    torch.cuda.synchronize()
    return s


def _prepare_fleet(case, seed):
    fleet = _fleet(case["models"])
    stream = torch.cuda.Stream()
    frames, models = {}, []
    for model, H, W in fleet:
        if (H, W) not in frames:
            frames[H, W] = _scene(H, W, RING, seed + len(frames))
        algo, p = _params(model, case)
        models.append(fgs.Model(algo, H, W, p, stream=stream))
    s = dict(kind="fleet", models=models, i=0, rings=[frames[H, W] for _, H, W in fleet])
    for _ in range(max(_warm_frames(model) for model, _, _ in fleet)):
        _push_fleet(s)
    s["masks"] = [_mask_view(m) for m in models]
    s["state"] = _gmm_views(models[0]) if models[0].algo == fgs.FGS_GMM else {}
    torch.cuda.synchronize()
    return s


def _push_fleet(s):
    i = s["i"]
    s["i"] = i + 1
    at = [(i + j) % RING for j in range(len(s["models"]))]  # each camera at its own place in the sequence
    fgs.push_frames(s["models"], [r[0][k] for r, k in zip(s["rings"], at)], [r[1][k] for r, k in zip(s["rings"], at)])


SERVE_RING = 8


def _prepare_serve(case, seed):
    fleet = _fleet(case["models"])
    srv = Server(64 << 30, max_streams=len(fleet))
    frames, ids = {}, []
    for model, H, W in fleet:
        if (H, W) not in frames:
            rgb, depth, _ = _scene(H, W, SERVE_RING, seed + len(frames))
            frames[H, W] = rgb.cpu().numpy(), depth.cpu().numpy().view(np.uint16)
        ids.append(srv.open(*_open_args(model, H, W, case)))
    s = dict(kind="serve", srv=srv, ids=ids, i=0, rings=[frames[H, W] for _, H, W in fleet],
             masks=[np.empty((H, W), np.uint8) for _, H, W in fleet])
    for _ in range(48):  # past the N fill frames
        _serve_round(s)
    return s


def _open_args(model, H, W, case):
    algo, p = _params(model, case)
    return algo, H, W, p


def _serve_round(s):
    i = s["i"]
    s["i"] = i + 1
    tickets = [s["srv"].submit(sid, r[0][(i + j) % SERVE_RING], r[1][(i + j) % SERVE_RING])
               for j, (sid, r) in enumerate(zip(s["ids"], s["rings"]))]
    for t, mask in zip(tickets, s["masks"]):
        s["srv"].wait(t, mask)
    return s["masks"]


def _prepare_window(case, seed):
    T, H, W = case["T"], case["H"], case["W"]
    rgb, depth, gt = _scene(H, W, T, seed)
    p = fgs.fgs_gmm_params_default()
    p.Kc = p.Kd = case["K"]
    theta = torch.tensor([0.01, 2.5, 1.0], device="cuda", requires_grad=True)
    return dict(kind="window", window=GmmWindow(T, H, W, p, case["every"]), theta=theta, rgb=rgb, depth=depth, gt=gt)


def run(s):
    kind = s["kind"]
    if kind == "fleet":
        _push_fleet(s)
        return dict(masks=s["masks"], state=s["state"])
    if kind == "serve":
        return _serve_round(s)
    if kind == "window":
        theta = s["theta"]
        theta.grad = None
        Z, has = GmmWindowFunction.apply(theta, s["rgb"], s["depth"], s["window"])
        window_bce_loss(Z, has, s["gt"]).backward()
        return dict(Z=Z.detach(), has=has, grad=theta.grad)
    m, i = s["m"], s["i"]
    if kind == "score":
        s["i"] = i + s["n"]
        for k in range(s["n"]):
            j = (i + k) % RING
            m.push(s["rgb"][j], s["depth"][j])
            m.eval_accumulate(s["gt"][j])
            m.mask_into(s["mask"])
            fgs.median_mask(s["mask"], s["radius"], s["smooth"][k])
            fgs.fgs_static_mask(m.handle, s["static"][k].data_ptr(), m.W, fgs.FGS_MEM_DEVICE)
        counts = m.eval_read(reset=True)
        return dict(counts=list(counts), mask=s["mask"], smooth=s["smooth"], static=s["static"])
    s["i"] = i + 1
    m.push(s["rgb"][i % RING], s["depth"][i % RING])
    if kind == "camera":
        m.mask_into(s["mask"])
        return dict(mask=s["mask"], state=s["state"])
    if kind == "host":
        return m.mask_host()
    blob = s["blob"]
    fgs.fgs_copy_state(m.handle, blob.data_ptr(), blob.numel(), fgs.FGS_MEM_DEVICE)
    fgs.fgs_set_state(s["standby"].handle, blob.data_ptr(), blob.numel(), fgs.FGS_MEM_DEVICE)
    return dict(header=blob[:64], payload=blob[64:].view(torch.float32) if s["float"] else blob[64:])


# ---------------------------------------------------------------------------- work
def _step_bytes(model, px, per_channel=0):
    """One frame of one model: state that has to be read, state that changes on every pixel
    (weights, the matched Gaussian), the frame (5 bytes) and the mask (1)."""
    if model.startswith("gmm"):
        k = model[3:].split("/")
        Kc, Kd = int(k[0]), int(k[-1])
        return px * ((20 * Kc + 12 * Kd + 8 * Kc * per_channel) + 4 * (Kc + Kd) + 24 + 8 * per_channel + 6)
    if model.startswith("pbasg"):
        return px * (8 * int(model[5:]) + 48 + 6)
    return px * (4 * int(model[4:]) + 40 + 6)


def _step_flops(model, px):
    if model.startswith("gmm"):
        k = model[3:].split("/")
        return px * (30 * int(k[0]) + 20 * int(k[-1]))
    return px * 16 * int(model[5:] if model.startswith("pbasg") else model[4:])


def work(case):
    kind = case["kind"]
    if kind in ("fleet", "serve"):
        f = _fleet(case["models"])
        return dict(bytes=sum(_step_bytes(m, H * W) for m, H, W in f), flops=sum(_step_flops(m, H * W) for m, H, W in f))
    px = case["H"] * case["W"]
    if kind == "window":  # frames and ground truth in, scores and flags out, their gradient in
        n = px * case["T"]
        return dict(bytes=n * (5 + 1 + 4 + 1 + 4), flops=n * case["K"] * (50 + 60))
    b, f = _step_bytes(case["model"], px, case.get("var_mode", 0)), _step_flops(case["model"], px)
    if kind == "score":  # and per frame: ground truth, copied mask, smoothed mask, counter there and back, static mask
        return dict(bytes=case["frames"] * (b + px * 8), flops=case["frames"] * f)
    if kind == "checkpoint":  # and the state read, written to the blob, read and written again
        return dict(bytes=b + 4 * px * _state_bytes(case["model"]), flops=f)
    return dict(bytes=b, flops=f)


def _state_bytes(model):
    if model.startswith("gmm"):
        k = model[3:].split("/")
        return 20 * int(k[0]) + 12 * int(k[-1])
    if model.startswith("pbasg"):
        return 24 * int(model[5:]) + 48
    return 8 * int(model[4:]) + 40


# ---------------------------------------------------------------------------- in 64 bits
F64 = torch.float64


def _f32(x):
    return float(np.float32(x))


class _Mixture64:
    """One mixture of every pixel in float64, Gaussians by rank: w [K, n], mu [K, C, n],
    v [K, V, n] (V = 1, or C with a variance per channel)."""

    def __init__(self, K, C, n, v_init, v_min, alpha, per_channel, rho_mode):
        self.K, self.C, self.V = K, C, C if per_channel else 1
        self.v_init, self.v_min = (v_init / 3, v_min / 3) if per_channel else (v_init, v_min)
        self.alpha, self.rho_mode = alpha, rho_mode
        self.w = torch.zeros((K, n), dtype=F64, device="cuda")
        self.mu = torch.zeros((K, C, n), dtype=F64, device="cuda")
        self.v = torch.full((K, self.V, n), self.v_init, dtype=F64, device="cuda")

    def step(self, X, active, lam2, T_bg=_f32(0.7), w_init=_f32(0.05)):
        """Classifies X [C, n] on the mixtures before the update, updates where active; returns
        whether there is a score and delta.  Choices are made on values, outside autograd."""
        K, w, mu, v = self.K, self.w, self.mu, self.v
        alpha = self.alpha
        a0 = float(alpha)  # the weights reach the scores through choices alone
        e2 = (X[None] - mu) ** 2
        q = (e2 / v).sum(1) if self.V > 1 else e2.sum(1) / v[:, 0]
        with torch.no_grad():
            over = torch.cumsum(w, 0) > T_bg
            B = torch.where(over.any(0), over.int().argmax(0) + 1, (w > 0).sum(0))
            ranks = torch.arange(K, device="cuda")[:, None]
            inside = (ranks < B) | (ranks == 0)
            amin = torch.where(inside, q, math.inf).argmin(0)
            used = w[0] > 0
            fits = (w > 0) & (q < lam2)
            matched, ks = fits.any(0), fits.int().argmax(0)
            hit = (ranks == ks) & matched & active
            put = (ranks == K - 1) & ~matched & active
            wn = torch.where(active, (1 - a0) * w, w)
            wn = torch.where(hit, wn + a0, wn)
            if self.rho_mode == 1:
                rho = (a0 / torch.where(hit, wn, 1.0))[:, None]
        if self.rho_mode == 0:
            rho = alpha
        delta = q.gather(0, amin[None])[0]
        mn = mu + rho * (X[None] - mu)
        d2 = (X[None] - mn) ** 2
        d2 = d2 if self.V > 1 else d2.sum(1, keepdim=True)
        vn = (v + rho * (d2 - v)).clamp(min=self.v_min)
        mu = torch.where(hit[:, None], mn, mu)
        v = torch.where(hit[:, None], vn, v)
        mu = torch.where(put[:, None], X[None], mu)
        v = torch.where(put[:, None], torch.full_like(v, self.v_init), v)
        with torch.no_grad():
            wn = torch.where(put, torch.full_like(wn, w_init), wn)
            wn = torch.where(active, wn / wn.sum(0), wn)
            order = torch.sort(wn / v.sum(1).sqrt(), dim=0, descending=True, stable=True).indices
            order = torch.where(active, order, ranks.expand_as(order))
            self.w = wn.gather(0, order)
        self.mu = mu.gather(0, order[:, None].expand_as(mu))
        self.v = v.gather(0, order[:, None].expand_as(v))
        return used, delta


def _inputs64(rgb, depth):
    X = rgb.reshape(-1, 3).t().to(F64)
    D = depth.reshape(-1).to(torch.int64)
    code = ((255 * D + 5000) // 10000).clamp(1, 255)
    return X, torch.where(D > 0, code, 0).to(F64)[None], D > 0


def _gmm64(case, seed, frames):
    """The mixtures after `frames` pushes of the ring, and the last mask."""
    model, H, W = case["model"], case["H"], case["W"]
    dH, dW = case.get("dH", 0), case.get("dW", 0)
    rgb, depth, _ = _scene(H, W, RING, seed, dH, dW)
    if dH:
        ty = ((2 * torch.arange(H, device="cuda") + 1) * dH) // (2 * H)
        tx = ((2 * torch.arange(W, device="cuda") + 1) * dW) // (2 * W)
    k = model[3:].split("/")
    alpha, per, rho = _f32(case.get("alpha", 0.01)), case.get("var_mode", 0) == 1, case.get("rho_mode", 0)
    n = H * W
    mc = _Mixture64(int(k[0]), 3, n, 675.0, 12.0, alpha, per, rho)
    md = _Mixture64(int(k[-1]), 1, n, 25.0, 1.0, alpha, False, rho)
    lam2 = 2.5 * 2.5
    fg = None
    with torch.no_grad():
        for i in range(frames):
            j = i % RING
            d = depth[j][ty][:, tx] if dH else depth[j]
            X, D, valid = _inputs64(rgb[j], d)
            uc, dc = mc.step(X, torch.ones_like(valid), lam2)
            ud, dd = md.step(D, valid, lam2)
            ud = ud & valid
            Z = torch.where(uc, dc - lam2, 0.0) + torch.where(ud, dd - lam2, 0.0)
            fg = (uc | ud) & (Z >= 0)
    return mc, md, fg.reshape(H, W).to(torch.uint8) * 255


def _state64(mc, md):
    out = {}
    for name, m in (("c", mc), ("d", md)):
        for k in range(m.K):
            out["w_%s.%d.0" % (name, k)] = m.w[k]
            for c in range(m.C):
                out["mu_%s.%d.%d" % (name, k, c)] = m.mu[k, c]
            for c in range(m.V):
                out["v_%s.%d.%d" % (name, k, c)] = m.v[k, c]
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "window":
        return _window64(case, seed)
    if kind == "fleet":  # (masks are whole numbers)
        model, H, W = _fleet(case["models"])[0]
        if not model.startswith("gmm"):
            return None
        mc, md, _ = _gmm64(dict(case, model=model, H=H, W=W), seed, _warm_frames(model) + 1)
        return dict(masks=None, state=_state64(mc, md))
    if kind in ("camera", "checkpoint") and case["model"].startswith("gmm"):
        mc, md, _ = _gmm64(case, seed, _warm_frames(case["model"]) + 1)
        if kind == "camera":
            return dict(mask=None, state=_state64(mc, md))
        parts = [x.reshape(-1) for x in (mc.w, mc.mu, mc.v, md.w, md.mu, md.v)]
        return dict(header=None, payload=torch.cat(parts))
    return None  # masks, counts and bytes


def _window64(case, seed):
    T, H, W, K = case["T"], case["H"], case["W"], case["K"]
    rgb, depth, gt = _scene(H, W, T, seed)
    theta = torch.tensor([_f32(0.01), 2.5, 1.0], dtype=F64, device="cuda", requires_grad=True)
    n = H * W
    mc = _Mixture64(K, 3, n, 675.0, 12.0, theta[0], False, 0)
    md = _Mixture64(K, 1, n, 25.0, 1.0, theta[0], False, 0)
    lam2 = theta[1] * theta[1]
    Zs, has = [], []
    for t in range(T):
        X, D, valid = _inputs64(rgb[t], depth[t])
        uc, dc = mc.step(X, torch.ones_like(valid), lam2)
        ud, dd = md.step(D, valid, lam2)
        ud = ud & valid
        zero = torch.zeros_like(dc)
        Zs.append(torch.where(uc, dc - lam2, zero) + torch.where(ud, theta[2] * (dd - lam2), zero))
        has.append(uc | ud)
    Z, has = torch.stack(Zs), torch.stack(has)
    w, y = has[1:].to(F64), (gt[1:] != 0).reshape(T - 1, n).to(F64)
    loss = torch.nn.functional.binary_cross_entropy_with_logits(Z[1:], y, weight=w, reduction="sum")
    (loss / w.sum().clamp_min(1.0)).backward()
    return dict(Z=Z.detach().reshape(T, H, W), has=None, grad=theta.grad)
