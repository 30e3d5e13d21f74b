"""The renderer's workloads as a user's program calls them.

A case is one pass of a tracking or mapping program: a frame rendered, one
training step over one or many views, one tracking iteration, the map's
expansion.  `listed()` names the standing ones (the sizes of this repository's
benchmark, tests and configurations), `draw(rng)` gives others of the same
ranges, `prepare` makes the inputs and the planned renderer, `run` is one pass
through the public entry points, `exact` evaluates the same pass in plain
float64 torch, and `work` states the bytes and operations a pass cannot do
without.

Case fields: op ("forward", "step", "track", "autograd", "expand"), n
(Gaussians), scene ("room": the indoor box, 70 % of the means on floor and
walls; "front": a cloud in front of the camera), views ("WxH" or
"k*WxH+..."), pose ("identity", "scattered" keyframes inside the room, "near":
hypotheses around the identity pose), focal (focal length in image widths), sh
(degree-1 spherical-harmonic colour), graph (the step replayed from a HIP
graph), params (gradients of the Gaussians, or of the poses alone), add
(gradients added to cleared buffers instead of written), mask (pixel mask).
"""
import math

import numpy as np
import torch

import paper_2311_11700_amd as gsr

W_RGB, W_DEPTH = 1.0, 0.1
TAU_T, TAU_D, GAMMA, ETA = 0.5, 0.1, 0.1, 0.01
LOGIT_INIT = -2.1972246
TILE = 16


def _case(name, op, n, views, **kw):
    c = dict(name=name, op=op, n=n, views=views, scene="room", pose="identity", focal=0.5, sh=False, graph=False,
             params=True, add=False, mask=False)
    c.update(kw)
    return c


def listed():
    tum = 517.3 / 640.0
    return [
        # The smallest render: 2 000 Gaussians, a thumbnail (latency and launches).
        _case("render_small", "forward", 2000, "160x120", scene="front", focal=150.0 / 160.0),
        # A tracking iteration of the coarse stage.
        _case("track_coarse", "track", 150_000, "160x120", params=False, focal=tum),
        # A tracking iteration of the fine stage: selected Gaussians, outlier cap.
        _case("track_fine", "track", 150_000, "640x480", params=False, focal=tum, mask=True),
        # An evaluation render of a Replica-sized frame.
        _case("render_replica", "forward", 300_000, "1200x680"),
        # Mapping on one Replica-sized keyframe, the loop replayed from a graph.
        _case("step_replica", "step", 300_000, "1200x680", graph=True),
        # The same with spherical-harmonic colour, called eagerly.
        _case("step_replica_sh", "step", 300_000, "1200x680", sh=True),
        # A user's own loss through autograd, poses included, on a TUM-sized frame.
        _case("autograd_tum", "autograd", 300_000, "640x480", focal=tum),
        # A few keyframes of odd sizes, masked pixels, gradients added to cleared buffers.
        _case("step_ragged", "step", 100_003, "641x479+317x233+97x33", pose="scattered", focal=0.7, add=True, mask=True),
        # Bundle adjustment over sixteen keyframes of mixed resolution.
        _case("step_16_keyframes", "step", 1_000_000, "4*320x240+8*640x480+4*1200x680", pose="scattered", focal=0.65,
              graph=True),
        # Relocalisation: 72 pose hypotheses in one call, pose gradients alone.
        _case("hypotheses", "step", 500_000, "64*600x340+8*1200x680", pose="near", params=False),
        # Map expansion on a new keyframe: the adding and the deleting step.
        _case("expand_replica", "expand", 300_000, "1200x680"),
    ]


def draw(rng):
    op = rng.choice(["forward", "step", "step", "step", "track", "autograd", "expand"])
    n = int(math.exp(rng.uniform(math.log(1500), math.log(600_000))))
    w = int(math.exp(rng.uniform(math.log(96), math.log(1280))))
    h = max(17, int(w * rng.uniform(0.5, 0.8)))
    views, pose = "%dx%d" % (w, h), rng.choice(["identity", "scattered"])
    if op == "step" and rng.random() < 0.5:
        k = rng.randint(2, 12)
        while k > 1 and (k * w * h > 3_000_000 or k * n > 4_000_000):
            k -= 1
        views, pose = "%d*%dx%d" % (k, w, h), rng.choice(["scattered", "near"])
    pose_only = op == "track" or (op == "step" and rng.random() < 0.25)
    return dict(op=op, n=n, views=views, scene="room", pose=pose, focal=round(rng.uniform(0.5, 0.9), 3),
                sh=op in ("forward", "step", "autograd") and rng.random() < 0.3, graph=op == "step" and rng.random() < 0.4,
                params=not pose_only, add=op == "step" and rng.random() < 0.3, mask=op in ("step", "track") and rng.random() < 0.4)


def work(case):
    """Bytes: every parameter, target and pixel input read once, every output
    written once.  FLOPs: a room's pixels blend about 80 Gaussians before they
    stop (20 operations each forward, 70 backward); the thin cloud of the
    small render about 20."""
    px, n = sum(w * h for w, h in _sizes(case)), case["n"]
    per = 4 * (23 if case["sh"] else 14)
    depth = 80 if case["scene"] == "room" else 20
    if case["op"] == "forward":
        return dict(bytes=n * per + px * 24, flops=px * depth * 20)
    if case["op"] == "expand":
        # three images and the colour in, a new Gaussian per unreliable pixel out; the deleting step's arrays
        return dict(bytes=px * (12 + 12 + 1) + px * 56 + n * (16 + 4 + 1), flops=px * 40 + n * 60)
    out = n * per if case["params"] else 0
    return dict(bytes=n * per + px * 16 + out, flops=px * depth * (20 + 70))


# ------------------------------------------------------------------ inputs

def _sizes(case):
    out = []
    for part in case["views"].split("+"):
        k, wh = part.split("*") if "*" in part else ("1", part)
        w, h = wh.split("x")
        out += [(int(w), int(h))] * int(k)
    return out


class _Cam:
    def __init__(self, fx, cx, cy, R, t, width, height):
        f = np.float32
        self.fx = self.fy = float(f(fx))
        self.cx, self.cy = float(f(cx)), float(f(cy))
        self.R, self.t = np.asarray(R, f), np.asarray(t, f)
        self.width, self.height = width, height


def _rotation(axis_angle):
    th = float(np.linalg.norm(axis_angle))
    k = np.asarray(axis_angle) / max(th, 1e-12)
    K = np.array([[0, -k[2], k[1]], [k[2], 0, -k[0]], [-k[1], k[0], 0]])
    return np.eye(3) + math.sin(th) * K + (1 - math.cos(th)) * K @ K


def _poses(case, rng):
    for _ in _sizes(case):
        if case["pose"] == "identity":
            # (the camera's own spot, a few millimetres and tenths of a degree off it)
            yield _rotation(rng.normal(0, 0.003, 3)), rng.normal(0, 0.003, 3)
        elif case["pose"] == "near":
            yield (_rotation(rng.normal(0, math.radians(2.0) / math.sqrt(3), 3)), rng.normal(0, 0.05 / math.sqrt(3), 3))
        else:
            # A keyframe inside the room looking at one of its surfaces, 1.5 m away or more.
            c = np.array([-2.5, -1.0, 0.0]) + rng.random(3) * np.array([5.0, 2.0, 3.0])
            while True:
                p = np.array([-3.0, -1.5, -0.5]) + rng.random(3) * np.array([6.0, 3.0, 4.0])
                axis, side = [(1, 1.5), (2, 3.5), (2, -0.5), (0, -3.0), (0, 3.0)][rng.integers(5)]
                p[axis] = side
                if np.linalg.norm(p - c) >= 1.5:
                    break
            z = (p - c) / np.linalg.norm(p - c)
            x = np.cross([0.0, 1.0, 0.0], z)
            x = x / np.linalg.norm(x) if np.linalg.norm(x) > 1e-6 else np.array([1.0, 0, 0])
            a = math.radians(rng.normal(0, 5.0))
            y = np.cross(z, x)
            R = np.stack([math.cos(a) * x + math.sin(a) * y, -math.sin(a) * x + math.cos(a) * y, z])
            yield R, -R @ c


def _cameras(case, seed):
    rng = np.random.default_rng(seed + 77)
    return [_Cam(case["focal"] * w, (w - 1) / 2, (h - 1) / 2, R, t, w, h)
            for (w, h), (R, t) in zip(_sizes(case), _poses(case, rng))]


def _room_depth(cam, gen):
    """Depth of the empty room along every pixel's ray, 2 % noise, a tenth of the readings missing."""
    dev = torch.device("cuda")
    y, x = torch.meshgrid(torch.arange(cam.height, device=dev), torch.arange(cam.width, device=dev), indexing="ij")
    d = torch.stack([(x - cam.cx) / cam.fx, (y - cam.cy) / cam.fy, torch.ones_like(x, dtype=torch.float32)], -1)
    R = torch.as_tensor(cam.R, device=dev)
    w = d.reshape(-1, 3) @ R
    o = -(R.T @ torch.as_tensor(cam.t, device=dev))
    lo, hi = torch.tensor([-3.0, -1.5, -0.5], device=dev), torch.tensor([3.0, 1.5, 3.5], device=dev)
    s = torch.where(w > 0, (hi - o) / w, torch.where(w < 0, (lo - o) / w, torch.full_like(w, 1e9))).amin(1)
    s = s * (1 + 0.02 * torch.randn(s.shape, generator=gen, device=dev))
    return torch.where(torch.rand(s.shape, generator=gen, device=dev) < 0.1, torch.zeros_like(s), s)


def _colour(cam, gen):
    """A smooth colour image with 5 % noise, planar [3 H W]."""
    low = torch.rand(1, 3, 7, 9, generator=gen, device="cuda")
    img = torch.nn.functional.interpolate(low, size=(cam.height, cam.width), mode="bilinear", align_corners=True)[0]
    return (img + 0.05 * torch.randn(img.shape, generator=gen, device="cuda")).reshape(-1)


def _scene(case, gen):
    n = case["n"]
    rand = lambda *s: torch.rand(*s, generator=gen, device="cuda")  # noqa: E731
    randn = lambda *s: torch.randn(*s, generator=gen, device="cuda")  # noqa: E731
    if case["scene"] == "front":
        mean = torch.cat([2 * rand(n, 2) - 1, 1 + 4 * rand(n, 1)], 1)
    else:
        lo = torch.tensor([-3.0, -1.5, -0.5], device="cuda")
        mean = lo + rand(n, 3) * torch.tensor([6.0, 3.0, 4.0], device="cuda")
        area = torch.tensor([24.0, 18.0, 18.0, 12.0, 12.0], device="cuda")
        which = torch.searchsorted((area / area.sum()).cumsum(0), rand(n)).clamp(max=4)
        jitter, surface = 0.01 * randn(n), rand(n) < 0.7
        for k, (axis, value) in enumerate([(1, 1.5), (2, 3.5), (2, -0.5), (0, -3.0), (0, 3.0)]):
            mean[:, axis] = torch.where(surface & (which == k), value + jitter, mean[:, axis])
    q = randn(n, 4)
    p = dict(mean=mean, log_scale=-3 + 0.5 * randn(n, 3), quat=q / q.norm(dim=1, keepdim=True), opacity_logit=randn(n))
    if case["sh"]:
        p["sh"] = torch.cat([2 * rand(n, 1, 3), 0.3 * randn(n, 3, 3)], 1)
    else:
        p["rgb"] = rand(n, 3)
    return {k: v.contiguous() for k, v in p.items()}


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    cams = _cameras(case, seed)
    d = dict(cams=cams, par=_scene(case, gen))
    if case["op"] == "forward":
        return d
    if case["pose"] == "near":
        # Every hypothesis is compared with the one observed frame (per resolution).
        made = {}
        for c in cams:
            if (c.width, c.height) not in made:
                b = _Cam(c.fx, c.cx, c.cy, np.eye(3), np.zeros(3), c.width, c.height)
                made[c.width, c.height] = (_colour(b, gen), _room_depth(b, gen))
        obs = [made[c.width, c.height] for c in cams]
    else:
        obs = [(_colour(c, gen), _room_depth(c, gen)) for c in cams]
    d["t_rgb"], d["t_depth"] = torch.cat([o[0] for o in obs]), torch.cat([o[1] for o in obs])
    P = d["t_depth"].numel()
    d["pixels"] = (torch.rand(P, generator=gen, device="cuda") < 0.9).to(torch.uint8) if case["mask"] else None
    if case["op"] == "track":
        d["cap"] = torch.full((1,), 2.5, device="cuda")
        if case["mask"]:  # the fine stage's reliable Gaussians
            d["select"] = (torch.rand(case["n"], generator=gen, device="cuda") < 0.95).to(torch.uint8)
    if case["op"] == "autograd":
        d["xi"] = 0.01 * torch.randn(len(cams), 6, generator=gen, device="cuda")
    if case["op"] == "expand":
        u = torch.rand(P, generator=gen, device="cuda")
        d["T"] = torch.where(u < 0.1, torch.ones_like(u), torch.rand(P, generator=gen, device="cuda") ** 2)
        d["depth"] = d["t_depth"] + 0.1 * torch.randn(P, generator=gen, device="cuda")
    return d


# ------------------------------------------------------------------ a pass

def _gaussians(par, mask=None):
    return gsr.Gaussians(par["mean"], par["log_scale"], par["quat"], par["opacity_logit"], par.get("rgb"), mask, par.get("sh"))


def _flags(case):
    f = gsr.GSR_POSE_GRAD | (gsr.GSR_GAUSS_GRAD if case["params"] else 0)
    return f if case["add"] else f | gsr.GSR_GRAD_OVERWRITE


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"], n, sizes = case, case["n"], _sizes(case)
    s["cams_d"] = gsr.pack_cameras(s["cams"])
    s["g"] = _gaussians(s["par"], s.get("select"))
    s["cfg"] = gsr.Config(flags=_flags(case))
    r = s["r"] = gsr.Renderer(0)
    r.plan(n, sizes)
    if case["op"] == "forward":
        s["out"] = r.new_images()
    if case["op"] in ("step", "track"):
        s["grads"] = r.new_grads(n, sh=case["sh"]) if case["params"] else {"d_pose": torch.zeros(len(sizes), 6, device="cuda")}
        s["loss"] = torch.zeros(1, device="cuda")
        s["clear"] = [t for t in s["grads"].values() if t is not None] + [s["loss"]]
    if case["op"] == "track":
        s["px"], s["cap_out"] = torch.zeros(r.total_pixels, device="cuda"), torch.zeros(1, device="cuda")
    if case["op"] == "autograd":
        s["leaves"] = [t.clone().requires_grad_() for t in
                       (s["par"]["mean"], s["par"]["log_scale"], s["par"]["quat"], s["par"]["opacity_logit"],
                        s["par"]["sh" if case["sh"] else "rgb"], s["xi"])]
        s["m_depth"] = (s["t_depth"] > 0).float()
    if case["op"] == "expand":
        px = r.total_pixels
        z = lambda *sh: torch.zeros(*sh, device="cuda")  # noqa: E731
        s["new"] = dict(mean=z(px, 3), log_scale=z(px, 3), quat=z(px, 4), opacity_logit=z(px), rgb=z(px, 3))
        s["count"] = torch.zeros(1, dtype=torch.int64, device="cuda")
        s["flag"] = torch.zeros(px, dtype=torch.uint8, device="cuda")
        s["logit"], s["decayed"] = z(n), torch.zeros(n, dtype=torch.uint8, device="cuda")
    if case["graph"]:
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            r.graph_capture(s["g"], s["cams_d"], s["cfg"], s["t_rgb"], s["t_depth"], s["pixels"], W_RGB, W_DEPTH,
                            grads=s["grads"], loss=s["loss"], stream=stream)
        torch.cuda.current_stream().wait_stream(stream)
    return s


def run(s):
    case, r = s["case"], s["r"]
    if case["op"] == "forward":
        return r.render_forward(s["g"], s["cams_d"], s["cfg"], out=s["out"])
    if case["op"] == "step":
        if case["add"]:
            torch._foreach_zero_(s["clear"])
        if case["graph"]:
            r.graph_launch()
        else:
            r.render_l1_fused(s["g"], s["cams_d"], s["cfg"], s["t_rgb"], s["t_depth"], s["pixels"], W_RGB, W_DEPTH,
                              grads=s["grads"], loss=s["loss"])
        return dict(s["grads"], loss=s["loss"])
    if case["op"] == "track":
        r.render_l1_fused(s["g"], s["cams_d"], s["cfg"], s["t_rgb"], s["t_depth"], s["pixels"], W_RGB, W_DEPTH,
                          out={"loss": s["px"]}, grads=s["grads"], loss=s["loss"], loss_cap=s["cap"])
        r.loss_median(s["px"], s["pixels"], 10.0, cap_out=s["cap_out"])
        return dict(d_pose=s["grads"]["d_pose"], loss=s["loss"], px=s["px"], cap=s["cap_out"])
    if case["op"] == "autograd":
        mean, ls, q, op, col, xi = s["leaves"]
        rgb, depth, T = gsr.render(r, mean, ls, q, op, col, s["cams_d"], s["cfg"], pose_xi=xi, check=False)
        loss = ((rgb - s["t_rgb"]).abs().mean() + 0.1 * ((depth - s["t_depth"]) * s["m_depth"]).abs().mean()
                + 0.01 * T.mean())
        grads = torch.autograd.grad(loss, s["leaves"])
        return dict(loss=loss.detach(), rgb=rgb.detach(), depth=depth.detach(), grads=list(grads))
    c = s["cams"][0]
    r.expand_add(s["cams_d"], s["T"], s["depth"], s["t_depth"], s["t_rgb"], s["new"], 0, r.total_pixels, TAU_T, TAU_D,
                 pixel_flag=s["flag"], count=s["count"])
    r.expand_delete(s["g"], s["cams_d"], s["t_depth"], c.width, c.height, GAMMA, ETA, logit_out=s["logit"],
                    decayed=s["decayed"])
    return dict(s["new"], count=s["count"], flag=s["flag"], logit=s["logit"], decayed=s["decayed"])


# ------------------------------------------------------------------ the same in 64 bits
#
# Projection by the EWA splatting equations, per-tile lists over the 3-sigma
# rectangles in depth order, front-to-back blending with prefix products;
# gradients by torch's autograd with the set of blended entries held fixed.

_F = lambda v: float(np.float32(v))  # noqa: E731  (a constant as the float32 the renderer is given)
A_MIN, A_MAX, T_MIN, Z_NEAR, LOW, GUARD = _F(1 / 255), _F(0.99), _F(1e-4), _F(0.2), _F(0.3), _F(1.3)


def _pose64(cam, xi):
    o = torch.zeros((), dtype=torch.float64, device="cuda")
    r, p = xi[:3], xi[3:]
    M = torch.stack([torch.stack([o, -p[2], p[1], r[0]]), torch.stack([p[2], o, -p[0], r[1]]),
                     torch.stack([-p[1], p[0], o, r[2]]), torch.stack([o, o, o, o])])
    T0 = torch.eye(4, dtype=torch.float64)
    T0[:3, :3], T0[:3, 3] = torch.as_tensor(cam.R).double(), torch.as_tensor(cam.t).double()
    T = torch.linalg.matrix_exp(M) @ T0.cuda()
    return T[:3, :3], T[:3, 3]


def _project64(par, cam, xi, keep):
    W, t = _pose64(cam, xi)
    q = par["quat"] / par["quat"].norm(dim=1, keepdim=True)
    w, x, y, z = q.unbind(1)
    Rq = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y), 2 * (x * y + w * z),
                      1 - 2 * (x * x + z * z), 2 * (y * z - w * x), 2 * (x * z - w * y), 2 * (y * z + w * x),
                      1 - 2 * (x * x + y * y)], 1).view(-1, 3, 3)
    M = (W @ Rq) * par["log_scale"].exp()[:, None, :]
    S = M @ M.transpose(1, 2)
    X = par["mean"] @ W.T + t
    px, py, pz = X.unbind(1)
    ok = keep & (pz > Z_NEAR)
    zs = torch.where(ok, pz, torch.ones_like(pz))
    lx, ly = GUARD * 0.5 * cam.width / cam.fx, GUARD * 0.5 * cam.height / cam.fy
    rx, ry = (px / zs).clamp(-lx, lx), (py / zs).clamp(-ly, ly)
    J0, J2, K1, K2 = cam.fx / zs, -cam.fx * rx / zs, cam.fy / zs, -cam.fy * ry / zs
    a0, a2 = J0 * S[:, 0, 0] + J2 * S[:, 2, 0], J0 * S[:, 0, 2] + J2 * S[:, 2, 2]
    a1 = J0 * S[:, 0, 1] + J2 * S[:, 2, 1]
    b1, b2 = K1 * S[:, 1, 1] + K2 * S[:, 2, 1], K1 * S[:, 1, 2] + K2 * S[:, 2, 2]
    A, B, C = a0 * J0 + a2 * J2 + LOW, a1 * K1 + a2 * K2, b1 * K1 + b2 * K2 + LOW
    det = A * C - B * B
    u, v = cam.fx * px / zs + cam.cx, cam.fy * py / zs + cam.cy
    if "sh" in par:
        d = par["mean"] + (W.T @ t)
        d = d / d.norm(dim=1, keepdim=True)
        c0, c1 = 0.5 / math.sqrt(math.pi), math.sqrt(3 / (4 * math.pi))
        k = par["sh"]
        col = c0 * k[:, 0] + c1 * (d[:, 1:2] * k[:, 1] + d[:, 2:3] * k[:, 2] + d[:, 0:1] * k[:, 3])
    else:
        col = par["rgb"]
    two = torch.stack([u, v, C / det, -B / det, A / det, torch.sigmoid(par["opacity_logit"]), *col.unbind(1), pz], 1)
    with torch.no_grad():
        TX, TY = -(-cam.width // TILE), -(-cam.height // TILE)
        hx, hy = 3 * A.sqrt(), 3 * C.sqrt()
        x0, x1 = ((u - hx) / TILE).floor().clamp(min=0), ((u + hx) / TILE).floor().clamp(max=TX - 1)
        y0, y1 = ((v - hy) / TILE).floor().clamp(min=0), ((v + hy) / TILE).floor().clamp(max=TY - 1)
        ok = ok & (det > 0) & (x0 <= x1) & (y0 <= y1)
        idx = ok.nonzero()[:, 0]
        x0, x1, y0, y1 = (e[idx].long() for e in (x0, x1, y0, y1))
        wd = x1 - x0 + 1
        cnt = wd * (y1 - y0 + 1)
        who = torch.repeat_interleave(torch.arange(idx.numel(), device="cuda"), cnt)
        j = torch.arange(who.numel(), device="cuda") - (cnt.cumsum(0) - cnt)[who]
        tile = (y0[who] + j // wd[who]) * TX + x0[who] + j % wd[who]
        bits = pz[idx].float().view(torch.int32).long()[who]
        order = torch.sort((tile << 32) | bits, stable=True)[1]
        lst = idx[who[order]]
        starts = torch.searchsorted(tile[order].contiguous(), torch.arange(TX * TY + 1, device="cuda"))
    return two, lst, starts, TX, TY


def _alpha64(g, px, py):
    dx, dy = g[:, :, 0:1] - px[:, None, :], g[:, :, 1:2] - py[:, None, :]
    oG = g[:, :, 5:6] * torch.exp(-0.5 * (g[:, :, 2:3] * dx * dx + g[:, :, 4:5] * dy * dy) - g[:, :, 3:4] * dx * dy)
    return oG.clamp(max=A_MAX)


def _entries(lst, starts, tiles, first, length):
    at = starts[tiles][:, None] + first + torch.arange(length, device="cuda")[None, :]
    have = at < starts[tiles + 1][:, None]
    return lst[at.clamp(max=max(lst.numel() - 1, 0))], have


def _needed(two, lst, starts, tiles, px, py):
    """Entries of each tile's list that its pixels look at before all have stopped."""
    need, P, first, step = torch.zeros_like(tiles), torch.ones_like(px), 0, 128
    at = torch.arange(tiles.numel(), device="cuda")
    at = at[starts[tiles + 1] > starts[tiles]]
    while at.numel():
        nxt = []
        for a in at.split(256):
            ids, have = _entries(lst, starts, tiles[a], first, step)
            al = _alpha64(two[ids], px[a], py[a])
            al = torch.where((al >= A_MIN) & have[:, :, None], al, torch.zeros_like(al))
            P[a] = (1 - al).prod(1) * P[a]
            need[a] = (starts[tiles[a] + 1] - starts[tiles[a]]).clamp(max=first + step)
            nxt.append(a[(P[a] >= T_MIN).any(1) & (starts[tiles[a] + 1] - starts[tiles[a]] > first + step)])
        at, first = torch.cat(nxt), first + step
    return need


def _view64(par, cam, xi, keep, pixel_loss):
    """One view's images; with pixel_loss(C, D, T, pixel) -> loss, also its
    gradient added into the leaves (par, xi), and the loss per pixel."""
    two, lst, starts, TX, TY = _project64(par, cam, xi, keep)
    q = two.detach()
    dev, P = "cuda", cam.width * cam.height
    img = dict(rgb=torch.zeros(3, P, dtype=torch.float64, device=dev), depth=torch.zeros(P, dtype=torch.float64, device=dev),
               T=torch.ones(P, dtype=torch.float64, device=dev), loss=torch.zeros(P, dtype=torch.float64, device=dev))
    tiles = torch.arange(TX * TY, device=dev)
    k = torch.arange(TILE * TILE, device=dev)
    ix, iy = (tiles % TX)[:, None] * TILE + k % TILE, (tiles // TX)[:, None] * TILE + k // TILE
    inside = (ix < cam.width) & (iy < cam.height)
    pix = (iy * cam.width + ix).clamp(max=P - 1)
    px, py = ix.double(), iy.double()
    with torch.no_grad():
        need = _needed(q, lst, starts, tiles, px, py)
    acc = torch.zeros_like(q)
    order = torch.argsort(need, descending=True)
    lens = need[order].tolist()
    b = 0
    while b < len(lens):
        L = max(lens[b], 1)
        e = min(len(lens), b + max(1, (1 << 24) // (L * 256)))
        t = order[b:e]
        b = e
        ids, have = _entries(lst, starts, t, 0, L)
        have = have & (torch.arange(L, device=dev)[None, :] < need[t][:, None])
        g = (q[ids] if lst.numel() else torch.zeros(*ids.shape, 10, dtype=torch.float64, device=dev)).requires_grad_()
        with torch.set_grad_enabled(pixel_loss is not None):
            al = _alpha64(g, px[t], py[t])
            gate = (al >= A_MIN) & have[:, :, None]
            with torch.no_grad():
                stop = gate & ((1 - torch.where(gate, al, torch.zeros_like(al))).cumprod(1) < T_MIN)
                used = gate & (stop.cumsum(1) == 0)
            ac = torch.where(used, al, torch.zeros_like(al))
            Tr = (1 - ac).cumprod(1)
            w = ac * torch.cat([torch.ones_like(Tr[:, :1]), Tr[:, :-1]], 1)
            CD = torch.stack([(w * g[:, :, f:f + 1]).sum(1) for f in (6, 7, 8, 9)], -1)
            Tf = Tr[:, -1]
            loss = pixel_loss(CD[..., :3], CD[..., 3], Tf, pix[t]) if pixel_loss is not None else None
        m = inside[t]
        if loss is not None:
            kept, shown = loss
            (kept * m).sum().backward()
            acc.index_add_(0, ids.reshape(-1), g.grad.reshape(-1, 10))
            img["loss"][pix[t][m]] = shown.detach()[m]
        with torch.no_grad():
            img["rgb"][:, pix[t][m]] = CD[m][:, :3].T
            img["depth"][pix[t][m]] = CD[m][:, 3]
            img["T"][pix[t][m]] = Tf[m]
    if pixel_loss is not None:
        two.backward(torch.where(torch.isfinite(acc), acc, torch.zeros_like(acc)))
    return img


def _l1_64(d, off, P, cap, w_rgb, w_depth, w_T=0.0):
    rgb, dep = d["t_rgb"][3 * off:3 * (off + P)].double().view(3, P), d["t_depth"][off:off + P].double()
    m = torch.ones(P, dtype=torch.float64, device="cuda") if d["pixels"] is None else d["pixels"][off:off + P].double()

    def f(C, D, T, pix):
        own = w_rgb * (C - rgb[:, pix].movedim(0, -1)).abs().sum(-1) + w_depth * (dep[pix] > 0) * (D - dep[pix]).abs() + w_T * T
        shown = own * m[pix]
        return (shown if cap is None else torch.where(shown.detach() > cap, torch.zeros_like(shown), shown)), shown
    return f


def exact(case, seed):
    d = _inputs(case, seed)
    if case["op"] == "expand":
        return _expand64(case, d)
    par = {k: v.double().requires_grad_(case["op"] != "forward") for k, v in d["par"].items()}
    xi = d["xi"].double() if "xi" in d else torch.zeros(len(d["cams"]), 6, dtype=torch.float64, device="cuda")
    xi.requires_grad_(case["op"] != "forward")
    keep = d["select"] != 0 if "select" in d else torch.ones(case["n"], dtype=torch.bool, device="cuda")
    cap = float(d["cap"]) if "cap" in d else None
    P_all = sum(c.width * c.height for c in d["cams"])
    w = (1 / (3 * P_all), _F(0.1) / P_all, 0.01 / P_all) if case["op"] == "autograd" else (W_RGB, _F(W_DEPTH), 0.0)
    img, off = [], 0
    for v, c in enumerate(d["cams"]):
        P = c.width * c.height
        f = None if case["op"] == "forward" else _l1_64(d, off, P, cap, *w)
        img.append(_view64(par, c, xi[v], keep, f))
        off += P
    cat = lambda k: torch.cat([i[k].reshape(-1) for i in img])  # noqa: E731
    if case["op"] == "forward":
        return dict(rgb=cat("rgb"), depth=cat("depth"), T_final=cat("T"), last=None)
    px = cat("loss")
    total = (px if cap is None else px[px <= cap]).sum().reshape(1)
    if case["op"] == "track":
        seen = px if d["pixels"] is None else px[d["pixels"] != 0]
        return dict(d_pose=xi.grad, loss=total, px=px, cap=10.0 * seen.sort()[0][(seen.numel() - 1) // 2].reshape(1))
    names = ("mean", "log_scale", "quat", "opacity_logit", "sh" if case["sh"] else "rgb")
    if case["op"] == "autograd":
        return dict(loss=total.reshape(()), rgb=cat("rgb"), depth=cat("depth"), grads=[par[k].grad for k in names] + [xi.grad])
    out = dict(d_pose=xi.grad, loss=total)
    if case["params"]:
        out.update({"d_" + k: par[k].grad for k in names})
        if case["sh"]:
            out["d_rgb"] = None
    return out


def _expand64(case, d):
    c = d["cams"][0]
    T, D, Dh = d["T"].double(), d["t_depth"].double(), d["depth"].double()
    hit = (D > 0) & ((1 - T < _F(TAU_T)) | ((D - Dh).abs() > _F(TAU_D)))
    p = hit.nonzero()[:, 0]
    x, y, z = (p % c.width).double(), (p // c.width).double(), D[p]
    R, t = torch.as_tensor(c.R).double().cuda(), torch.as_tensor(c.t).double().cuda()
    X = torch.stack([z * (x - c.cx) / c.fx, z * (y - c.cy) / c.fy, z], 1)
    rows = dict(mean=(X - t) @ R, log_scale=(z / c.fx).log()[:, None].expand(-1, 3), opacity_logit=torch.full_like(z, _F(LOGIT_INIT)),
                quat=torch.tensor([1.0, 0, 0, 0], dtype=torch.float64, device="cuda").expand(p.numel(), 4),
                rgb=d["t_rgb"].double().view(3, -1)[:, p].T)
    out = {}
    for k, v in rows.items():
        out[k] = torch.zeros(T.numel(), *v.shape[1:], dtype=torch.float64, device="cuda")
        out[k][:p.numel()] = v
    Xc = d["par"]["mean"].double() @ R.T + t
    zc = Xc[:, 2]
    ok = zc > Z_NEAR
    zs = torch.where(ok, zc, torch.ones_like(zc))
    ux, uy = (c.fx * Xc[:, 0] / zs + c.cx + 0.5).floor(), (c.fy * Xc[:, 1] / zs + c.cy + 0.5).floor()
    ok = ok & (ux >= 0) & (ux < c.width) & (uy >= 0) & (uy < c.height)
    Do = D[torch.where(ok, uy * c.width + ux, torch.zeros_like(ux)).long()]
    gone = ok & (Do > 0) & ((Do - zc) * Xc.norm(dim=1) / zs > _F(GAMMA))
    lam = d["par"]["opacity_logit"].double()
    o2 = _F(ETA) * torch.sigmoid(lam)
    return dict(out, count=None, flag=None, logit=torch.where(gone, torch.log(o2 / (1 - o2)), lam), decayed=None)
