"""The workloads this library is measured on: what a mapping or tracking
program has it do, through the public entry points of `binding` and `learned`.

Kinds (the field "kind" of a case):
  train      one optimisation step of a map (project, bin, sort, render, object
             loss, backward, Adam), captured once as a HIP graph and replayed
  autograd   the differentiable render inside a torch program: forward and
             gradient for the upstream gradients of the program's own loss
  tracking   one pose iteration against a frame: bin, render, loss, backward,
             pose gradient read by the host
  crops      one step of the plain optimiser over a batch of object crops, each
             with its own segment of Gaussians, in one graph
  net_train  one training step of the initialisation network
  net_start  the learned start of new crops: network, fallback, Gaussians
  ids        the evaluation render (instance channels and id map) and the
             objects' mask boxes
  quadrics   the dual-quadric fit of all objects and its refinement (FP64)
  increment  masks of unstable pixels and the Gaussians added there

Arithmetic is FP32 except the quadrics' FP64 (the rasteriser's FP64 build
serves gradient checks, not maps).  Scenes are synthetic: the room, keyframe,
single-view and crop shapes of `scenes.py` and `crops.py`, drawn here on the
GPU; target frames are ray-cast from the objects' spheres and the room's box.
"""
import math

import numpy as np
import torch

from paper_2503_02223_amd import binding as B
from paper_2503_02223_amd import learned as L

DEV = "cuda"
ROOM_LO, ROOM_HI = (-3.0, -1.5, -2.0), (3.0, 1.5, 2.0)


# ------------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest map: 2,000 Gaussians in a 128x96 view, where the launches count
        dict(name="train_2k_128x96", kind="train", scene="box", n=2000, width=128, height=96, objects=3, views=1,
             jobs=0, tile="8x8"),
        # the benchmark's map step: 200k Gaussians, 20 objects, one 640x480 view
        dict(name="train_200k_640x480", kind="train", scene="room", n=200_000, width=640, height=480, objects=20,
             views=1, jobs=0, tile="8x8"),
        # the largest: 1.2M Gaussians in eight keyframes and eight per-object jobs (the tile its autotuner picks)
        dict(name="train_keyframes_1200k", kind="train", scene="ring", n=1_200_000, width=640, height=480, objects=40,
             views=8, jobs=8, tile="16x8"),
        # a large view through autograd, colour and depth only
        dict(name="autograd_1M_1200x680", kind="autograd", scene="ring_room", n=1_000_000, width=1200, height=680,
             objects=20, probs=False, tile="8x8"),
        # an ordinary, ragged view through autograd with instance channels, at the context's default tile
        dict(name="autograd_30k_333x251_probs", kind="autograd", scene="room", n=30_011, width=333, height=251,
             objects=8, probs=True, tile="16x16"),
        # tracking one frame against the 200k map
        dict(name="tracking_200k_640x480", kind="tracking", scene="room", n=200_000, width=640, height=480,
             objects=20, tile="8x8"),
        # label generation: sixteen 128x128 crops per launch
        dict(name="crops_16x128", kind="crops", crops=16, size=128),
        # training the initialisation network: batches of 32 crops
        dict(name="net_train_32x128", kind="net_train", crops=32, size=128),
        # the learned start of one new object
        dict(name="net_start_1x128", kind="net_start", crops=1, size=128),
        # evaluation render with instance channels, id map and mask boxes
        dict(name="ids_200k_640x480", kind="ids", scene="room", n=200_000, width=640, height=480, objects=20,
             tile="16x16"),
        # object quadrics of a keyframe batch
        dict(name="quadrics_40x8", kind="quadrics", objects=40, views=8),
        # densification over a keyframe batch
        dict(name="increment_8x640x480", kind="increment", views=8, width=640, height=480, objects=40),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["train", "train", "train", "autograd", "autograd", "tracking", "crops", "crops", "net_train",
                       "net_train", "net_start", "ids", "quadrics", "increment"])
    c = dict(kind=kind)
    if kind == "train":
        scene = rng.choice(["box", "room", "room", "ring"])
        if scene == "box":
            c.update(scene=scene, n=_log_int(rng, 500, 20_000), width=rng.randint(64, 200), height=rng.randint(48, 160),
                     objects=3, views=1, jobs=0)
        elif scene == "room":
            c.update(scene=scene, n=_log_int(rng, 10_000, 400_000), width=rng.randint(240, 800),
                     height=rng.randint(180, 600), objects=rng.randint(4, 30), views=1, jobs=0)
        else:
            v = rng.randint(2, 6)
            c.update(scene=scene, n=_log_int(rng, 50_000, 700_000), width=rng.randint(320, 640),
                     height=rng.randint(240, 480), objects=rng.randint(10, 40), views=v, jobs=rng.randint(0, v))
        c["tile"] = rng.choice(["8x8", "8x8", "16x8", "16x16"])
    elif kind in ("autograd", "ids"):
        c.update(scene=rng.choice(["room", "ring_room"]), n=_log_int(rng, 5_000, 500_000),
                 width=rng.randint(200, 1000), height=rng.randint(150, 680), objects=rng.randint(3, 20),
                 tile=rng.choice(["8x8", "16x16", "16x8"]))
        if kind == "autograd":
            c["probs"] = rng.random() < 0.5
    elif kind == "tracking":
        c.update(scene="room", n=_log_int(rng, 20_000, 400_000), width=rng.randint(240, 800),
                 height=rng.randint(180, 600), objects=rng.randint(4, 30), tile=rng.choice(["8x8", "8x8", "16x16"]))
    elif kind in ("crops", "net_start"):
        c.update(crops=rng.randint(1, 16), size=16 * rng.randint(4, 10))
    elif kind == "net_train":
        c.update(crops=rng.randint(4, 32), size=16 * rng.randint(3, 9))
    elif kind == "quadrics":
        c.update(objects=rng.randint(5, 60), views=rng.randint(4, 14))
    else:
        c.update(views=rng.randint(1, 10), width=rng.randint(200, 900), height=rng.randint(150, 600),
                 objects=rng.randint(4, 40))
    return c


# ------------------------------------------------------------------- inputs
class _Rng:
    """Seeded draws: the large arrays on the GPU, the small ones on the host."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV).manual_seed(seed)
        self.h = np.random.default_rng(seed)

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.g, device=DEV)

    def uniform(self, *shape):
        return torch.rand(*shape, generator=self.g, device=DEV)


def _camera(R, t, f, W, H, cx=None, cy=None):
    return dict(R=np.asarray(R, np.float64), t=np.asarray(t, np.float64), fx=float(f), fy=float(f),
                cx=W / 2 if cx is None else cx, cy=H / 2 if cy is None else cy, width=int(W), height=int(H))


def _look_at(pos, target, f, W, H):
    z = np.asarray(target, np.float64) - pos
    z /= np.linalg.norm(z)
    x = np.cross([0.0, 1.0, 0.0], z)
    x /= np.linalg.norm(x)
    R = np.stack([x, np.cross(z, x), z])
    return _camera(R, -R @ pos, f, W, H)


def _scene(case, seed):
    """Gaussian parameters [14][n], ids, cameras, K, the objects' spheres and
    the counts of Gaussians per object (object k's are contiguous)."""
    r = _Rng(seed)
    n, W, H, n_obj = case["n"], case["width"], case["height"], case["objects"]
    kind = case["scene"]
    lo, hi = (torch.tensor(v, device=DEV).view(3, 1) for v in (ROOM_LO, ROOM_HI))
    if kind == "box":  # the single-view scene: ids mixed over one volume
        mu = 2 * r.uniform(3, n) - 1
        mu[2] += 3.0
        ls = -3.0 + 0.5 * r.normal(3, n)
        ids = (r.uniform(n) * n_obj).to(torch.int32).clamp_(max=n_obj - 1)
        eta = r.normal(n)
        cams = [_camera(np.eye(3), np.zeros(3), 110.0 * W / 128, W, H)]
        K, spheres, counts, first = n_obj, None, None, None
    else:
        surface = kind == "ring"
        if surface:
            counts = np.exp(r.h.uniform(np.log(1e3), np.log(8e4), n_obj)) * n / 1.2e6
            counts = (counts * min(1.0, 0.8 * n / counts.sum())).astype(np.int64) + 16
            a, q = r.h.uniform(0, 2 * np.pi, n_obj), 1.2 * np.sqrt(r.h.uniform(0, 1, n_obj))
            centres = np.stack([q * np.cos(a), r.h.uniform(-0.8, 0.8, n_obj), q * np.sin(a)], 1)
            sigma, (ls_m, ls_s) = 0.06, (-4.5, 0.4)
        else:
            counts = np.full(n_obj, int(0.7 * n) // n_obj)
            centres = r.h.uniform(ROOM_LO, ROOM_HI, size=(n_obj, 3))
            sigma, (ls_m, ls_s) = 0.3, (-4.0, 0.7)
        n_bg = n - int(counts.sum())
        bg = lo + (hi - lo) * r.uniform(3, n_bg)
        if surface:  # on the walls, floor and ceiling
            area = np.array([12.0, 12.0, 24.0, 24.0, 18.0, 18.0])
            face = torch.multinomial(torch.tensor(area, device=DEV), n_bg, True, generator=r.g)
            axis = face // 2
            side = torch.where(face % 2 == 0, lo[axis, 0], hi[axis, 0])
            bg.scatter_(0, axis.view(1, -1), side.view(1, -1))
        owner = torch.cat([torch.zeros(n_bg, dtype=torch.int64, device=DEV),
                           torch.repeat_interleave(torch.arange(1, n_obj + 1, device=DEV),
                                                   torch.tensor(counts, device=DEV))])
        c = torch.tensor(centres, dtype=torch.float32, device=DEV)
        mu = torch.cat([bg, c[owner[n_bg:] - 1].T + sigma * r.normal(3, n - n_bg)], 1)
        ids = owner.to(torch.int32)
        ls = ls_m + ls_s * r.normal(3, n)
        eta = 1.5 * r.normal(n)
        first = n_bg + np.concatenate([[0], np.cumsum(counts)[:-1]])
        spheres, K = (centres, 1.6 * sigma), n_obj + 1
        if kind == "room":
            s = min(W / 640, H / 480)
            cams = [_camera(np.eye(3), [0.0, 0.0, 7.63], 600.0 * s, W, H)]
        else:
            views = case.get("views", 1)
            angles = np.sort(r.h.uniform(0, 2 * np.pi, views)) if views > 1 else [0.0]
            f = 600.0 * W / (640 if surface else 1200)
            cams = [_look_at(np.array([2 * np.sin(a), 0.0, -2 * np.cos(a)]), np.zeros(3), f, W, H) for a in angles]
    quat = torch.nn.functional.normalize(r.normal(4, n), dim=0)
    params = torch.cat([mu, ls, quat, eta.view(1, n), r.uniform(3, n)]).contiguous()
    return dict(params=params, ids=ids.contiguous(), cams=cams, K=K, spheres=spheres, first=first, counts=counts)


def _observed(sc, case, seed):
    """Frames a camera would see: objects as spheres in front of the room's
    walls, with sensor noise and holes in the depth.  Without spheres (the
    single-view scene) patches of ids over a slanted plane."""
    r = _Rng(seed + 7919)
    W, H, cams, K = case["width"], case["height"], sc["cams"], sc["K"]
    V = len(cams)
    v, u = torch.meshgrid(torch.arange(H, device=DEV) + 0.5, torch.arange(W, device=DEV) + 0.5, indexing="ij")
    depth = torch.zeros(V, H, W, device=DEV)
    ids = torch.full((V, H, W), -1, dtype=torch.int32, device=DEV)
    for i, cam in enumerate(cams):
        if sc["spheres"] is None:
            depth[i] = 2.5 + 1.0 * u / W
            patch = torch.randint(-1, K, ((H + 15) // 16, (W + 15) // 16), generator=r.g, device=DEV)
            ids[i] = patch.repeat_interleave(16, 0).repeat_interleave(16, 1)[:H, :W].to(torch.int32)
            continue
        R, t = (torch.tensor(cam[k], dtype=torch.float32, device=DEV) for k in ("R", "t"))
        d = torch.stack([(u - cam["cx"]) / cam["fx"], (v - cam["cy"]) / cam["fy"], torch.ones_like(u)], -1)
        dw, o = d @ R, -(R.T @ t)  # world rays, scaled so that their parameter is the camera depth
        lo, hi = (torch.tensor(x, device=DEV) for x in (ROOM_LO, ROOM_HI))
        near, far = (lo - o) / dw, (hi - o) / dw
        enter, leave = torch.minimum(near, far).amax(-1), torch.maximum(near, far).amin(-1)
        best = torch.where((leave > enter) & (leave > 0.2), leave, torch.zeros_like(leave))
        ids[i][best > 0] = 0
        best = torch.where(best > 0, best, torch.full_like(best, 1e9))
        centres, rad = sc["spheres"]
        aa = (dw * dw).sum(-1)
        for k, c in enumerate(centres):
            oc = o - torch.tensor(c, dtype=torch.float32, device=DEV)
            bb, cc = (dw * oc).sum(-1), float(oc @ oc) - rad * rad
            disc = bb * bb - aa * cc
            z = (-bb - disc.clamp_min(0).sqrt()) / aa
            hit = (disc > 0) & (z > 0.2) & (z < best)
            best = torch.where(hit, z, best)
            ids[i][hit] = k + 1
        depth[i] = torch.where(best < 1e8, best, torch.zeros_like(best))
    depth *= 1 + 0.01 * r.normal(V, H, W)
    depth[r.uniform(V, H, W) < 0.03] = 0.0
    tone = r.uniform(K + 1, 3)[ids.long() + 1].permute(0, 3, 1, 2)
    color = (tone + 0.1 * r.normal(V, 3, H, W)).clamp_(0, 1)
    return dict(color=color.contiguous(), depth=depth.clamp_min(0).contiguous(), id=ids.contiguous())


def _jobs(sc, case, tgt):
    """Per-object jobs beside the keyframes: the objects largest in some
    keyframe, each alone in that view, inside its box and a margin."""
    W, H, V = case["width"], case["height"], len(sc["cams"])
    if not case["jobs"]:
        return {}, tgt, sc["cams"]
    idm = tgt["id"]
    cnt = torch.stack([(idm == k).sum((1, 2)) for k in range(1, sc["K"])]).cpu().numpy()
    n = sc["params"].shape[1]
    seg, win, job, jv = [(0, n)] * V, [(0, 0, W, H)] * V, [-1] * V, []
    for k in np.argsort(-cnt.max(1), kind="stable")[: case["jobs"]]:
        view = int(np.argmax(cnt[k]))
        ys, xs = np.nonzero((idm[view] == int(k) + 1).cpu().numpy())
        if not ys.size:
            continue
        win.append((max(int(xs.min()) - 8, 0), max(int(ys.min()) - 8, 0), min(int(xs.max()) + 9, W),
                    min(int(ys.max()) + 9, H)))
        seg.append((int(sc["first"][k]), int(sc["counts"][k])))
        job.append(int(k) + 1)
        jv.append(view)
    cams = sc["cams"] + [sc["cams"][v] for v in jv]
    tgt = {k: torch.cat([t, t[jv]]).contiguous() for k, t in tgt.items()}
    return dict(segments=seg, windows=win, jobs=job), tgt, cams


def _crops(case, seed):
    """Object crops: a textured, shaded ellipsoid per 110-pixel-focal crop,
    as r, g, b, depth, mask [B][5][S][S].  The mask is the quarter of the
    pixels nearest the object (so every seed has as many valid pixels)."""
    r = _Rng(seed)
    Bn, S = case["crops"], case["size"]
    v, u = torch.meshgrid(torch.arange(S, device=DEV) + 0.5, torch.arange(S, device=DEV) + 0.5, indexing="ij")
    d = torch.stack([(u - S / 2) / 110.0, (v - S / 2) / 110.0, torch.ones_like(u)], -1)
    out = torch.zeros(Bn, 5, S, S, device=DEV)
    for b in range(Bn):
        ax = torch.tensor(r.h.uniform(0.05, 0.3, 3), dtype=torch.float32, device=DEV)
        q, _ = np.linalg.qr(r.h.normal(size=(3, 3)))
        rho = float(ax.max())
        c = torch.tensor([0.0, 0.0, max(2.04 * rho * 128 / S, rho + 0.3)], device=DEV)
        M = (torch.tensor(q, dtype=torch.float32, device=DEV) / ax)  # unit sphere <- object
        e, oc = d @ M, -(c @ M)
        aa, bb, cc = (e * e).sum(-1), (e * oc).sum(-1), float(oc @ oc) - 1.0
        disc = bb * bb / aa - cc
        hit = torch.zeros_like(disc, dtype=torch.bool)
        hit.view(-1)[torch.topk(disc.reshape(-1), S * S // 4)[1]] = True
        disc = disc * aa
        z = (-bb - disc.clamp_min(0).sqrt()) / aa
        nrm = e * z.unsqueeze(-1) + oc
        k = torch.tensor(r.h.normal(size=(3, 3)) * 4, dtype=torch.float32, device=DEV)
        mix = 0.5 + 0.5 * torch.sin(nrm @ k).mean(-1)
        two = torch.tensor(r.h.uniform(0, 1, (2, 3)), dtype=torch.float32, device=DEV)
        shade = 0.6 + 0.4 * nrm[..., 2].neg().clamp(0, 1)
        rgb = (two[0].view(3, 1, 1) * mix + two[1].view(3, 1, 1) * (1 - mix)) * shade
        out[b, :3] = torch.where(hit, (rgb + 0.02 * r.normal(3, S, S)).clamp(0, 1), torch.zeros_like(rgb))
        out[b, 3] = torch.where(hit, z, torch.zeros_like(z))
        out[b, 4] = hit.float()
    return out.contiguous()


def _crop_scene(case, seed):
    """Crops and the Gaussians of their valid pixels some way into the plain
    optimisation (moved, stretched, turned), one segment per crop."""
    rgbdm = _crops(case, seed)
    r = _Rng(seed + 104729)
    S = case["size"]
    ok = (rgbdm[:, 4] > 0.5) & (rgbdm[:, 3] > 0)
    b, y, x = ok.nonzero(as_tuple=True)
    n = int(b.numel())
    d = rgbdm[b, 3, y, x]
    mu = torch.stack([(x + 0.5 - S / 2) / 110.0 * d, (y + 0.5 - S / 2) / 110.0 * d, d]) + 0.002 * r.normal(3, n)
    ls = torch.log(d / 110.0) + 0.2 * r.normal(3, n)
    quat = torch.tensor([1.0, 0, 0, 0], device=DEV).view(4, 1) + 0.1 * r.normal(4, n)
    rgb = rgbdm[b, :3, y, x].T + 0.05 * r.normal(3, n)
    params = torch.cat([mu, ls, quat, (2.0 + 0.5 * r.normal(n)).view(1, n), rgb]).contiguous()
    counts = torch.bincount(b, minlength=case["crops"]).cpu().numpy()
    seg = [(int(f), int(c)) for f, c in zip(np.concatenate([[0], np.cumsum(counts)[:-1]]), counts)]
    cams = [_camera(np.eye(3), np.zeros(3), 110.0, S, S)] * case["crops"]
    tgt = dict(color=rgbdm[:, :3].contiguous(), depth=rgbdm[:, 3].contiguous(),
               id=torch.where(ok, 0, -1).to(torch.int32).contiguous())
    return dict(params=params, ids=torch.zeros(n, dtype=torch.int32, device=DEV), cams=cams, K=1), tgt, seg


def _quadric_inputs(case, seed):
    """Objects seen by ring keyframes: the observed boxes are the tangent
    boxes of their ellipsoids, a pixel or so off."""
    h = np.random.default_rng(seed)
    n, V, W, H = case["objects"], case["views"], 640, 480
    cams = [_look_at(np.array([3 * np.sin(a), h.uniform(-1, 1), -3 * np.cos(a)]), np.zeros(3), 500.0, W, H)
            for a in 2 * np.pi * np.arange(V) / V]
    Ps = np.stack([np.array([[c["fx"], 0, c["cx"]], [0, c["fy"], c["cy"]], [0, 0, 1]]) @ np.concatenate(
        [c["R"], c["t"].reshape(3, 1)], 1) for c in cams])
    boxes, obj, view = [], [], []
    for k in range(n):
        q, _ = np.linalg.qr(h.normal(size=(3, 3)))
        Z = np.eye(4)
        Z[:3, :3], Z[:3, 3] = q, h.uniform(-0.6, 0.6, 3)
        Q = Z @ np.diag([*(h.uniform(0.08, 0.3, 3) ** 2), -1.0]) @ Z.T
        for v in range(V):
            C = Ps[v] @ Q @ Ps[v].T
            C = C / C[2, 2]
            dx, dy = math.sqrt(C[0, 2] ** 2 - C[0, 0]), math.sqrt(C[1, 2] ** 2 - C[1, 1])
            boxes.append(np.array([C[0, 2] - dx, C[1, 2] - dy, C[0, 2] + dx, C[1, 2] + dy]) + 0.7 * h.normal(size=4))
            obj.append(k)
            view.append(v)
    t = lambda a, dt: torch.tensor(np.asarray(a), dtype=dt, device=DEV)  # noqa: E731
    return dict(boxes=t(boxes, torch.float64), obj=t(obj, torch.int32), view=t(view, torch.int32),
                Ps=t(Ps.reshape(V, 12), torch.float64), wh=t([[W, H]] * V, torch.int32))


def _increment_inputs(case, seed):
    """A rendered batch of frames beside the observed one: right for most
    pixels, with missing geometry and wrong colours in patches."""
    n_obj = case["objects"]
    r = _Rng(seed + 31)
    angles = np.sort(r.h.uniform(0, 2 * np.pi, case["views"]))
    a, q = r.h.uniform(0, 2 * np.pi, n_obj), 1.2 * np.sqrt(r.h.uniform(0, 1, n_obj))
    centres = np.stack([q * np.cos(a), r.h.uniform(-0.8, 0.8, n_obj), q * np.sin(a)], 1)
    W, H = case["width"], case["height"]
    cams = [_look_at(np.array([2 * np.sin(x), 0.0, -2 * np.cos(x)]), np.zeros(3), 600.0 * W / 640, W, H) for x in angles]
    sc = dict(cams=cams, K=n_obj + 1, spheres=(centres, 0.1))
    tgt = _observed(sc, case, seed)
    V = case["views"]
    patch = r.uniform(V, (H + 15) // 16, (W + 15) // 16).repeat_interleave(16, 1).repeat_interleave(16, 2)[:, :H, :W]
    color = torch.where((patch < 0.1).unsqueeze(1), r.uniform(V, 3, H, W), tgt["color"] + 0.03 * r.normal(V, 3, H, W))
    depth = torch.where(patch > 0.93, torch.zeros_like(tgt["depth"]), tgt["depth"] + 0.02 * r.normal(V, H, W))
    p_t = torch.where(patch > 0.93, 0.3 * r.uniform(V, H, W), 0.6 + 0.4 * r.uniform(V, H, W))
    img = dict(color=color.contiguous(), depth=depth.contiguous(), p_target=p_t.contiguous())
    img.update(t_final=torch.zeros_like(p_t), last=torch.zeros_like(tgt["id"]), target=tgt["id"])
    return cams, tgt, img


def _labels(case, seed):
    r = _Rng(seed + 15485863)
    lab = 0.1 * r.normal(case["crops"], 5, case["size"], case["size"])
    lab[:, 1] += 2.0
    return lab.contiguous()


def _theta_layers(seed):
    """He-normal layers 5-32-64-64-6 with small biases; the predicted
    log-error (channel 5) starts at 2."""
    h = np.random.default_rng(seed + 271)
    ch = (5, 32, 64, 64, 6)
    layers = [(h.normal(0.0, math.sqrt(2.0 / (9 * a)), (b, a, 3, 3)).astype(np.float32),
               (0.01 * h.normal(size=b)).astype(np.float32)) for a, b in zip(ch[:-1], ch[1:])]
    layers[3][1][5] += 2.0
    return layers


CHAN_W = [4.0, 0.5, 20.0, 20.0, 20.0]


# ------------------------------------------------------------------- the passes
def _tile(case):
    w, h = case["tile"].split("x")
    return B.Context(tile_w=int(w), tile_h=int(h))


def _late_lrs(extent=1.0):
    """Learning rates at the end of the usual exponential decay to 1%."""
    return [0.01 * x for x in B.default_lrs(extent)]


def _upstream(case, K, seed):
    r = _Rng(seed + 65537)
    W, H = case["width"], case["height"]
    n = W * H
    g = [torch.sign(r.normal(1, 3, H, W)) / (3 * n), torch.sign(r.normal(1, H, W)) / n, 0.1 * r.normal(1, H, W) / n]
    if case["probs"]:
        g.append(r.normal(1, K, H, W) / n)
    return g


def _tracking_cam(cam):
    """The frame's camera, half a degree and 4 cm off."""
    a = np.array([0.006, -0.005, 0.003])
    th = np.linalg.norm(a)
    k = a / th
    X = np.array([[0, -k[2], k[1]], [k[2], 0, -k[0]], [-k[1], k[0], 0]])
    E = np.eye(3) + math.sin(th) * X + (1 - math.cos(th)) * X @ X
    return dict(cam, R=E @ cam["R"], t=E @ cam["t"] + np.array([0.03, -0.025, 0.01]))


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case)
    if kind == "train":
        sc = _scene(case, seed)
        opts, tgt, cams = _jobs(sc, case, _observed(sc, case, seed))
        s["tr"] = B.Trainer(sc["params"], sc["ids"], cams, sc["K"], tgt, lrs=_late_lrs(), ctx=_tile(case), **opts)
        s["graph"] = s["tr"].capture()
    elif kind == "crops":
        sc, tgt, seg = _crop_scene(case, seed)
        s["tr"] = B.Trainer(sc["params"], sc["ids"], sc["cams"], 1, tgt, lrs=_late_lrs(0.3), ctx=L.crop_context(),
                            segments=seg, capacity=max(4096, 48 * sc["params"].shape[1]))
        s["graph"] = s["tr"].capture()
    elif kind == "autograd":
        sc = _scene(case, seed)
        s["r"] = B.Rasterizer(sc["cams"], case["n"], sc["K"], ctx=_tile(case))
        s["p"] = sc["params"].requires_grad_(True)
        s["ids"] = sc["ids"]
        s["g"] = _upstream(case, sc["K"], seed)
        s["r"].bin(sc["params"].detach(), sc["ids"])  # sizes the pair list, as a program's first frame does
    elif kind == "tracking":
        sc = _scene(case, seed)
        cam = _tracking_cam(sc["cams"][0])
        s.update(p=sc["params"], ids=sc["ids"], cam=cam, tgt=_observed(sc, case, seed))
        s["r"] = r = B.Rasterizer([cam], case["n"], sc["K"], ctx=_tile(case))
        r.bin(s["p"], s["ids"])
        s["img"] = r.frame.new_images(target=s["tgt"]["id"])
        s["gi"] = dict(d_color=torch.empty_like(s["img"]["color"]), d_depth=torch.empty_like(s["img"]["depth"]),
                       d_p_target=torch.empty_like(s["img"]["depth"]))
        s["loss"] = torch.zeros(4, dtype=torch.float64, device=DEV)
        s["pose"] = torch.empty(1, 6, dtype=torch.float64, device=DEV)
    elif kind == "ids":
        sc = _scene(case, seed)
        s.update(p=sc["params"], ids=sc["ids"])
        s["r"] = B.Rasterizer(sc["cams"], case["n"], sc["K"], ctx=_tile(case))
        s["r"].bin(s["p"], s["ids"])
    elif kind == "net_train":
        s["x"], s["lab"] = _crops(case, seed), _labels(case, seed)
        s["net"] = L.Net(theta=L.pack_layers(_theta_layers(seed)))
        s["out"] = torch.empty(case["crops"], 6, case["size"], case["size"], device=DEV)
    elif kind == "net_start":
        s["x"] = _crops(case, seed)
        s["net"] = L.Net(theta=L.pack_layers(_theta_layers(seed)))
        s["net"].workspace(case["crops"], case["size"], case["size"])
        c = L.valid_counts(s["x"].cpu().numpy())
        s["off"] = np.concatenate([[0], np.cumsum(c)]).astype(np.int64)
        s["cams"] = [_camera(np.eye(3), np.zeros(3), 110.0, case["size"], case["size"])] * case["crops"]
    elif kind == "quadrics":
        s["ctx"] = B.Context()
        s.update(_quadric_inputs(case, seed))
    else:
        cams, s["tgt"], s["img"] = _increment_inputs(case, seed)
        V, W, H = case["views"], case["width"], case["height"]
        s["frame"] = B.Frame(B.Context(), cams, 0, case["objects"] + 1, 0)
        s["masks"] = torch.empty(V, H, W, dtype=torch.uint8, device=DEV)
        s["obj"] = torch.zeros(2 * (case["objects"] + 1), dtype=torch.int32, device=DEV)
        cap = V * W * H // 2
        s["params"] = torch.zeros(14, cap, device=DEV)
        s["ids"] = torch.zeros(cap, dtype=torch.int32, device=DEV)
        s["counts"] = torch.zeros(V + 1, dtype=torch.int64, device=DEV)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind in ("train", "crops"):
        s["graph"].replay()
        t = s["tr"]
        return dict(loss=t.loss, color=t.img["color"], depth=t.img["depth"], t_final=t.img["t_final"],
                    p_target=t.img["p_target"], params=t.params, m=t.m, v=t.v)
    if kind == "autograd":
        out = B.rasterize(s["p"], s["ids"], s["r"], want_probs=case["probs"])
        used = out if case["probs"] else out[:3]
        g, = torch.autograd.grad(used, s["p"], s["g"])
        return dict(color=out[0].detach(), depth=out[1].detach(), t_final=out[2].detach(), probs=out[3].detach(),
                    grad=g)
    if kind == "tracking":
        r = s["r"]
        r.cams[0] = s["cam"]
        r.frame.cams[0] = B.make_cameras([s["cam"]])[0]
        r.bin(s["p"], s["ids"], grow=True)
        f = r.frame
        f.render_forward(s["img"])
        f.object_loss(s["img"], s["tgt"], s["gi"], s["loss"])
        f.render_backward(s["img"], s["gi"])
        f.pose_backward(s["p"], s["pose"])
        # the host takes the pose step; the gradient is a sum of FP32 terms and is handed on as such
        return dict(loss=s["loss"], pose=s["pose"].cpu().to(torch.float32), color=s["img"]["color"],
                    depth=s["img"]["depth"], t_final=s["img"]["t_final"])
    if kind == "ids":
        img = s["r"].forward(s["p"], s["ids"], probs=True, id_map=True)
        boxes, obj, view = B.id_boxes(s["r"].ctx, img["id_map"], case["objects"] + 1)
        return dict(color=img["color"], depth=img["depth"], t_final=img["t_final"], probs=img["probs"],
                    id_map=img["id_map"], obj=obj, view=view, boxes=torch.where(obj.view(-1, 1) >= 0, boxes, 0.0))
    if kind == "net_train":
        net = s["net"]
        net.train_step(s["x"], s["lab"], CHAN_W, 2e-5, out=s["out"])
        return dict(out=s["out"], loss=net.loss, grad=net.grad)
    if kind == "net_start":
        net = s["net"]
        out = net.forward(s["x"])
        use, mean = net.fallback(s["x"], out, 1e3)
        params, ids, _ = L.init_gaussians(net.ctx, s["x"], s["cams"], s["off"], out, use)
        return dict(out=out, use=use, mean=mean, params=params, ids=ids)
    if kind == "quadrics":
        fit = B.fit_dual_quadric(s["ctx"], s["boxes"], s["obj"], s["view"], s["Ps"], case["objects"], img_wh=s["wh"])
        ref = B.refine_quadrics(s["ctx"], s["boxes"], s["obj"], s["view"], s["Ps"], fit, img_wh=s["wh"])
        return {k: ref[k] for k in ("status", "mu", "R", "axes", "Q", "loss", "iou")}
    s["frame"].incremental_masks(s["img"], s["tgt"], s["masks"], s["obj"])
    s["frame"].densify(s["tgt"], s["masks"], s["params"], s["ids"], 0, s["counts"])
    return dict(masks=s["masks"], obj=s["obj"], params=s["params"], ids=s["ids"], counts=s["counts"])


# ------------------------------------------------------------------- what a pass cannot do without
def work(case):
    """Inputs read once and outputs written once; operations: about 85 per
    (pixel, Gaussian) evaluation forward and backward together (25 forward
    alone), 64 pixels in a Gaussian's 3-sigma ellipse at the scenes' scales."""
    kind = case["kind"]
    if kind in ("train", "crops", "autograd", "tracking", "ids"):
        if kind == "crops":
            n = case["crops"] * case["size"] ** 2 // 4
            px, items = case["crops"] * case["size"] ** 2, n
        else:
            n, px = case["n"], case["width"] * case["height"] * case.get("views", 1)
            items = n * case.get("views", 1)
        K = case.get("objects", 0) + 1
        if kind in ("train", "crops"):
            return dict(bytes=n * (6 * 56 + 4) + px * (20 + 24), flops=items * 64 * 85)
        if kind == "autograd":
            per = 20 + (4 * K if case["probs"] else 0)
            return dict(bytes=n * (2 * 56 + 4) + px * 2 * per, flops=items * 64 * 85)
        if kind == "tracking":
            return dict(bytes=n * 60 + px * (20 + 24) + 48, flops=items * 64 * 85)
        return dict(bytes=n * 60 + px * (20 + 4 * K + 4) + K * 40, flops=items * 64 * 25)
    if kind in ("net_train", "net_start"):
        px = case["crops"] * case["size"] ** 2
        mac = 9 * (5 * 32 + 32 * 64 + 64 * 64 + 64 * 6)
        if kind == "net_train":
            return dict(bytes=px * 4 * (5 + 5 + 6) + 69296 * 4 * 7, flops=2 * px * (3 * mac - 9 * 5 * 32))
        return dict(bytes=px * 4 * (5 + 6) + px // 4 * 60 + 69296 * 2, flops=2 * px * mac)
    if kind == "quadrics":
        n = case["objects"] * case["views"]
        return dict(bytes=n * 48 + case["objects"] * 8 * 31 + case["views"] * 104, flops=n * 100 * 600)
    px = case["views"] * case["width"] * case["height"]
    return dict(bytes=px * (36 + 1) + px // 10 * 60, flops=px * 20)


# ------------------------------------------------------------------- the same in 64 bits
def _project64(p, cam):
    """EWA projection of every Gaussian: (mx, my, A, B, C, opacity, z) and
    which are in front of the camera, differentiable."""
    W, t = (torch.tensor(cam[k], dtype=torch.float64, device=DEV) for k in ("R", "t"))
    x, y, z = (W @ p[0:3] + t.view(3, 1)).unbind(0)
    o = torch.sigmoid(p[10])
    w, i, j, k = torch.nn.functional.normalize(p[6:10], dim=0).unbind(0)
    R = torch.stack([1 - 2 * (j * j + k * k), 2 * (i * j - w * k), 2 * (i * k + w * j),
                     2 * (i * j + w * k), 1 - 2 * (i * i + k * k), 2 * (j * k - w * i),
                     2 * (i * k - w * j), 2 * (j * k + w * i), 1 - 2 * (i * i + j * j)]).view(3, 3, -1)
    vis = z > 0.2
    zs = torch.where(vis, z, torch.ones_like(z))
    lx, ly = 0.65 * cam["width"] / cam["fx"], 0.65 * cam["height"] / cam["fy"]
    ux, uy = (x / zs).clamp(-lx, lx), (y / zs).clamp(-ly, ly)
    T0 = (cam["fx"] / zs) * W[0].view(3, 1) - (cam["fx"] * ux / zs) * W[2].view(3, 1)
    T1 = (cam["fy"] / zs) * W[1].view(3, 1) - (cam["fy"] * uy / zs) * W[2].view(3, 1)
    S = torch.exp(p[3:6])
    U0, U1 = ((T0.unsqueeze(1) * R).sum(0) * S, (T1.unsqueeze(1) * R).sum(0) * S)
    a, b, c = (U0 * U0).sum(0) + 0.3, (U0 * U1).sum(0), (U1 * U1).sum(0) + 0.3
    det = a * c - b * b
    g = torch.stack([cam["fx"] * x / zs + cam["cx"], cam["fy"] * y / zs + cam["cy"], c / det, -b / det, a / det, o, z,
                     p[11], p[12], p[13]], 1)
    return g, vis & (det > 0), 3 * a.sqrt(), 3 * c.sqrt()


def _blend64(g, ids, u, v, K, tgt):
    """Front-to-back blending of g (depth order) at pixel centres u, v:
    colour, depth, T_final, instance channels (K > 0), target probability."""
    dx, dy = u.view(-1, 1) - g[:, 0], v.view(-1, 1) - g[:, 1]
    Q = g[:, 2] * dx * dx + 2 * g[:, 3] * dx * dy + g[:, 4] * dy * dy
    raw = g[:, 5] * torch.exp(-0.5 * Q)
    al = torch.where((Q <= 9) & (raw >= 1 / 255), raw.clamp(max=0.99), torch.zeros_like(raw))
    with torch.no_grad():
        keep = torch.cumprod(1 - al, 1) >= 1e-4
    al = torch.where(keep, al, torch.zeros_like(al))
    T = torch.cumprod(1 - al, 1)
    w = al * torch.cat([torch.ones_like(T[:, :1]), T[:, :-1]], 1)
    out = [w @ g[:, 7:10], w @ g[:, 6], T[:, -1]]
    if K:
        out.append(w @ torch.nn.functional.one_hot(ids, K).to(w.dtype))
    if tgt is not None:
        pt = (w * (ids.view(1, -1) == tgt.view(-1, 1))).sum(1)
        out.append(torch.where(tgt == -1, T[:, -1], pt))
    return out


def _view64(p, ids, cam, K=0, tgt=None, seg=None, win=None, up=None):
    """One view's images, or (with `up`, the gradients of color, depth,
    t_final, then probs or p_target) the gradient with respect to p."""
    W, H = cam["width"], cam["height"]
    lo, n = seg if seg else (0, p.shape[1])
    x0, y0, x1, y1 = win if win else (0, 0, W, H)
    q = p[:, lo:lo + n].detach().clone().requires_grad_(up is not None)
    gall, vis, ex, ey = _project64(q, cam)
    gi = ids[lo:lo + n].long()
    with torch.no_grad():
        vis = vis & (gall[:, 0] + ex > x0) & (gall[:, 0] - ex < x1) & (gall[:, 1] + ey > y0) & (gall[:, 1] - ey < y1)
        sel = vis.nonzero().view(-1)
        sel = sel[torch.sort(gall[sel, 6].float(), stable=True)[1]]
        g, gid, bx, by = gall.detach()[sel], gi[sel], ex.detach()[sel], ey.detach()[sel]
    shapes = [(3,), (), ()] + ([(K,)] if K else []) + ([()] if tgt is not None else [])
    img = [torch.zeros(H, W, *sh, dtype=torch.float64, device=DEV) for sh in shapes]
    img[2][:] = 1.0
    if tgt is not None:
        img[-1][:] = (tgt == -1).double()
    acc = torch.zeros_like(g)
    for yy in range(y0, y1, 32):
        for xx in range(x0, x1, 32):
            ye, xe = min(yy + 32, y1), min(xx + 32, x1)
            k = ((g[:, 0] + bx > xx) & (g[:, 0] - bx < xe) & (g[:, 1] + by > yy) & (g[:, 1] - by < ye)).nonzero().view(-1)
            if not k.numel():
                continue
            v, u = torch.meshgrid(torch.arange(yy, ye, device=DEV) + 0.5, torch.arange(xx, xe, device=DEV) + 0.5,
                                  indexing="ij")
            u, v = u.reshape(-1).double(), v.reshape(-1).double()
            t = tgt[yy:ye, xx:xe].reshape(-1) if tgt is not None else None
            if up is None:
                for im, o in zip(img, _blend64(g[k], gid[k], u, v, K, t)):
                    im[yy:ye, xx:xe] = o.view(ye - yy, xe - xx, *o.shape[1:])
            else:
                gk = g[k].requires_grad_(True)
                outs = _blend64(gk, gid[k], u, v, K, t)
                ups = [a[yy:ye, xx:xe].reshape(o.shape) for a, o in zip(up, outs)]
                acc.index_add_(0, k, torch.autograd.grad(outs, gk, ups)[0])
    if up is None:
        return img
    full = torch.zeros_like(gall)
    full[sel] = acc
    grad = torch.zeros_like(p)
    grad[:, lo:lo + n] = torch.nan_to_num(torch.autograd.grad(gall, q, full)[0])
    return grad


def _loss64(imgs, tgt, jobs, wins):
    """The object loss over views and its gradients (colour, depth, target probability)."""
    cols, deps, ces, masks = 0.0, 0.0, 0.0, []
    nc = nv = no = 0
    for v, (c, d, _, pt) in enumerate(imgs):
        inw = torch.zeros(d.shape, dtype=torch.bool, device=DEV)
        x0, y0, x1, y1 = wins[v] if wins else (0, 0, d.shape[1], d.shape[0])
        inw[y0:y1, x0:x1] = True
        col = inw if jobs[v] < 0 else inw & (tgt["id"][v] == jobs[v])
        val = col & (tgt["depth"][v] > 0)
        dc, dd = c - tgt["color"][v].double().permute(1, 2, 0), d - tgt["depth"][v].double()
        cols, deps = cols + dc[col].abs().sum(), deps + dd[val].abs().sum()
        ces = ces - torch.log(pt[inw].clamp_min(1e-6)).sum()
        nc, nv, no = nc + int(col.sum()), nv + int(val.sum()), no + int(inw.sum())
        masks.append((inw, col, val, dc, dd, pt))
    parts = [cols / max(1, 3 * nc), deps / max(1, nv), ces / max(1, no)]
    ups = [(torch.sign(dc) * col.unsqueeze(-1) / max(1, 3 * nc), torch.sign(dd) * val / max(1, nv),
            torch.zeros_like(dd), torch.where(inw & (pt >= 1e-6), -1.0 / pt.clamp_min(1e-6), torch.zeros_like(pt))
            / max(1, no)) for inw, col, val, dc, dd, pt in masks]
    return torch.stack([sum(parts), *parts]), ups


def _step64(p, ids, cams, tgt, opts):
    """Images, loss and parameter gradient of one training step."""
    V = len(cams)
    seg, win, jobs = opts.get("segments"), opts.get("windows"), opts.get("jobs") or [-1] * V
    tv = [tgt["id"][v] if jobs[v] < 0 else torch.where(tgt["id"][v] == jobs[v], jobs[v], -1) for v in range(V)]
    arg = [dict(tgt=tv[v], seg=seg[v] if seg else None, win=win[v] if win else None) for v in range(V)]
    imgs = [_view64(p, ids, cams[v], **arg[v]) for v in range(V)]
    loss, ups = _loss64(imgs, tgt, jobs, win)
    return imgs, loss, lambda: sum(_view64(p, ids, cams[v], up=ups[v], **arg[v]) for v in range(V))


def _train64(sc, cams, tgt, opts, lrs):
    """The captured step's warm-up step, then the pass: two Adam steps."""
    p = sc["params"].double()
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    lr = torch.tensor(lrs, dtype=torch.float64, device=DEV).view(14, 1)
    for k in (1, 2):
        imgs, loss, grad = _step64(p, sc["ids"], cams, tgt, opts)
        g = grad()
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        p = p - lr * (m / (1 - 0.9 ** k)) / ((v / (1 - 0.999 ** k)).sqrt() + 1e-15)
    st = [torch.stack(x) for x in zip(*imgs)]
    return dict(loss=loss, color=st[0].permute(0, 3, 1, 2).contiguous(), depth=st[1], t_final=st[2], p_target=st[3],
                params=p, m=m, v=v)


def _net64(x, layers):
    """The network in 64 bits: outputs [B][6][S][S]."""
    S = x.shape[-1]
    d = x[:, 3].double()
    ok = (x[:, 4] > 0.5) & (d > 0)
    dmin = torch.where(ok, d, torch.full_like(d, math.inf)).amin((1, 2), keepdim=True)
    rel = torch.where(ok, 4 * (d - dmin) / dmin, torch.zeros_like(d))
    h = torch.cat([x[:, :3].double(), rel.unsqueeze(1), ok.double().unsqueeze(1)], 1).permute(0, 2, 3, 1)
    for i, (w, b) in enumerate(layers):
        h = torch.nn.functional.pad(h, (0, 0, 1, 1, 1, 1))
        h = sum(h[:, dy:dy + S, dx:dx + S] @ w[:, :, dy, dx].T for dy in range(3) for dx in range(3)) + b
        if i < 3:
            h = h.relu()
    return h.permute(0, 3, 1, 2), ok


def _layers64(seed, grad=False):
    return [tuple(torch.tensor(a, dtype=torch.float64, device=DEV).requires_grad_(grad) for a in wb)
            for wb in _theta_layers(seed)]


def _packed(grads):
    """Layer gradients in the library's flat order ([cout_pad][9][cin_pad] and biases, channels padded to 16)."""
    out = []
    for w, b in grads:
        co, ci = w.shape[:2]
        cop, cip = -(-co // 16) * 16, -(-ci // 16) * 16
        blk = torch.zeros(cop, 9, cip, dtype=torch.float64, device=DEV)
        blk[:co, :, :ci] = w.reshape(co, ci, 9).permute(0, 2, 1)
        out += [blk.reshape(-1), torch.nn.functional.pad(b, (0, cop - co))]
    return torch.cat(out)


def _gaussians64(x, b, y, xx, f, cx, cy, opacity):
    d = x[b, 3, y, xx].double()
    n = d.numel()
    p = torch.zeros(14, n, dtype=torch.float64, device=DEV)
    p[0], p[1], p[2] = (xx + 0.5 - cx) / f * d, (y + 0.5 - cy) / f * d, d
    p[3:6] = torch.log(d / f)
    p[6] = 1.0
    p[10] = math.log(opacity / (1 - opacity))
    p[11:14] = x[b, :3, y, xx].T.double()
    return p


def _quadrics64(case, q):
    """Fit by singular value decomposition and 100 Adam steps on the IoU loss."""
    n, V = case["objects"], case["views"]
    Ps, box = q["Ps"].view(V, 3, 4), q["boxes"].view(n, V, 4)
    wh = q["wh"].double()
    Qs = []
    for k in range(n):
        rows = []
        for v in range(V):
            lim = [box[k, v, 0] > 1, box[k, v, 1] > 1, box[k, v, 2] < wh[v, 0] - 1, box[k, v, 3] < wh[v, 1] - 1]
            for e, (on, ax) in enumerate(zip(lim, (0, 1, 0, 1))):
                if bool(on):
                    pi = Ps[v, ax] - box[k, v, e] * Ps[v, 2]
                    pi = pi / pi.norm()
                    a, b, c, d = pi.unbind()
                    rows.append(torch.stack([a * a, 2 * a * b, 2 * a * c, 2 * a * d, b * b, 2 * b * c, 2 * b * d,
                                             c * c, 2 * c * d, d * d]))
        s = torch.linalg.svd(torch.stack(rows).cpu())[2][-1]
        Qk = s[torch.tensor([[0, 1, 2, 3], [1, 4, 5, 6], [2, 5, 7, 8], [3, 6, 8, 9]])]
        Qs.append(Qk / -Qk[3, 3])
    Q = torch.stack(Qs)
    mu = -Q[:, :3, 3]
    ev, R = torch.linalg.eigh(Q[:, :3, :3] + mu.unsqueeze(2) * mu.unsqueeze(1))
    if bool((ev <= 0).any()):
        return None
    R = torch.where((torch.linalg.det(R) < 0).view(-1, 1, 1) & (torch.arange(3) == 0), -R, R)
    Ps, box, wh = Ps.cpu(), box.cpu(), wh.cpu()
    # a unit quaternion of R: the eigenvector of its largest eigenvalue (Bar-Itzhack)
    quat = []
    for M in R:
        N = torch.tensor([[M[0, 0] + M[1, 1] + M[2, 2], M[2, 1] - M[1, 2], M[0, 2] - M[2, 0], M[1, 0] - M[0, 1]],
                          [M[2, 1] - M[1, 2], M[0, 0] - M[1, 1] - M[2, 2], M[1, 0] + M[0, 1], M[2, 0] + M[0, 2]],
                          [M[0, 2] - M[2, 0], M[1, 0] + M[0, 1], M[1, 1] - M[0, 0] - M[2, 2], M[2, 1] + M[1, 2]],
                          [M[1, 0] - M[0, 1], M[2, 0] + M[0, 2], M[2, 1] + M[1, 2], M[2, 2] - M[0, 0] - M[1, 1]]])
        quat.append(torch.linalg.eigh(N)[1][:, 3])
    th = torch.cat([mu, torch.stack(quat), 0.5 * torch.log(ev)], 1)

    def unpack(t):
        w, x, y, z = torch.nn.functional.normalize(t[:, 3:7], dim=1).unbind(1)
        R = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                         2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                         2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).view(-1, 3, 3)
        return t[:, :3], R, torch.exp(t[:, 7:])

    def quadric(t):
        mu, R, ax = unpack(t)
        Z = torch.eye(4, dtype=torch.float64).expand(n, 4, 4).clone()
        Z[:, :3, :3], Z[:, :3, 3] = R, mu
        D = torch.cat([ax * ax, -torch.ones(n, 1, dtype=torch.float64)], 1)
        return (Z * D.unsqueeze(1)) @ Z.transpose(1, 2)

    def ious(t):
        C = torch.einsum("vai,nij,vbj->nvab", Ps, quadric(t), Ps)
        c = C / C[..., 2:, 2:]
        dx2, dy2 = c[..., 0, 2] ** 2 - c[..., 0, 0], c[..., 1, 2] ** 2 - c[..., 1, 1]
        ok = (C[..., 2, 2] < 0) & (dx2 > 0) & (dy2 > 0)
        dx, dy = torch.where(ok, dx2, 1.0).sqrt(), torch.where(ok, dy2, 1.0).sqrt()
        lim = torch.cat([wh, wh], 1)
        b = torch.stack([c[..., 0, 2] - dx, c[..., 1, 2] - dy, c[..., 0, 2] + dx, c[..., 1, 2] + dy], -1)
        b = torch.minimum(b.clamp_min(0), lim)
        iw = torch.minimum(b[..., 2], box[..., 2]) - torch.maximum(b[..., 0], box[..., 0])
        ih = torch.minimum(b[..., 3], box[..., 3]) - torch.maximum(b[..., 1], box[..., 1])
        inter = iw.clamp_min(0) * ih.clamp_min(0)
        area = lambda r: (r[..., 2] - r[..., 0]) * (r[..., 3] - r[..., 1])  # noqa: E731
        return torch.where(ok, inter / (area(b) + area(box) - inter), torch.zeros_like(inter))

    m, v, first = torch.zeros_like(th), torch.zeros_like(th), None
    for k in range(1, 101):
        th = th.detach().requires_grad_(True)
        J = (1 - ious(th)).sum(1)
        first = J.detach() if first is None else first
        g, = torch.autograd.grad(J.sum(), th)
        with torch.no_grad():
            m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
            th = th - 0.01 * (m / (1 - 0.9 ** k)) / ((v / (1 - 0.999 ** k)).sqrt() + 1e-15)
    th = th.detach()
    mu, R, ax = unpack(th)
    iou = ious(th)
    return dict(status=None, mu=mu, R=None, axes=ax, Q=quadric(th), loss=torch.stack([first, (1 - iou).sum(1)], 1),
                iou=iou.reshape(-1))


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        sc = _scene(case, seed)
        opts, tgt, cams = _jobs(sc, case, _observed(sc, case, seed))
        return _train64(sc, cams, tgt, opts, _late_lrs())
    if kind == "crops":
        sc, tgt, seg = _crop_scene(case, seed)
        return _train64(sc, sc["cams"], tgt, dict(segments=seg), _late_lrs(0.3))
    if kind == "autograd":
        sc = _scene(case, seed)
        K = sc["K"] if case["probs"] else 0
        p, cam = sc["params"].double(), sc["cams"][0]
        img = _view64(p, sc["ids"], cam, K=K)
        up = [g[0].double() for g in _upstream(case, sc["K"], seed)]
        up = [up[0].permute(1, 2, 0), up[1], up[2]] + ([up[3].permute(1, 2, 0)] if K else [])
        return dict(color=img[0].permute(2, 0, 1)[None].contiguous(), depth=img[1][None], t_final=img[2][None],
                    probs=img[3].permute(2, 0, 1)[None].contiguous() if K else None,
                    grad=_view64(p, sc["ids"], cam, K=K, up=up))
    if kind == "tracking":
        sc = _scene(case, seed)
        cam, tgt = _tracking_cam(sc["cams"][0]), _observed(sc, case, seed)
        p = sc["params"].double()
        imgs, loss, grad = _step64(p, sc["ids"], [cam], tgt, {})
        g = grad()
        # moving the camera renders what moving every Gaussian by the inverse motion renders
        R, t = (torch.tensor(cam[k], dtype=torch.float64, device=DEV) for k in ("R", "t"))
        pc, gc = R @ p[0:3] + t.view(3, 1), R @ g[0:3]
        s, u, ds, du = p[6], p[7:10], g[6], g[7:10]
        phi = 0.5 * (-u * ds + s * du + torch.linalg.cross(u, du, dim=0))
        pose = torch.cat([(torch.linalg.cross(pc, gc, dim=0) + R @ phi).sum(1), gc.sum(1)])
        c, d, T, _ = imgs[0]
        return dict(loss=loss, pose=pose.view(1, 6), color=c.permute(2, 0, 1)[None].contiguous(), depth=d[None],
                    t_final=T[None])
    if kind == "ids":
        sc = _scene(case, seed)
        img = _view64(sc["params"].double(), sc["ids"], sc["cams"][0], K=sc["K"])
        return dict(color=img[0].permute(2, 0, 1)[None].contiguous(), depth=img[1][None], t_final=img[2][None],
                    probs=img[3].permute(2, 0, 1)[None].contiguous(), id_map=None, obj=None, view=None, boxes=None)
    if kind == "net_train":
        x, lab, ly = _crops(case, seed), _labels(case, seed).double(), _layers64(seed, True)
        out, ok = _net64(x, ly)
        cw = torch.tensor(CHAN_W, dtype=torch.float64, device=DEV).view(1, 5, 1, 1)
        s = (cw * (out[:, :5] - lab) ** 2).sum(1)
        all_ = s + (out[:, 5] - torch.log(s.detach() + 1e-4)) ** 2
        M = max(1, int(ok.sum()))
        loss = all_[ok].sum() / M
        flat = torch.autograd.grad(loss, [a for wb in ly for a in wb])
        return dict(out=out.detach(), loss=torch.stack([loss, s[ok].sum() / M]).detach(),
                    grad=_packed(list(zip(flat[0::2], flat[1::2]))))
    if kind == "net_start":
        x = _crops(case, seed)
        out, ok = _net64(x, _layers64(seed))
        b, y, xx = ok.nonzero(as_tuple=True)
        S = case["size"]
        mean = torch.stack([out[i, 5][ok[i]].mean() for i in range(case["crops"])])
        p = _gaussians64(x, b, y, xx, 110.0, S / 2, S / 2, 0.9)
        p[3:6] += out[b, 0, y, xx]
        p[10] = out[b, 1, y, xx]
        p[11:14] += out[b, 2:5, y, xx].T
        return dict(out=out, use=None, mean=mean, params=p, ids=None)
    if kind == "quadrics":
        return _quadrics64(case, _quadric_inputs(case, seed))
    cams, tgt, img = _increment_inputs(case, seed)
    idt, obs = tgt["id"], tgt["depth"] > 0
    has = (idt >= 0) & (idt <= case["objects"])
    geo = has & ((img["p_target"].double() < 0.5) | (obs & ((img["depth"].double() - tgt["depth"].double()).abs() > 0.1)))
    rgb = has & ((img["color"].double() - tgt["color"].double()).abs().mean(1) > 0.1)
    v, y, x = (obs & (geo | rgb)).nonzero(as_tuple=True)
    src = torch.cat([tgt["color"], tgt["depth"].unsqueeze(1)], 1)
    f, W, H = cams[0]["fx"], case["width"], case["height"]
    p = _gaussians64(src, v, y, x, f, W / 2, H / 2, 0.9)
    p[10] = torch.where(geo[v, y, x], p[10], -p[10])
    Rt = torch.tensor(np.stack([c["R"].T for c in cams]), dtype=torch.float64, device=DEV)[v]
    t = torch.tensor(np.stack([c["t"] for c in cams]), dtype=torch.float64, device=DEV)[v]
    p[0:3] = (Rt @ (p[0:3].T - t).unsqueeze(2))[:, :, 0].T
    full = torch.zeros(14, case["views"] * W * H // 2, dtype=torch.float64, device=DEV)
    k = min(p.shape[1], full.shape[1])
    full[:, :k] = p[:, :k]
    return dict(masks=None, obj=None, params=full, ids=None, counts=None)
