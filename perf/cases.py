"""Workloads of the framework's public entry points, for timing and for comparing outputs.

Every case names a kind of call and its sizes; the inputs are synthetic and
made from the seed alone, with the distributions of the benchmark's scenes (64
anisotropic clusters and 10% background, log-scales N(-4.5, 0.7^2), opacities
sigmoid(N(0.5, 1.5^2)), views on a jittered orbit).

  pass       gs.sensitivity on one scene and its views (projection, depth
             sort, binning, both compositing passes)
  plan       one run of a gs.Plan over several uneven scenes (graph replay)
  objective  gs.render_objective of a weighted draw on every ray
  judge      the same on 1% of the 8x8 pixel blocks, and gs.coreset_error of
             its per-view sums: how a draw is judged
  sample     gs.sample_coreset on sensitivities that are there
  features   learned.features and learned.feature_stats of a scene
  predict    Proposal.predict and learned.mixture over every Gaussian
  train      Proposal.train_step on one batch
"""
import math
import types

import numpy as np
import torch

import paper_2607_02721_amd as gs
from paper_2607_02721_amd import learned

MODES = {"rgbsum": gs.QUERY_RGBSUM, "nocolor": gs.QUERY_NOCOLOR, "l2": gs.QUERY_L2, "channel": gs.QUERY_CHANNEL}
AGGREGATES = {"ray": gs.AGG_RAY, "tile": gs.AGG_TILE, "image": gs.AGG_IMAGE, "scene": gs.AGG_SCENE}
OBJECTIVES = {"full": gs.OBJ_FULL, "fixed": gs.OBJ_FIXED}

# Bounds of the drawn sizes, and the (Gaussian, view, pixel) work of the
# largest listed pass, which no drawn case exceeds.
N_LO, N_HI = 2_000, 1_000_000
PIXELS_720P = 1280 * 720
WORK_HI = 1_000_000 * 100


def _pass(name, n, views, width, height, *, degree=3, fmt="f32", mode="rgbsum", aggregate="ray", tile="16x16"):
    return {"name": name, "kind": "pass", "n": n, "views": views, "width": width, "height": height, "degree": degree,
            "fmt": fmt, "mode": mode, "aggregate": aggregate, "tile": tile}


def listed():
    return [
        # a scene of a test or a preview: launches and host time count
        _pass("pass_tiny", 2_000, 4, 64, 64, degree=0),
        # the small end of a batch of captured scenes, one call, default tile
        _pass("pass_small", 50_000, 24, 640, 360),
        # a full scene, every view in one call, with the tuned binning tile
        _pass("pass_scene", 1_000_000, 100, 1280, 720, tile="32x32"),
        # half-size storage, photographs of an odd size, the default tile
        _pass("pass_odd_mixed16", 437_113, 13, 1237, 823, fmt="mixed16"),
        # per-image queries (aggregated objectives), ordinary sizes
        _pass("pass_image", 250_000, 20, 960, 540, aggregate="image", tile="32x32"),
        # several uneven scenes as one plan, replayed as pruning rounds do
        {"name": "plan_batch", "kind": "plan", "scenes": 4, "n_lo": 50_000, "n_hi": 400_000, "views": 16,
         "width": 1280, "height": 720, "tile": "16x16"},
        # the weighted objective on every ray: the full-resolution judge
        {"name": "objective_rays", "kind": "objective", "n": 300_000, "views": 20, "width": 1280, "height": 720,
         "degree": 3, "mode": "rgbsum", "objective": "fixed", "m_frac": 0.1, "tile": "16x16"},
        # the cheap judge of a draw: 1% of the 8x8 blocks of every view
        {"name": "judge_blocks", "kind": "judge", "n": 1_000_000, "views": 100, "width": 1280, "height": 720,
         "degree": 3, "mode": "rgbsum", "objective": "fixed", "m_frac": 0.1, "tile": "16x16"},
        # a draw of 10% from the sensitivities of a full scene
        {"name": "sample_scene", "kind": "sample", "n": 1_000_000, "m": 100_000},
        # the proposal's inputs for a full scene
        {"name": "features_scene", "kind": "features", "n": 1_000_000, "degree": 3, "fmt": "f32"},
        # the proposal's scores for a full scene
        {"name": "predict_scene", "kind": "predict", "n": 1_000_000},
        # one training step at the default batch
        {"name": "train_batch", "kind": "train", "n": 16_384},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo=64, hi=1920):
    width = _log_uniform(rng, lo, hi)
    return width, max(32, int(width * rng.uniform(0.5, 0.8)))


def _views_for(rng, n, width, height, lo=2, hi=100, work=WORK_HI):
    most = int(work / max(1.0, n * max(0.05, width * height / PIXELS_720P)))
    return max(1, min(_log_uniform(rng, lo, hi), most))


def draw(rng):
    kind = rng.choice(["pass"] * 6 + ["plan"] + ["objective"] * 2 + ["judge"] + ["sample"] * 2 + ["features"] * 2 +
                      ["predict", "train", "train"])
    n = _log_uniform(rng, N_LO, N_HI)
    if kind == "sample":
        return {"kind": kind, "n": n, "m": max(1, int(n * math.exp(rng.uniform(math.log(0.01), math.log(2.0)))))}
    if kind == "features":
        return {"kind": kind, "n": n, "degree": rng.choice([0, 1, 2, 3, 3, 3]),
                "fmt": rng.choice(["f32", "f32", "mixed16"])}
    if kind == "predict":
        return {"kind": kind, "n": n}
    if kind == "train":
        return {"kind": kind, "n": _log_uniform(rng, 256, 65_536)}
    width, height = _size(rng)
    if kind == "plan":
        hi = max(10_000, n // 4)
        return {"kind": kind, "scenes": rng.randint(2, 5), "n_lo": max(1_000, int(hi * rng.uniform(0.05, 0.5))),
                "n_hi": hi, "views": _views_for(rng, hi, width, height, 4, 24, 2e7), "width": width,
                "height": height, "tile": rng.choice(["16x16", "32x32"])}
    tile = rng.choice(["16x16"] * 3 + ["32x32"] * 3 + ["16x32", "32x16", "8x16"])
    mode = rng.choice(["rgbsum"] * 4 + ["nocolor", "l2"])
    degree = rng.choice([0, 1, 2, 3, 3, 3, 3])
    if kind in ("objective", "judge"):
        work = WORK_HI if kind == "judge" else WORK_HI / 8
        return {"kind": kind, "n": n, "views": _views_for(rng, n, width, height, 2, 60, work), "width": width,
                "height": height, "degree": degree, "mode": mode, "objective": "fixed",
                "m_frac": rng.choice([0.01, 0.05, 0.1, 0.2]), "tile": tile}
    aggregate = rng.choice(["ray"] * 5 + ["tile", "image", "scene"])
    if aggregate == "ray" and rng.random() < 0.15:
        mode = "channel"
    if aggregate == "tile" and "8" in tile:
        tile = "16x16"
    return {"kind": kind, "n": n, "views": _views_for(rng, n, width, height, 2, 100, WORK_HI / 2), "width": width,
            "height": height, "degree": degree, "fmt": rng.choice(["f32", "f32", "mixed16"]), "mode": mode,
            "aggregate": aggregate, "tile": tile}


# --- inputs ---------------------------------------------------------------

def _generator(seed, stream):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 1009 + stream)


def _unit_quats(g, n):
    q = torch.randn(4, n, generator=g, device="cuda", dtype=torch.float64)
    return q / q.norm(dim=0, keepdim=True)


def _rotations(q):
    w, x, y, z = q
    return torch.stack([torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)]),
                        torch.stack([2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)]),
                        torch.stack([2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)])]).permute(2, 0, 1)


def _scene_planes(n, degree, seed, stream=0):
    """float32 device planes (mean, log_scale, quat, opacity, sh) of a clustered scene."""
    g = _generator(seed, 17 + stream)
    f = dict(generator=g, device="cuda", dtype=torch.float64)
    clusters = 64
    centres = torch.rand(clusters, 3, **f) * 1.4 - 0.7
    weights = -torch.log(torch.rand(clusters, **f).clamp_min(1e-12))
    sig = 0.02 + 0.18 * torch.rand(clusters, 3, **f)
    rot = _rotations(_unit_quats(g, clusters))
    n_bg = int(round(0.1 * n))
    which = torch.bucketize(torch.rand(n - n_bg, **f), torch.cumsum(weights / weights.sum(), 0)).clamp_max(clusters - 1)
    z = torch.randn(n - n_bg, 3, **f) * sig[which]
    pts = centres[which] + (rot[which] * z[:, None, :]).sum(-1)
    pts = torch.cat([pts, torch.rand(n_bg, 3, **f) * 2 - 1])[torch.randperm(n, generator=g, device="cuda")]
    k = (degree + 1) ** 2
    sh = torch.randn(k, 3, n, **f) * 0.1
    sh[0] = (torch.rand(3, n, **f) - 0.5) / 0.28209479177387814
    log_scale = torch.randn(3, n, **f) * 0.7 - 4.5
    if degree == 0 and n <= 4_000:   # the small scene: fewer, larger Gaussians
        log_scale = torch.randn(3, n, **f) * 0.5 - 3.5
    opacity = torch.sigmoid(0.5 + 1.5 * torch.randn(n, **f))
    return [t.float().contiguous() for t in (pts.T, log_scale, _unit_quats(g, n), opacity, sh)]


def _stored(planes, fmt):
    if fmt == "f32":
        return planes
    kinds = (torch.bfloat16, torch.bfloat16, torch.float16, torch.float16, torch.bfloat16)
    return [p.to(k).contiguous() for p, k in zip(planes, kinds)]


def _scene(n, degree, fmt, seed, stream=0):
    return gs.DeviceScene(*_stored(_scene_planes(n, degree, seed, stream), fmt), degree,
                          gs.ATTR_MIXED16 if fmt == "mixed16" else gs.ATTR_F32)


def _views(count, width, height, seed, stream=0):
    """Cameras on a jittered orbit of radius 3 that look at the scene's middle (host arrays)."""
    rng = np.random.default_rng([int(seed), 23, stream])
    w2c, intr, size = [], [], []
    for k in range(count):
        az = 2 * math.pi * (k + rng.uniform(-0.5, 0.5)) / count
        el = math.radians(15 + rng.uniform(-10, 10))
        target = rng.normal(0, 0.02, 3)
        eye = target + 3 * (1 + rng.uniform(-0.05, 0.05)) * np.array(
            [math.cos(el) * math.cos(az), math.cos(el) * math.sin(az), math.sin(el)])
        forward = (target - eye) / np.linalg.norm(target - eye)
        right = np.cross(forward, [0.0, 0.0, 1.0])
        right /= np.linalg.norm(right)
        R = np.stack([right, np.cross(forward, right), forward])
        w2c.append(np.concatenate([R, (-R @ eye)[:, None]], 1).reshape(12))
        fx = width / 2 / math.tan(math.radians(30))
        intr.append([fx, fx, width / 2, height / 2])
        size.append([width, height])
    return types.SimpleNamespace(world_to_cam=np.array(w2c), intrinsics=np.array(intr),
                                 size=np.array(size, dtype=np.int32))


def _draw_weights(planes, m, seed):
    """Weights n_i / (m p_i) of m draws from a proposal that favours large, opaque Gaussians."""
    g = _generator(seed, 31)
    p = planes[3].double() * torch.exp(planes[1].double().mean(0)) + 1e-4
    p = p / p.sum()
    cdf = torch.cumsum(p, 0)
    hits = torch.bucketize(torch.rand(m, generator=g, device="cuda", dtype=torch.float64), cdf).clamp_max(p.numel() - 1)
    counts = torch.bincount(hits, minlength=p.numel()).double()
    return (counts / (m * p)).contiguous()


def _block_keep(case, seed):
    """Per view, which 8x8 pixel blocks are judged (1% of them): bool [views][blocks y][blocks x]."""
    by, bx = (case["height"] + 7) // 8, (case["width"] + 7) // 8
    keep = torch.rand(case["views"], by, bx, generator=_generator(seed, 37), device="cuda") < 0.01
    keep[:, by // 2, bx // 2] = True
    return keep


def _ray_mask(case, seed):
    keep = _block_keep(case, seed)
    parts = [k.repeat_interleave(8, 0)[:case["height"]].repeat_interleave(8, 1)[:, :case["width"]].reshape(-1)
             for k in keep]
    bits = torch.cat(parts)
    bits = torch.cat([bits, bits.new_zeros(-bits.numel() % 32)]).view(-1, 8).to(torch.uint8)
    words = (bits << torch.arange(8, device="cuda", dtype=torch.uint8)).sum(1, dtype=torch.uint8)
    return words.view(torch.int32)


def _feature_rows(n, seed):
    """Rows of raw features and their normalisation, with the scales of a real scene's columns."""
    g = _generator(seed, 41)
    scale = torch.cat([torch.full((3,), 0.5), torch.full((3,), 0.7), torch.full((4,), 0.5), torch.tensor([1.5]),
                       torch.full((3,), 1.0), torch.full((45,), 0.1), torch.tensor([0.8, 0.8, 0.1, 0.1, 2.0])]).cuda()
    shift = torch.cat([torch.zeros(3), torch.full((3,), -4.5), torch.zeros(4), torch.tensor([0.5]), torch.zeros(48),
                       torch.tensor([-4.0, -3.6, 0.6, 0.95, 9.0])]).cuda()
    feat = torch.randn(n, 64, generator=g, device="cuda") * scale + shift
    return feat.contiguous(), torch.stack([shift, 1 / scale]).contiguous()


def _mlp_params(seed):
    """Network parameters as initialisation leaves them (uniform weights by fan-in and fan-out), small biases."""
    g = _generator(seed, 47)
    parts = []
    for rows, cols in ((256, 64), (256, 256), (256, 256), (1, 256)):
        a = math.sqrt(6.0 / (rows + cols))
        parts += [(torch.rand(rows * cols, generator=g, device="cuda") * 2 - 1) * a,
                  torch.randn(rows, generator=g, device="cuda") * 0.02]
    return torch.cat(parts)


def _targets(feat, norm, seed):
    z = (feat - norm[0]) * norm[1]
    return (-6 + 1.5 * torch.tanh(z[:, 3]) + z[:, 10] - 0.5 * z[:, 59] * z[:, 62]).contiguous()


def _shares(n, seed):
    """Sensitivities as a pass leaves them: many zeros, a long tail, some near 1."""
    g = _generator(seed, 43)
    s = torch.exp(-3.5 * torch.randn(n, generator=g, device="cuda").abs())
    return torch.where(torch.rand(n, generator=g, device="cuda") < 0.3, torch.zeros_like(s), s).contiguous()


def _plan_parts(case):
    """(Gaussians, views) of each scene: sizes spread over the case's range, the views over a factor of two."""
    k = case["scenes"]
    out = []
    for i in range(k):
        t = i / max(1, k - 1)
        n = int(round(case["n_lo"] ** (1 - t) * case["n_hi"] ** t))
        out.append((n, max(1, int(round(case["views"] * (1 - 0.5 * ((i * 2) % k) / k))))))
    return out


def _tile(case):
    w, h = case["tile"].split("x")
    return int(w), int(h)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "pass":
        return {"case": case, "scene": _scene(case["n"], case["degree"], case["fmt"], seed),
                "views": _views(case["views"], case["width"], case["height"], seed)}
    if kind == "plan":
        parts = _plan_parts(case)
        scenes = [_scene(n, 3, "f32", seed, 100 * i) for i, (n, _) in enumerate(parts)]
        views = [_views(v, case["width"], case["height"], seed, 100 * i) for i, (_, v) in enumerate(parts)]
        return {"case": case, "plan": gs.Plan(scenes, views, tile=_tile(case))}
    if kind in ("objective", "judge"):
        planes = _scene_planes(case["n"], case["degree"], seed)
        return {"case": case, "scene": gs.DeviceScene(*planes, case["degree"]),
                "views": _views(case["views"], case["width"], case["height"], seed),
                "weights": _draw_weights(planes, max(1, int(case["m_frac"] * case["n"])), seed),
                "mask": _ray_mask(case, seed) if kind == "judge" else None}
    if kind == "sample":
        return {"case": case, "sens": _shares(case["n"], seed), "seed": int(seed)}
    if kind == "features":
        return {"case": case, "scene": _scene(case["n"], case["degree"], case["fmt"], seed)}
    if kind in ("predict", "train"):
        feat, norm = _feature_rows(case["n"], seed)
        prop = learned.Proposal(seed=int(seed))
        prop.set_norm(norm)
        prop.params.copy_(_mlp_params(seed))
        state = {"case": case, "prop": prop, "feat": feat}
        if kind == "train":
            state["targets"] = _targets(feat, norm, seed)
            state["grad"] = torch.empty_like(prop.params)
        return state
    raise ValueError(kind)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "pass":
        return gs.sensitivity(state["scene"], state["views"], query_mode=MODES[case["mode"]],
                              aggregate=AGGREGATES[case["aggregate"]], tile=_tile(case))[0]
    if kind == "plan":
        return state["plan"].run()
    if kind == "objective":
        out = gs.render_objective(state["scene"], state["views"], state["weights"], OBJECTIVES[case["objective"]],
                                  query_mode=MODES[case["mode"]], diag=False, tile=_tile(case))
        return {"per_ray": out["per_ray"], "per_view": out["per_view"]}
    if kind == "judge":
        out = gs.render_objective(state["scene"], state["views"], state["weights"], OBJECTIVES[case["objective"]],
                                  query_mode=MODES[case["mode"]], ray_mask=state["mask"], per_ray=False, diag=False,
                                  tile=_tile(case))
        return {"per_view": out["per_view"], "error": gs.coreset_error(out["per_view"])}
    if kind == "sample":
        counts, weights, support = gs.sample_coreset(state["sens"], case["m"], state["seed"])
        return {"counts": counts, "weights": weights, "support": support}
    if kind == "features":
        feat = learned.features(state["scene"])
        return {"features": feat, "stats": learned.feature_stats(feat)}
    if kind == "predict":
        y = state["prop"].predict(state["feat"])
        return {"log_s": y, "scores": learned.mixture(y)}
    if kind == "train":
        loss = state["prop"].train_step(state["feat"], state["targets"], lr=1e-3, grad=state["grad"])
        return {"loss": loss, "grad": state["grad"], "params": state["prop"].params, "adam": state["prop"].adam}
    raise ValueError(kind)


# --- work -------------------------------------------------------------------

MLP_FLOP_PER_ROW = 2 * (64 * 256 + 256 * 256 + 256 * 256 + 256)
MLP_PARAMS = 64 * 256 + 256 + 2 * (256 * 256 + 256) + 257


def _gaussian_bytes(degree, fmt):
    return (11 + 3 * (degree + 1) ** 2) * (2 if fmt == "mixed16" else 4)


def _scene_flops(n, views, width, height, passes, share=1.0):
    """Projection (about 300 operations per Gaussian and view) and compositing: about 105 (Gaussian, pixel)
    pairs per Gaussian and view at 1280x720, of which a ray needs about 115 at most, 16 operations each."""
    rays = float(views) * width * height * share
    pairs = min(115.0 * rays, 105.0 * n * views * (width * height / PIXELS_720P) * share)
    return 300.0 * n * views + 16.0 * pairs * passes


def work(case):
    kind = case["kind"]
    if kind == "pass":
        n = case["n"]
        return {"bytes": n * (_gaussian_bytes(case["degree"], case["fmt"]) + 4.0),
                "flops": _scene_flops(n, case["views"], case["width"], case["height"], 2)}
    if kind == "plan":
        parts = _plan_parts(case)
        return {"bytes": sum(n * (_gaussian_bytes(3, "f32") + 4.0) for n, _ in parts),
                "flops": sum(_scene_flops(n, v, case["width"], case["height"], 2) for n, v in parts)}
    if kind in ("objective", "judge"):
        n, rays = case["n"], float(case["views"]) * case["width"] * case["height"]
        return {"bytes": n * (_gaussian_bytes(case["degree"], "f32") + 8.0) + (4 * rays if kind == "objective" else rays / 8),
                "flops": _scene_flops(n, case["views"], case["width"], case["height"], 1,
                                      1.0 if kind == "objective" else 0.01)}
    if kind == "sample":
        n, m = case["n"], case["m"]
        return {"bytes": n * (4.0 + 4.0 + 8.0), "flops": 10.0 * n + m * (100.0 + 2 * math.log2(n + 1))}
    if kind == "features":
        n = case["n"]
        return {"bytes": n * (_gaussian_bytes(case["degree"], case["fmt"]) + 256.0), "flops": n * (16 * 8 * 8 + 200.0)}
    n = case["n"]
    if kind == "predict":
        return {"bytes": n * (256.0 + 8.0), "flops": float(n) * MLP_FLOP_PER_ROW}
    return {"bytes": n * 260.0 + MLP_PARAMS * 4.0 * 7, "flops": 3.0 * n * MLP_FLOP_PER_ROW}


# --- the same in 64 bits ----------------------------------------------------

def _sh_colours(planes, degree, cam):
    d = planes[0] - cam[:, None]
    x, y, z = d / d.norm(dim=0, keepdim=True)
    xx, yy, zz = x * x, y * y, z * z
    Y = [torch.full_like(x, 0.28209479177387814), 0.48860251190291992 * y, 0.48860251190291992 * z,
         0.48860251190291992 * x, 1.0925484305920792 * x * y, 1.0925484305920792 * y * z,
         0.31539156525252005 * (3 * zz - 1), 1.0925484305920792 * x * z, 0.54627421529603959 * (xx - yy),
         0.59004358992664352 * y * (3 * xx - yy), 2.8906114426405538 * x * y * z,
         0.45704579946446572 * y * (5 * zz - 1), 0.37317633259011540 * z * (5 * zz - 3),
         0.45704579946446572 * x * (5 * zz - 1), 1.4453057213202769 * z * (xx - yy),
         0.59004358992664352 * x * (xx - 3 * yy)]
    c = torch.zeros(3, x.numel(), dtype=torch.float64, device=x.device)
    for k in range((degree + 1) ** 2):
        c += Y[k][None] * planes[4][k]
    return (c + 0.5).clamp_min(0)


def _project(planes, degree, views, v):
    """One view's Gaussians front to back: index, mean, conic, alpha, colours and pixel bounds, in 64 bits."""
    P = torch.tensor(views.world_to_cam[v].reshape(3, 4), dtype=torch.float64, device="cuda")
    fx, fy, cx, cy = (float(t) for t in views.intrinsics[v])
    W, H = (int(t) for t in views.size[v])
    R, t = P[:, :3], P[:, 3]
    p = R @ planes[0] + t[:, None]
    x, y, z = p
    ok = z > 0.2
    z = torch.where(ok, z, torch.ones_like(z))
    q = planes[2] / planes[2].norm(dim=0, keepdim=True)
    M = _rotations(q) * torch.exp(planes[1]).T[:, None, :]
    zero = torch.zeros_like(z)
    J = torch.stack([torch.stack([fx / z, zero, -fx * x / z ** 2]), torch.stack([zero, fy / z, -fy * y / z ** 2])])
    half = (J.permute(2, 0, 1)[:, :, :, None] * R[None, None]).sum(2)           # [n][2][3]: J R
    half = (half[:, :, :, None] * M[:, None]).sum(2)                            # J R M
    sxx = (half[:, 0] ** 2).sum(1) + float(np.float32(0.3))
    syy = (half[:, 1] ** 2).sum(1) + float(np.float32(0.3))
    sxy = (half[:, 0] * half[:, 1]).sum(1)
    det = sxx * syy - sxy ** 2
    mx, my = fx * x / z + cx, fy * y / z + cy
    rx, ry = 3 * sxx.sqrt(), 3 * syy.sqrt()
    ok &= (det > 0) & (mx + rx >= 0.5) & (mx - rx <= W - 0.5) & (my + ry >= 0.5) & (my - ry <= H - 0.5)
    index = torch.nonzero(ok).flatten()
    index = index[torch.sort(z[index].float(), stable=True).indices]
    c = _sh_colours(planes, degree, -(R.T @ t))
    pick = lambda a: a[index]  # noqa: E731
    return {"index": index, "mx": pick(mx), "my": pick(my), "rx": pick(rx), "ry": pick(ry), "a": pick(syy / det),
            "b": pick(-sxy / det), "c": pick(sxx / det), "alpha": pick(planes[3]), "rgb": c[:, index]}


def _blocks(case, seed, v):
    W, H = case["width"], case["height"]
    if case["kind"] == "judge":
        for by, bx in torch.nonzero(_block_keep(case, seed)[v]).tolist():
            yield 8 * bx, min(8 * bx + 8, W), 8 * by, min(8 * by + 8, H)
        return
    for y0 in range(0, H, 64):
        for x0 in range(0, W, 64):
            yield x0, min(x0 + 64, W), y0, min(y0 + 64, H)


def _contributions(g, box, mode):
    """(which of the view's Gaussians, their contributions to each pixel of the box [queries][K][h][w])."""
    x0, x1, y0, y1 = box
    near = torch.nonzero((g["mx"] + g["rx"] >= x0) & (g["mx"] - g["rx"] <= x1) & (g["my"] + g["ry"] >= y0) &
                         (g["my"] - g["ry"] <= y1)).flatten()
    col = lambda name: g[name][near][:, None]  # noqa: E731
    dx = torch.arange(x0, x1, device="cuda", dtype=torch.float64)[None] + 0.5 - col("mx")
    dy = torch.arange(y0, y1, device="cuda", dtype=torch.float64)[None] + 0.5 - col("my")
    d2 = (col("a") * dx * dx)[:, None, :] + (2 * col("b") * dx)[:, None, :] * dy[:, :, None] + (col("c") * dy * dy)[:, :, None]
    rho = torch.where(d2 <= 9.0, col("alpha")[:, :, None] * torch.exp(-0.5 * d2), torch.zeros_like(d2))
    T = torch.cumprod(1 - rho, 0)
    rt = rho * torch.cat([torch.ones_like(T[:1]), T[:-1]]) if near.numel() else rho
    rgb = g["rgb"][:, near][:, :, None, None]
    if mode == "nocolor":
        a = rt[None]
    elif mode == "l2":
        a = ((rgb ** 2).sum(0) * rt ** 2)[None]
    elif mode == "channel":
        a = rgb * rt[None]
    else:
        a = (rgb.sum(0) * rt)[None]
    return near, a


def _ratio(a, A):
    return torch.where(A > 0, a / torch.where(A > 0, A, torch.ones_like(A)), torch.zeros_like(a))


def _exact_pass(planes, degree, views, case, seed):
    n, agg = planes[3].numel(), case.get("aggregate", "ray")
    s = torch.zeros(n, dtype=torch.float64, device="cuda")
    num, den = torch.zeros_like(s), 0.0
    for v in range(len(views.size)):
        g = _project(planes, degree, views, v)
        for box in _blocks(case, seed, v):
            near, a = _contributions(g, box, case.get("mode", "rgbsum"))
            if not near.numel():
                continue
            ids = g["index"][near]
            if agg == "ray":
                for part in a:
                    s.index_reduce_(0, ids, _ratio(part, part.sum(0, keepdim=True)).amax((1, 2)), "amax")
            elif agg == "tile":
                pad = torch.nn.functional.pad(a[0], (0, -a.shape[3] % 16, 0, -a.shape[2] % 16))
                pad = pad.view(pad.shape[0], pad.shape[1] // 16, 16, pad.shape[2] // 16, 16).sum((2, 4))
                s.index_reduce_(0, ids, _ratio(pad, pad.sum(0, keepdim=True)).amax((1, 2)), "amax")
            else:
                num.index_add_(0, ids, a[0].sum((1, 2)))
        if agg == "image":
            s = torch.maximum(s, num / num.sum().clamp_min(1e-300))
            num.zero_()
    if agg == "scene":
        s = num / num.sum().clamp_min(1e-300)
    return s


def _exact_objective(planes, degree, views, weights, case, seed):
    rays = case["width"] * case["height"]
    per_ray = torch.zeros(len(views.size), rays, dtype=torch.float64, device="cuda")
    per_view = torch.zeros(len(views.size), 3, dtype=torch.float64, device="cuda")
    for v in range(len(views.size)):
        g = _project(planes, degree, views, v)
        image = per_ray[v].view(case["height"], case["width"])
        for box in _blocks(case, seed, v):
            near, a = _contributions(g, box, case["mode"])
            if not near.numel():
                continue
            A = a[0].sum(0)
            Aw = (weights[g["index"][near]][:, None, None] * a[0]).sum(0)
            image[box[2]:box[3], box[0]:box[1]] = A if case["objective"] == "full" else Aw
            per_view[v, 0] += A.sum()
            per_view[v, 1] += Aw.sum()
    return per_ray.reshape(-1), per_view


def _exact_features(planes, degree):
    n = planes[3].numel()
    feat = torch.zeros(n, 64, dtype=torch.float64, device="cuda")
    q = planes[2] / planes[2].norm(dim=0, keepdim=True)
    feat[:, 0:3], feat[:, 3:6] = planes[0].T, planes[1].T
    feat[:, 6:10] = (q * torch.where(planes[2][0] < 0, -1.0, 1.0)).T
    alpha = planes[3].clamp(1e-6, 1 - 1e-6)
    feat[:, 10] = torch.log(alpha / (1 - alpha))
    k = 3 * (degree + 1) ** 2
    feat[:, 11:11 + k] = planes[4].reshape(k, n).T
    pts = planes[0].T.contiguous()
    for i in range(0, n, 2048):
        rows = pts[i:i + 2048]
        d2 = sum((rows[:, None, c] - pts[None, :, c]) ** 2 for c in range(3))
        d2[torch.arange(rows.shape[0]), torch.arange(i, i + rows.shape[0])] = math.inf
        best = torch.topk(d2, 16, dim=1, largest=False)
        dist, near = best.values.sqrt(), planes[3][best.indices]
        feat[i:i + 2048, 59] = torch.log(dist.mean(1))
        feat[i:i + 2048, 60] = torch.log(dist[:, 15])
        feat[i:i + 2048, 61], feat[i:i + 2048, 62] = near.mean(1), near.amax(1)
        feat[i:i + 2048, 63] = torch.log(near.sum(1) / (4 / 3 * math.pi * dist[:, 15] ** 3))
    return feat


def _layers(params):
    at, out = 0, []
    for rows, cols in ((256, 64), (256, 256), (256, 256), (1, 256)):
        out.append((params[at:at + rows * cols].view(rows, cols), params[at + rows * cols:at + rows * cols + rows]))
        at += rows * cols + rows
    return out


def _network(params, feat, norm):
    h = (feat.double() - norm[0].double()) * norm[1].double()
    layers = _layers(params)
    for W, b in layers[:3]:
        h = torch.nn.functional.silu(h @ W.T + b)
    return h @ layers[3][0][0] + layers[3][1][0]


def exact(case, seed):
    kind = case["kind"]
    if kind in ("plan", "sample"):
        return None
    if kind in ("pass", "objective", "judge"):
        blocks = case["views"] * math.ceil(case["width"] / 64) * math.ceil(case["height"] / 64)
        pairs = case["n"] * case["views"] * 9_000.0 * max(0.5, case["width"] * case["height"] / PIXELS_720P)
        if kind != "judge" and (pairs > 6e10 or blocks > 10_000):
            return None
        fmt = case.get("fmt", "f32")
        stored = _scene_planes(case["n"], case["degree"], seed)
        planes = [p.double() for p in _stored(stored, fmt)]
        views = _views(case["views"], case["width"], case["height"], seed)
        if kind == "pass":
            return _exact_pass(planes, case["degree"], views, case, seed)
        weights = _draw_weights(stored, max(1, int(case["m_frac"] * case["n"])), seed)
        per_ray, per_view = _exact_objective(planes, case["degree"], views, weights, case, seed)
        if kind == "objective":
            return {"per_ray": per_ray, "per_view": per_view}
        error = float(((per_view[:, 1] - per_view[:, 0]).abs() / per_view[:, 0].clamp_min(1e-300)).max())
        return {"per_view": per_view, "error": error}
    if kind == "features":
        if case["n"] > 150_000:
            return None
        planes = [p.double() for p in _stored(_scene_planes(case["n"], case["degree"], seed), case["fmt"])]
        feat = _exact_features(planes, case["degree"])
        std = feat.std(0, unbiased=False)
        flat = std < 1e-10
        return {"features": feat, "stats": torch.stack([feat.mean(0), torch.where(flat, 1.0, 1 / std.clamp_min(1e-300))])}
    feat, norm = _feature_rows(case["n"], seed)
    params = _mlp_params(seed).double().requires_grad_(kind == "train")
    if kind == "predict":
        with torch.no_grad():
            y = torch.cat([_network(params, part, norm) for part in feat.split(65_536)])
        e = torch.exp(y - y.max())
        return {"log_s": y, "scores": 0.9 * e / e.sum() + 0.1 / case["n"]}
    loss = ((_network(params, feat, norm) - _targets(feat, norm, seed).double()) ** 2).mean()
    loss.backward()
    g = params.grad
    m, v = 0.1 * g, 0.001 * g * g
    new = params.detach() - 1e-3 * (m / 0.1) / ((v / 0.001).sqrt() + 1e-8)
    return {"loss": loss.detach().reshape(1), "grad": g, "params": new, "adam": torch.cat([m, v])}
