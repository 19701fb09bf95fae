"""Timed workloads of the rasterizer and of the kernels around it.

Each case is one pass through the package's public entry points, the way a
SLAM program calls them: single keyframes (captured, eager and through
autograd), batches of agents' keyframes, the fused map, novel views, one
refinement step, the image losses, the optimiser update, the merging of a
borrowed submap and the seeding of a new keyframe.  Inputs are drawn on the
GPU from the seed alone, with the distributions of synth/scenes.py: Gaussians
uniform in a 6 x 3 x 4 m room, log-scales N(-3, 0.5), random rotations,
opacity logits N(0, 1), cameras inside the room with a 90 degree horizontal
field of view.

`exact` is the same mathematics in FP64 with plain torch, written from the
definitions (EWA projection, per-tile front-to-back compositing, autograd for
the gradients).
"""
import math

import numpy as np
import torch

ROOM_LO, ROOM_HI = (-3.0, -1.5, -2.0), (3.0, 1.5, 2.0)
Y00 = 0.28209479177387814
ALPHA_MAX = float(np.float32(0.99))
ALPHA_MIN = float(np.float32(1.0) / np.float32(255.0))
T_MIN = float(np.float32(1e-4))
Z_NEAR = 0.2
GRADS = ("d_means", "d_log_scales", "d_quats", "d_opacity_logits", "d_colors", "d_pose")


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest call: a coarse preview of a few Gaussians in front of
        # one camera, where launches and latency are everything
        dict(name="plain-2k-128x96", kind="render", sets="2000", views=1, width=128, height=96,
             sh=0, layout="front", form="eager", novel=0, cols=1, alpha=False, bg=0.0),
        # mapping of one keyframe, the step captured once and replayed
        dict(name="keyframe-300k-1200x680", kind="render", sets="300000", views=1, width=1200,
             height=680, sh=0, layout="centre", form="graph", novel=0, cols=1, alpha=False,
             bg=0.0),
        # tracking: one keyframe with its pose delta through autograd
        dict(name="autograd-1m-1200x680", kind="render", sets="1000000", views=1, width=1200,
             height=680, sh=0, layout="centre", form="autograd", novel=0, cols=1, alpha=False,
             bg=0.0),
        # a novel view of a map with view-dependent colour: forward only
        dict(name="novel-1m-sh3-1200x680", kind="render", sets="1000000", views=1, width=1200,
             height=680, sh=3, layout="free", form="eager", novel=1, cols=1, alpha=False, bg=1.0),
        # a few uneven submaps at an odd image size, every image gradient used
        dict(name="ragged-3x3-517x389-sh1", kind="render", sets="17001,50333,90007", views=3,
             width=517, height=389, sh=1, layout="circle", form="eager", novel=0, cols=1,
             alpha=True, bg=0.5),
        # every agent's submap with its window of keyframes in one batch
        dict(name="multi-agent-6x8-640x480", kind="render",
             sets="50000,120000,200000,300000,400000,600000", views=8, width=640, height=480,
             sh=0, layout="circle", form="eager", novel=0, cols=2, alpha=False, bg=0.0),
        # the fused map: novel views and keyframes of one large SH map
        dict(name="fused-3m-sh3-48x1200x680", kind="render", sets="3000000", views=48, width=1200,
             height=680, sh=3, layout="free", form="eager", novel=16, cols=2, alpha=False, bg=0.0),
        # one step of the joint refinement, up to its gradients
        dict(name="refine-400k-sh3-8x640x480", kind="refine", sets="400000", views=8, width=640,
             height=480, sh=3, layout="free"),
        # the image side of the refinement loss over a batch of keyframes
        dict(name="losses-48x640x480", kind="losses", views=48, width=640, height=480),
        # the Gaussian side of a mapping step: isotropy term, then Adam
        dict(name="update-1670k", kind="update", n=1670000, views=48),
        # a submap borrowed from another agent, moved, deduplicated, pruned
        dict(name="merge-350k-400k-8x640x480", kind="merge", n_target=350000, n_source=400000,
             views=8, width=640, height=480),
        # Gaussians seeded from a new keyframe
        dict(name="seed-1200x680", kind="seed", width=1200, height=680, stride=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["render"] * 6 + ["refine", "losses", "update", "merge", "seed"])
    w = _log(rng, 64, 1200)
    h = max(48, int(w * rng.uniform(0.5, 0.8)))
    sh = rng.choice([0, 0, 1, 2, 3])
    if kind == "render":
        form = rng.choice(["eager", "eager", "autograd", "graph"])
        if rng.random() < 0.6:  # one view
            novel = 1 if form == "eager" and rng.random() < 0.4 else 0
            return dict(kind=kind, sets=str(_log(rng, 1000, 1500000)), views=1, width=w, height=h,
                        sh=sh, layout=rng.choice(["free", "centre"]), form=form, novel=novel,
                        cols=1, alpha=rng.random() < 0.3, bg=rng.choice([0.0, 0.0, 1.0]))
        sets = [_log(rng, 5000, 400000) for _ in range(rng.randint(1, 6))]
        w, h = min(w, 900), min(h, 640)
        return dict(kind=kind, sets=",".join(map(str, sets)), views=rng.randint(2, 8), width=w,
                    height=h, sh=sh, layout="circle", form="eager", novel=rng.randint(0, 1),
                    cols=rng.choice([1, 2]), alpha=rng.random() < 0.3, bg=0.0)
    if kind == "refine":
        return dict(kind=kind, sets=str(_log(rng, 20000, 800000)), views=rng.randint(1, 16),
                    width=w, height=h, sh=sh, layout="free")
    if kind == "losses":
        return dict(kind=kind, views=_log(rng, 1, 48), width=w, height=h)
    if kind == "update":
        return dict(kind=kind, n=_log(rng, 2000, 3000000), views=rng.randint(1, 48))
    if kind == "merge":  # VGA-sized keyframes, as the submaps are mapped from
        return dict(kind=kind, n_target=_log(rng, 10000, 500000),
                    n_source=_log(rng, 10000, 500000), views=rng.randint(1, 8),
                    width=rng.randint(600, 640), height=rng.randint(440, 480))
    return dict(kind=kind, width=w, height=h, stride=rng.choice([1, 1, 2, 3]))


# --------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device="cuda")


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda")


def _gaussians(g, n, sh, layout="room"):
    lo, hi = ((-1.0, -1.0, 2.0), (1.0, 1.0, 4.0)) if layout == "front" else (ROOM_LO, ROOM_HI)
    lo, hi = (torch.tensor(x, device="cuda") for x in (lo, hi))
    means = lo + (hi - lo) * _rand(g, n, 3)
    log_scales = _randn(g, n, 3) * 0.5 - 3.0
    quats = torch.nn.functional.normalize(_randn(g, n, 4), dim=1)
    opac = _randn(g, n)
    rgb = _rand(g, n, 3)
    if sh:
        k = (sh + 1) ** 2
        col = _randn(g, n, k, 3) * 0.1
        col[:, 0] = (rgb - 0.5) / Y00
        rgb = col
    return [x.contiguous() for x in (means, log_scales, quats, opac, rgb)]


def _look(center, yaw, pitch):
    fwd = np.array([math.sin(yaw) * math.cos(pitch), -math.sin(pitch),
                    math.cos(yaw) * math.cos(pitch)])
    right = np.cross([0.0, 1.0, 0.0], fwd)
    right /= np.linalg.norm(right)
    R = np.stack([right, np.cross(fwd, right), fwd])
    return np.concatenate([R, (-R @ np.asarray(center))[:, None]], axis=1)


def _cameras(case, seed):
    """(viewmats [V,3,4], intrinsics [V,4], view_set [V]) of a case."""
    rng = np.random.default_rng(int(seed) + 77)
    W, H = case["width"], case["height"]
    n_sets = len(str(case["sets"]).split(","))
    vm, vs = [], []
    for s in range(n_sets):
        for _ in range(case["views"]):
            th = rng.uniform(0, 2 * math.pi)
            if case["layout"] == "circle":  # on a circle, looking inward
                c = np.array([1.5 * math.cos(th), 0.0, 1.5 * math.sin(th)])
                vm.append(_look(c, math.atan2(-c[0], -c[2]) + math.radians(rng.uniform(-15, 15)),
                                0.0))
            elif case["layout"] == "free":  # anywhere in the room
                c = np.array([rng.uniform(-2, 2), rng.uniform(-0.5, 0.5), rng.uniform(-1.5, 1.5)])
                vm.append(_look(c, th, math.radians(rng.uniform(-15, 15))))
            elif case["layout"] == "front":
                vm.append(_look(np.zeros(3), 0.0, 0.0))
            else:
                vm.append(_look(rng.normal(0, 0.1, 3), th, 0.0))
            vs.append(s)
    f = 100.0 * W / 128.0 if case["layout"] == "front" else W / 2.0
    intr = np.tile(np.array([f, f, W / 2.0, H / 2.0]), (len(vm), 1))
    return (np.asarray(vm, np.float32), intr.astype(np.float32), np.asarray(vs, np.int32))


def _upstream(g, case, V):
    """Image gradients as the L1 terms hand them to the backward."""
    W, H = case["width"], case["height"]
    sign = lambda *s: torch.where(_rand(g, *s) < 0.5, -1.0, 1.0)
    gc = sign(V, 3, H, W) * (0.95 / (3 * V * H * W))
    gd = sign(V, H, W) * (0.25 / (V * H * W))
    ga = _randn(g, V, H, W) * (0.1 / (V * H * W)) if case.get("alpha") else None
    return gc, gd, ga


def _scene_inputs(case, seed):
    sizes = [int(x) for x in str(case["sets"]).split(",")]
    g = _gen(seed)
    arrays = _gaussians(g, sum(sizes), case["sh"],
                        "front" if case["layout"] == "front" else "room")
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    vm, intr, vs = _cameras(case, seed)
    return g, arrays, offs, vm, intr, vs


def _needs_grad(case, V):
    if not case.get("novel"):
        return None
    ng = np.ones(V, np.uint8)
    per = case["views"]  # the first `novel` views of every set are forward-only
    for s in range(V // per):
        ng[s * per:s * per + case["novel"]] = 0
    return ng


def _slanted(g, V, H, W, f):
    """Piecewise-planar depth with jitter and holes, and normal priors."""
    x = (torch.arange(W, device="cuda") + 0.5 - W / 2) / f
    y = (torch.arange(H, device="cuda") + 0.5 - H / 2) / f
    best = torch.full((V, H, W), 5.0, device="cuda")
    for _ in range(3):
        z0 = 1.5 + 2.5 * _rand(g, V, 1, 1)
        den = 1 - 0.3 * _randn(g, V, 1, 1) * x[None, None] - 0.3 * _randn(g, V, 1, 1) * y[None, :, None]
        best = torch.minimum(best, torch.where(den > 0.2, z0 / den.clamp(min=0.2), 5.0))
    d = best + 2e-3 * _randn(g, V, H, W)
    d = torch.where(_rand(g, V, H, W) < 0.02, 0.0, d).contiguous()
    p = torch.cat([0.3 * _randn(g, V, 2, H, W), -torch.ones((V, 1, H, W), device="cuda")], 1)
    return d, torch.nn.functional.normalize(p, dim=1).contiguous()


def _loss_inputs(case, seed):
    V, W, H = case["views"], case["width"], case["height"]
    g = _gen(seed)
    target = _rand(g, V, 3, H, W)
    color = (target + 0.2 * _randn(g, V, 3, H, W)).clamp(0, 1)
    depth, prior = _slanted(g, V, H, W, W / 2.0)
    tdepth = depth + 0.05 * _randn(g, V, H, W)
    expo = 0.05 * _randn(g, V, 2)
    intr = torch.tensor([[W / 2.0, W / 2.0, W / 2.0, H / 2.0]] * V, device="cuda")
    return color, target, depth, tdepth, prior, expo, intr


def _update_inputs(case, seed):
    g = _gen(seed)
    n, V = case["n"], case["views"]
    par = _gaussians(g, n, 0) + [torch.zeros((V, 6), device="cuda"),
                                 torch.zeros((V, 2), device="cuda")]
    grads = [1e-4 * torch.randn(p.shape, generator=g, device="cuda") for p in par]
    return par, grads


UPDATE_LR = (1.6e-4, 5e-3, 1e-3, 5e-2, 2.5e-3, 1e-3, 1e-3)


def _merge_inputs(case, seed):
    g = _gen(seed)
    tgt = _gaussians(g, case["n_target"], 0)
    tgt[0][:, 0] = -3.0 + 3.5 * _rand(g, case["n_target"])  # the target covers part of the room
    low = torch.randperm(case["n_target"], generator=g, device="cuda")[:case["n_target"] // 8]
    tgt[3].clamp_(-5.0, 5.0)[low] -= 12.0  # the rest of the target has faded away
    src = _gaussians(g, case["n_source"], 0)
    W, H, V = case["width"], case["height"], case["views"]
    cam = dict(case, sets="1", layout="circle")
    vm, intr, _ = _cameras(cam, seed)
    depth = (0.5 + 1.5 * _rand(g, V, H // 32 + 1, W // 32 + 1))
    depth = torch.nn.functional.interpolate(depth[:, None], size=(H, W), mode="bilinear")[:, 0]
    sims = np.array([[1.02, 0.9998, 0.01, -0.012, 0.008, 0.03, -0.02, 0.05]], np.float32)
    cu = lambda a: torch.from_numpy(a).cuda()
    return tgt, src, cu(vm), cu(intr), depth.contiguous(), cu(sims)


def _seed_inputs(case, seed):
    g = _gen(seed)
    W, H = case["width"], case["height"]
    depth, _ = _slanted(g, 1, H, W, W / 2.0)
    depth = torch.where(depth > 0, depth, 2.0)
    st = case["stride"]
    gw, m = -(-W // st), -(-W // st) * -(-H // st)
    hole = torch.randperm(m, generator=g, device="cuda")[:m // 50]  # no depth there
    depth[0, hole // gw * st, hole % gw * st] = 0.0
    vm = torch.from_numpy(_look((0.4, -0.1, -1.5), 0.1, 0.0).astype(np.float32)).cuda()
    intr = torch.tensor([W / 2.0, W / 2.0, W / 2.0, H / 2.0], device="cuda")
    return depth[0].contiguous(), _rand(g, 3, H, W), vm, intr


def prepare(case, seed):
    import paper_2605_10760_amd as gs
    kind = case["kind"]
    s = dict(case=case)
    if kind in ("render", "refine"):
        g, arrays, offs, vm, intr, vs = _scene_inputs(case, seed)
        V, W, H = len(vs), case["width"], case["height"]
        scene = gs.SceneTensors(*arrays, offs, case["sh"])
        views = gs.ViewTensors(torch.from_numpy(vm).cuda(), torch.from_numpy(intr).cuda(), vs, W,
                               H, _needs_grad(case, V))
        s.update(scene=scene, views=views)
        rast = gs.Rasterizer(W, H, max(1, gs.pairs_of(scene, views)), V,
                             bwd_cols=case.get("cols", 2))
        if V > 1:
            rast.fit_capacity(scene, views)
        s["rast"] = rast
        if kind == "refine":
            tc = _rand(g, V, 3, H, W)
            td = 0.2 + 3.8 * _rand(g, V, H, W)
            _, prior = _slanted(g, V, H, W, W / 2.0)
            s["opt"] = gs.Optimizer(rast, scene, views, tc, td, prior, gs.REFINE_WEIGHTS,
                                    gs.Rates().scaled(0.5), pose=True, exposure=True)
            s["opt"].exposure.copy_(0.05 * _randn(g, V, 2))
            return s
        gc, gd, ga = _upstream(g, case, V)
        bg = (case["bg"],) * 3
        s.update(gc=gc, gd=gd, ga=ga, bg=bg)
        if case["form"] == "autograd":
            s["leaves"] = [x.requires_grad_() for x in arrays]
            s["pose"] = torch.zeros((V, 6), device="cuda", requires_grad=True)
        else:
            s["buf"] = rast.new_state()
        if case["form"] == "graph":
            s["img"] = (torch.empty((V, 3, H, W), device="cuda"),
                        torch.empty((V, H, W), device="cuda"),
                        torch.empty((V, H, W), device="cuda"))
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                rast.forward(scene, views, bg=bg, state=s["buf"], out=s["img"])
                s["grads"] = rast.backward(scene, views, s["buf"], gc, gd, ga, bg=bg)
            torch.cuda.current_stream().wait_stream(side)
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"]):
                rast.forward(scene, views, bg=bg, state=s["buf"], out=s["img"])
                rast.backward(scene, views, s["buf"], gc, gd, ga, bg=bg, out=s["grads"])
        return s
    if kind == "losses":
        names = ("color", "target", "depth", "tdepth", "prior", "expo", "intr")
        s.update(zip(names, _loss_inputs(case, seed)))
        s["out"] = dict(d_color=torch.empty_like(s["color"]), d_depth=torch.empty_like(s["depth"]),
                        d_exposure=torch.empty_like(s["expo"]))
        s["ssim"] = torch.empty(1, device="cuda")
        s["ws"] = None
        return s
    if kind == "update":
        par, grads = _update_inputs(case, seed)
        s["adam"] = gs.Adam(list(zip(par, UPDATE_LR)), eps=1e-15)
        for p, q in zip(par, grads):
            p.grad = q
        s.update(par=par, grads=grads)
        return s
    if kind == "merge":
        tgt, src, vm, intr, depth, sims = _merge_inputs(case, seed)
        s.update(target=gs.SceneTensors(*tgt, np.array([0, case["n_target"]], np.int64), 0),
                 src=src, vm=vm, intr=intr, depth=depth, sims=sims,
                 offs=np.array([0, case["n_source"]], np.int64))
        return s
    s.update(zip(("depth", "color", "vm", "intr"), _seed_inputs(case, seed)))
    return s


# ----------------------------------------------------------------- one pass
def run(s):
    import paper_2605_10760_amd as gs
    case = s["case"]
    kind = case["kind"]
    if kind == "render":
        rast, scene, views, bg = s["rast"], s["scene"], s["views"], s["bg"]
        if case["form"] == "graph":
            s["graph"].replay()
            return dict(images=list(s["img"]), **s["grads"])
        if case["form"] == "autograd":
            for x in s["leaves"] + [s["pose"]]:
                x.grad = None
            c, d, a = gs.rasterize(rast, *s["leaves"], views.viewmats, views.intrinsics,
                                   scene.set_offsets, views.view_set, views.width, views.height,
                                   pose_delta=s["pose"], sh_degree=scene.sh_degree,
                                   needs_grad=views.needs_grad, bg=bg)
            outs, ups = ([c, d], [s["gc"], s["gd"]]) if s["ga"] is None else \
                ([c, d, a], [s["gc"], s["gd"], s["ga"]])
            torch.autograd.backward(outs, ups)
            g = {k: x.grad for k, x in zip(GRADS, s["leaves"] + [s["pose"]])}
            return dict(images=[c.detach(), d.detach(), a.detach()], **g)
        c, d, a, st = rast.forward(scene, views, bg=bg, state=s["buf"])
        if case["novel"] >= case["views"]:
            return dict(images=[c, d, a])
        g = rast.backward(scene, views, st, s["gc"], s["gd"], s["ga"], bg=bg)
        return dict(images=[c, d, a], **g)
    if kind == "refine":
        return s["opt"].gradients()
    if kind == "losses":
        o = gs.l1_loss_grad(s["color"], s["target"], s["depth"], s["tdepth"], s["expo"], 1.75,
                            0.25, out=s["out"])
        s["ws"] = gs.ssim_grad(s["color"], s["target"], o["d_color"], s["expo"], o["d_exposure"],
                               0.2, workspace=s["ws"], ssim_out=s["ssim"])
        gs.normal_loss_grad(s["depth"], s["prior"], s["intr"], o["d_depth"], 10.0)
        return dict(o, ssim=s["ssim"])
    if kind == "update":
        gs.iso_grad(s["par"][1], s["grads"][1], 1e-4)
        s["adam"].step()
        return dict(params=s["par"], m=s["adam"].m, v=s["adam"].v)
    if kind == "merge":
        src = s["src"]
        moved = gs.sim3_gaussians(src[0], src[1], src[2], s["offs"], s["sims"])
        t = s["target"]
        keep, voxels = gs.dedup(moved[0], t.means, t.log_scales, s["depth"], s["vm"], s["intr"])
        p = gs.prune(t)
        return dict(moved=list(moved), keep=keep, voxels=voxels, offs=p.set_offsets,
                    pruned=[p.means, p.log_scales, p.quats, p.opacity_logits, p.colors])
    return gs.seed(s["depth"], s["color"], s["vm"], s["intr"], stride=case["stride"],
                   opacity_logit=-0.7)


# ------------------------------------------------------------------- the work
def work(case):
    """Bytes: each input read once, each output written once.  Operations of
    the compositing: about 110 list entries per pixel of these scenes, 28
    operations each forward and 61 backward."""
    kind = case["kind"]
    if kind in ("render", "refine"):
        n = sum(int(x) for x in str(case["sets"]).split(","))
        V = case["views"] * len(str(case["sets"]).split(","))
        px = V * case["width"] * case["height"]
        par = 4.0 * n * (11 + 3 * (case["sh"] + 1) ** 2)
        if kind == "refine":
            return dict(bytes=2 * par + 8.0 * 7 * px / 2, flops=px * (110.0 * 89 + 900))
        back = V * (1 - case["novel"] / case["views"])
        gpx = px * back / V
        return dict(bytes=par + 20.0 * px + (par + 16.0 * gpx if back else 0.0),
                    flops=110.0 * (28 * px + 61 * gpx))
    if kind == "losses":
        px = float(case["views"] * case["width"] * case["height"])
        return dict(bytes=4.0 * (3 + 3 + 1 + 1 + 3 + 3 + 1) * px, flops=900.0 * px)
    if kind == "update":
        n = 14.0 * case["n"] + 8 * case["views"]
        return dict(bytes=28.0 * n + 12.0 * case["n"], flops=14.0 * n)
    if kind == "merge":
        return dict(bytes=4.0 * (24 * case["n_target"] + 20 * case["n_source"]) + case["n_source"]
                    + 4.0 * case["views"] * case["width"] * case["height"], flops=0.0)
    m = float(-(-case["width"] // case["stride"]) * -(-case["height"] // case["stride"]))
    return dict(bytes=72.0 * m, flops=60.0 * m)


# ------------------------------------------------------- the same in 64 bits
def _sh_basis(d, deg):
    x, y, z = d.unbind(-1)
    o = torch.ones_like(x)
    Y = [Y00 * o]
    if deg >= 1:
        k = math.sqrt(3 / (4 * math.pi))
        Y += [-k * y, k * z, -k * x]
    if deg >= 2:
        a, b = math.sqrt(15 / math.pi) / 2, math.sqrt(5 / math.pi) / 4
        Y += [a * x * y, -a * y * z, b * (2 * z * z - x * x - y * y), -a * x * z,
              a / 2 * (x * x - y * y)]
    if deg >= 3:
        a, b = math.sqrt(35 / (2 * math.pi)) / 4, math.sqrt(105 / math.pi) / 2
        c, e = math.sqrt(21 / (2 * math.pi)) / 4, math.sqrt(7 / math.pi) / 4
        Y += [-a * y * (3 * x * x - y * y), b * x * y * z, -c * y * (4 * z * z - x * x - y * y),
              e * z * (2 * z * z - 3 * x * x - 3 * y * y), -c * x * (4 * z * z - x * x - y * y),
              b / 2 * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)]
    return torch.stack(Y, -1)


def _project64(m, ls, q, o, col, sh, R, t, intr, W, H):
    """Screen-space record [n, 10] (u, v, A, B, C, sigma, r, g, b, z) and the
    half-extents [n, 2] of the alpha >= 1/255 ellipse."""
    fx, fy, cx, cy = (float(x) for x in intr)
    p = m @ R.T + t
    q = q / q.norm(dim=1, keepdim=True)
    w, x, y, z = q.unbind(1)
    Rq = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                      2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                      2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)],
                     1).view(-1, 3, 3)
    M = R @ (Rq * ls.exp()[:, None, :])  # n x 3 x 3: columns are the scaled axes
    rx, ry = p[:, 0] / p[:, 2], p[:, 1] / p[:, 2]
    lx, ly = 1.3 * (0.5 * W) / fx, 1.3 * (0.5 * H) / fy
    iz = 1 / p[:, 2]
    j0 = (fx * iz)[:, None] * M[:, 0] - (fx * rx.clamp(-lx, lx) * iz)[:, None] * M[:, 2]
    j1 = (fy * iz)[:, None] * M[:, 1] - (fy * ry.clamp(-ly, ly) * iz)[:, None] * M[:, 2]
    a, b, c = (j0 * j0).sum(1) + 0.3, (j0 * j1).sum(1), (j1 * j1).sum(1) + 0.3
    det = a * c - b * b
    sig = torch.sigmoid(o)
    if sh:
        d = m + R.T @ t  # camera centre: -R^T t
        d = d / d.norm(dim=1, keepdim=True)
        col = (0.5 + (_sh_basis(d, sh)[:, :, None] * col[:, :(sh + 1) ** 2]).sum(1)).clamp(min=0)
    rec = torch.cat([torch.stack([fx * rx + cx, fy * ry + cy, c / det, -b / det, a / det, sig], 1),
                     col, p[:, 2:3]], 1)
    with torch.no_grad():
        k2 = 2 * torch.log((255 * sig).clamp(min=1.0))
        ext = torch.stack([(k2 * a).sqrt(), (k2 * c).sqrt()], 1)
    return rec, ext


def _composite64(r, px, py):
    """Images [nt, 256, 5] (r, g, b, depth, alpha) of tiles' padded records
    r [nt, L, 10] (sigma 0 for padding) at pixel centres [nt, 256], and the
    smallest transmittance after the last entry before any stop."""
    dx, dy = r[:, None, :, 0] - px[..., None], r[:, None, :, 1] - py[..., None]
    pw = -0.5 * (r[:, None, :, 2] * dx * dx + r[:, None, :, 4] * dy * dy) - r[:, None, :, 3] * dx * dy
    al = (r[:, None, :, 5] * pw.exp()).clamp(max=ALPHA_MAX)
    al = torch.where((al >= ALPHA_MIN) & (pw <= 0), al, 0.0)
    lt = torch.log1p(-al).cumsum(2)
    Tn = lt.exp()
    T = torch.cat([torch.ones_like(Tn[..., :1]), Tn[..., :-1]], 2)
    w = torch.where(Tn >= T_MIN, al * T, 0.0)
    img = torch.matmul(w, r[:, :, 6:10])
    return torch.cat([img, w.sum(2, keepdim=True)], 2), Tn[..., -1]


class _View64(torch.autograd.Function):
    """Images [5, H, W] of one view from its records in depth order, tile by
    tile; the backward recomputes each group of tiles with autograd."""

    @staticmethod
    def forward(ctx, rec, lists, W, H):
        out = torch.zeros((5, H + 16, W + 16), dtype=rec.dtype, device=rec.device)
        groups = []
        pad = torch.cat([rec, torch.zeros_like(rec[:1])])  # last row: sigma 0
        for tx, ty, idx in lists(rec.shape[0]):
            px, py, lin = _tile_pixels(tx, ty, W + 16)
            L = min(256, idx.shape[1])
            while True:
                img, Tn = _composite64(pad[idx[:, :L]], px, py)
                if L == idx.shape[1] or bool((Tn < T_MIN).all()):
                    break
                L = min(2 * L, idx.shape[1])
            out.view(5, -1)[:, lin.reshape(-1)] = img.reshape(-1, 5).T
            groups.append((px, py, lin, idx[:, :L].clone()))
        ctx.save_for_backward(rec)
        ctx.groups, ctx.size = groups, (W, H)
        return out[:, :H, :W].contiguous()

    @staticmethod
    def backward(ctx, g):
        (rec,) = ctx.saved_tensors
        W, H = ctx.size
        gp = torch.zeros((5, H + 16, W + 16), dtype=g.dtype, device=g.device)
        gp[:, :H, :W] = g
        gp = gp.view(5, -1)
        pad = torch.cat([rec, torch.zeros_like(rec[:1])])
        total = torch.zeros_like(pad)
        for px, py, lin, idx in ctx.groups:
            r = pad[idx].requires_grad_()
            with torch.enable_grad():
                img, _ = _composite64(r, px, py)
            up = gp[:, lin.reshape(-1)].T.reshape(img.shape)
            (gr,) = torch.autograd.grad(img, r, up)
            total.index_add_(0, idx.reshape(-1), gr.reshape(-1, gr.shape[-1]))
        return total[:-1], None, None, None


def _tile_pixels(tx, ty, pitch):
    k = torch.arange(256, device=tx.device)
    x, y = tx[:, None] * 16 + k % 16, ty[:, None] * 16 + k // 16
    return x.double() + 0.5, y.double() + 0.5, y * pitch + x


def _tile_lists(u, v, ext, W, H, budget=12_000_000):
    """Generator over groups of tiles of similar list length: tile columns,
    rows, and the positions [nt, L] of their records (padded past the end)."""
    TX, TY = -(-W // 16), -(-H // 16)
    x0 = ((u - ext[:, 0] - 1) / 16).floor().clamp(0, TX).long()
    x1 = (((u + ext[:, 0] + 1) / 16).floor() + 1).clamp(0, TX).long()
    y0 = ((v - ext[:, 1] - 1) / 16).floor().clamp(0, TY).long()
    y1 = (((v + ext[:, 1] + 1) / 16).floor() + 1).clamp(0, TY).long()
    nx, ny = (x1 - x0).clamp(min=0), (y1 - y0).clamp(min=0)
    cnt = nx * ny

    def groups(n):
        pos = torch.repeat_interleave(torch.arange(n, device=u.device), cnt)
        k = torch.arange(pos.shape[0], device=u.device) - (cnt.cumsum(0) - cnt)[pos]
        tile = (y0[pos] + k // nx[pos]) * TX + x0[pos] + k % nx[pos]
        tile, order = tile.sort(stable=True)
        pos = pos[order]
        num = torch.bincount(tile, minlength=TX * TY)
        start = num.cumsum(0) - num
        by = num.argsort()
        by = by[num[by] > 0]
        lens = num[by].tolist()
        i = 0
        while i < len(lens):
            j = i + 1
            while j < len(lens) and (j + 1 - i) * 256 * min(lens[j], 512) <= budget:
                j += 1
            t, L = by[i:j], lens[j - 1]
            s = torch.arange(L, device=u.device)[None]
            ok = s < num[t][:, None]
            idx = torch.where(ok, pos[(start[t][:, None] + s).clamp(max=pos.shape[0] - 1)], n)
            yield t % TX, t // TX, idx
            i = j

    return groups


def _render64(arrays, offs, sh, vm, intr, vs, W, H, bg, images_grad):
    """Images of every view and, where images_grad(v, images) gives upstream
    gradients [5, H, W], the gradients of the parameters and poses."""
    par = [a.detach().double() for a in arrays]
    grads = [torch.zeros_like(a) for a in par]
    V = len(vs)
    pose = torch.zeros((V, 6), dtype=torch.float64, device="cuda")
    images = []
    for v in range(V):
        lo, hi = int(offs[vs[v]]), int(offs[vs[v] + 1])
        R32, t32 = torch.from_numpy(vm[v][:, :3]).cuda(), torch.from_numpy(vm[v][:, 3]).cuda()
        m32 = arrays[0][lo:hi].detach()
        # the depth key is FP32 by definition: ((r0 x + r1 y) + r2 z) + t
        z32 = ((R32[2, 0] * m32[:, 0] + R32[2, 1] * m32[:, 1]) + R32[2, 2] * m32[:, 2]) + t32[2]
        R, t = R32.double(), t32.double()
        near = (z32 > np.float32(Z_NEAR)).nonzero()[:, 0]
        rec, ext = _project64(*[p[lo:hi][near] for p in par], sh, R, t, intr[v], W, H)
        on = ((rec[:, 0] + ext[:, 0] > -2) & (rec[:, 0] - ext[:, 0] < W + 2)
              & (rec[:, 1] + ext[:, 1] > -2) & (rec[:, 1] - ext[:, 1] < H + 2)
              & (255 * rec[:, 5] > 1))
        sel = near[on]
        sel = sel[z32[sel].sort(stable=True)[1]]
        leaves = [p[lo:hi][sel].requires_grad_() for p in par]
        xi = torch.zeros(6, dtype=torch.float64, device="cuda", requires_grad=True)
        zero = xi[0] * 0
        K = torch.stack([zero, -xi[5], xi[4], xi[5], zero, -xi[3], -xi[4], xi[3], zero]).view(3, 3)
        rec, ext = _project64(*leaves, sh, R + K @ R, t + K @ t + xi[:3], intr[v], W, H)
        lists = _tile_lists(rec[:, 0].detach(), rec[:, 1].detach(), ext, W, H)
        img = _View64.apply(rec, lists, W, H)
        out = torch.cat([img[:3] + (1 - img[4:5]) * bg, img[3:]])
        images.append(out.detach())
        up = images_grad(v, out.detach()) if images_grad else None
        if up is not None:
            gs_ = torch.autograd.grad(out, leaves + [xi], up, allow_unused=True)
            for tot, gr in zip(grads, gs_):
                if gr is not None:
                    tot[lo:hi].index_add_(0, sel, gr)
            pose[v] = gs_[5]
    return torch.stack(images), dict(zip(GRADS, grads + [pose]))


def _blur64(x):
    w = np.exp(-np.arange(-5, 6) ** 2 / (2 * 1.5 ** 2))
    w = w / w.sum()
    H, W = x.shape[-2:]
    p = torch.nn.functional.pad(x, (5, 5, 0, 0))
    x = sum(float(w[k]) * p[..., k:k + W] for k in range(11))
    p = torch.nn.functional.pad(x, (0, 0, 5, 5))
    return sum(float(w[k]) * p[..., k:k + H, :] for k in range(11))


def _ssim64(x, y):
    """Sum of the SSIM map of images [3, H, W] (11 x 11 Gaussian window)."""
    mx, my = _blur64(x), _blur64(y)
    sxx, syy = _blur64(x * x) - mx * mx, _blur64(y * y) - my * my
    sxy = _blur64(x * y) - mx * my
    c1, c2 = 1e-4, 9e-4
    return ((2 * mx * my + c1) * (2 * sxy + c2)
            / ((mx * mx + my * my + c1) * (sxx + syy + c2))).sum()


def _normal64(d, prior, intr):
    """Sum over the interior pixels of 1 - N . prior for depth [H, W]."""
    fx, fy, cx, cy = (float(x) for x in intr)
    H, W = d.shape
    x = (torch.arange(W, device=d.device) + 0.5 - cx) / fx
    y = (torch.arange(H, device=d.device) + 0.5 - cy) / fy
    P = torch.stack([d * x[None], d * y[:, None], d])
    a, b = P[:, 2:, 1:-1] - P[:, :-2, 1:-1], P[:, 1:-1, 2:] - P[:, 1:-1, :-2]
    c = torch.linalg.cross(a, b, dim=0)
    ok = ((d[2:, 1:-1] > 0) & (d[:-2, 1:-1] > 0) & (d[1:-1, 2:] > 0) & (d[1:-1, :-2] > 0)
          & ((c * c).sum(0) > 0))
    c = torch.where(ok[None], c, torch.ones_like(c))
    n = c / (c * c).sum(0).sqrt()
    return torch.where(ok, 1 - (n * prior[:, 1:-1, 1:-1]).sum(0), 0.0).sum()


def _losses64(color, target, depth, tdepth, prior, intr, expo, weights, V):
    """Gradients of one view's refinement loss (batch of V views): d_color,
    d_depth, d_exposure, and the sum of its SSIM map."""
    w_col, w_dep, w_ssim, w_nrm = weights
    _, H, W = color.shape
    c, d, e = (x.detach().double().requires_grad_() for x in (color, depth, expo))
    y, td, pr = target.double(), tdepth.double(), prior.double()
    x = e[0].exp() * c + e[1]
    n = 3.0 * V * H * W
    ss = _ssim64(x, y)
    loss = w_col / n * (x - y).abs().sum() + w_dep * 3 / n * (d - td).abs().sum() - w_ssim / n * ss
    if H > 2 and W > 2:
        loss = loss + w_nrm / (V * (H - 2.0) * (W - 2.0)) * _normal64(d, pr, intr)
    return torch.autograd.grad(loss, [c, d, e]) + (ss.detach(),)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("render", "refine"):
        g, arrays, offs, vm, intr, vs = _scene_inputs(case, seed)
        V, W, H = len(vs), case["width"], case["height"]
        if kind == "refine":
            tc = _rand(g, V, 3, H, W)
            td = 0.2 + 3.8 * _rand(g, V, H, W)
            _, prior = _slanted(g, V, H, W, W / 2.0)
            expo = 0.05 * _randn(g, V, 2)
            d_expo = torch.zeros((V, 2), dtype=torch.float64, device="cuda")

            def loss_up(v, img):
                dc, dd, de, _ = _losses64(img[:3], tc[v], img[3], td[v], prior[v], intr[v],
                                          expo[v], (1.75, 0.25, 0.2, 10.0), V)
                d_expo[v] = de
                return torch.cat([dc, dd[None], torch.zeros_like(dd)[None]])

            _, grads = _render64(arrays, offs, case["sh"], vm, intr, vs, W, H, 0.0, loss_up)
            return dict(grads, d_exposure=d_expo)
        gc, gd, ga = _upstream(g, case, V)
        ng = _needs_grad(case, V)

        def given(v, img):
            if ng is not None and not ng[v]:
                return None
            a = torch.zeros_like(gd[v]) if ga is None else ga[v]
            return torch.cat([gc[v], gd[v][None], a[None]]).double()

        img, grads = _render64(arrays, offs, case["sh"], vm, intr, vs, W, H, case["bg"], given)
        images = [img[:, :3].contiguous(), img[:, 3].contiguous(), img[:, 4].contiguous()]
        if case["novel"] >= case["views"]:
            return dict(images=images)
        return dict(images=images, **grads)
    if kind == "losses":
        color, target, depth, tdepth, prior, expo, intr = _loss_inputs(case, seed)
        V = case["views"]
        per = [_losses64(color[v], target[v], depth[v], tdepth[v], prior[v], intr[v].tolist(),
                         expo[v], (1.75, 0.25, 0.2, 10.0), V) for v in range(V)]
        dc, dd, de, ss = (torch.stack(x) for x in zip(*per))
        return dict(d_color=dc, d_depth=dd, d_exposure=de,
                    ssim=(ss.sum() / color.numel()).view(1))
    if kind == "update":
        par, grads = _update_inputs(case, seed)
        par, grads = [p.double() for p in par], [q.double() for q in grads]
        s = par[1].exp()
        q = torch.sign(s - s.mean(1, keepdim=True))
        grads[1] = grads[1] + 1e-4 * s * (q - q.mean(1, keepdim=True))
        m = [0.1 * q for q in grads]
        v = [0.001 * q * q for q in grads]
        new = [p - lr * (a / 0.1) / ((b / 0.001).sqrt() + 1e-15)
               for p, lr, a, b in zip(par, UPDATE_LR, m, v)]
        return dict(params=new, m=m, v=v)
    if kind == "merge":
        tgt, src, _, _, _, sims = _merge_inputs(case, seed)
        sims = sims.double()[0]
        q = sims[1:5] / sims[1:5].norm()
        w, x, y, z = q.tolist()
        R = torch.tensor([[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
                          [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
                          [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]],
                         dtype=torch.float64, device="cuda")
        qm = torch.tensor([[w, -x, -y, -z], [x, w, -z, y], [y, z, w, -x], [z, -y, x, w]],
                          dtype=torch.float64, device="cuda")
        moved = [sims[0] * (src[0].double() @ R.T) + sims[5:8], src[1].double() + sims[0].log(),
                 src[2].double() @ qm.T]
        ok = tgt[3].double() >= math.log(0.005 / 0.995)
        n = int(ok.sum())
        return dict(moved=moved, keep=None, voxels=None, offs=np.array([0, n], np.int64),
                    pruned=[a[ok].double() for a in tgt])
    depth, color, vm, intr = (a.double() for a in _seed_inputs(case, seed))
    st, (H, W) = case["stride"], depth.shape
    fx, fy, cx, cy = intr.tolist()
    jj, ii = torch.meshgrid(torch.arange(0, H, st, device="cuda"),
                            torch.arange(0, W, st, device="cuda"), indexing="ij")
    z = depth[jj, ii]
    P = torch.stack([z * (ii + 0.5 - cx) / fx, z * (jj + 0.5 - cy) / fy, z], -1)
    tot, cnt = torch.zeros_like(z), torch.zeros_like(z)
    for dim, back in ((0, 1), (0, -1), (1, 1), (1, -1)):
        Q, zn = P.roll(back, dim), z.roll(back, dim).clone()
        edge = 0 if back == 1 else -1
        zn.select(dim, edge).zero_()
        near = zn > 0
        tot += torch.where(near, (Q - P).norm(dim=-1), 0.0)
        cnt += near
    sc = torch.where(cnt > 0, tot / cnt.clamp(min=1), z * st / fx)
    ok = z > 0
    pts = (P[ok] - vm[:, 3]) @ vm[:, :3]
    n = pts.shape[0]
    one = torch.zeros((n, 4), dtype=torch.float64, device="cuda")
    one[:, 0] = 1
    return dict(means=pts, log_scales=sc[ok].log()[:, None].expand(-1, 3).contiguous(), quats=one,
                opacity_logits=torch.full((n,), float(np.float32(-0.7)), dtype=torch.float64,
                                          device="cuda"),
                colors=color[:, jj[ok], ii[ok]].T.contiguous())
