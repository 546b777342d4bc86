"""Performance cases: the work a program gives this framework, with sizes,
seeded inputs, one pass through the public entry points, the bytes and
operations a pass cannot do without, and its outputs in 64 bits.

A case is one of four kinds:
  render    one view or several, forward or forward + backward, through the
            autograd function, the Rasterizer's own calls or a captured graph
  train     an optimisation step: render, photometric loss, backward, Adam
  loss      the L1 + SSIM gradient alone
  mcmc, densify   the population steps between optimisation steps

Scenes are drawn on the GPU with the distributions of the repository's own
workloads (`scenes.py`): a uniform box of primitives seen from distance 4, or
a room-scale mixture of flattened blobs seen from inside.
"""
import math

import torch

from paper_2501_16312_amd import linprim as L
from paper_2501_16312_amd import scenes
from paper_2501_16312_amd.graph import CapturedStep
from paper_2501_16312_amd.population import MCMC, PopulationControl
from paper_2501_16312_amd.render import Rasterizer, render

FIELDS = ("means", "quats", "dists", "opacity", "sh")
BG = (0.1, 0.2, 0.3)
BETA1, BETA2, EPS = 0.9, 0.999, 1e-15


def _view(name, **kw):
    case = {"name": name, "task": "render", "kind": "octa", "n": 1024, "scene": "box", "views": 1, "width": 128,
            "height": 128, "tile": 16, "sh_degree": 3, "backward": True, "via": "rasterizer", "exact_rays": False,
            "antialias": False, "depth": False, "radix": False, "size": 0.02}
    case.update(kw)
    return case


def listed():
    return [
        # the README's first program: a small scene through autograd, where
        # launches and the host path count
        _view("tiny_autograd", via="autograd", tile=8),
        # an interactive preview: forward only, low SH degree, default tile
        _view("preview_forward", n=20_000, scene="room", width=640, height=480, sh_degree=1, backward=False,
              size=0.06),
        # mid-size tetrahedra through autograd with the default tile
        _view("tetra_autograd_720p", kind="tetra", n=100_000, scene="room", width=1280, height=720, via="autograd",
              size=0.03),
        # the headline workload: 1M octahedra at 1080p, forward + backward
        _view("octa_1080p", n=1_000_000, scene="room", width=1920, height=1080, tile=8),
        # true pixel rays, an odd image size
        _view("exact_rays", n=300_000, scene="room", width=1597, height=1199, tile=8, exact_rays=True, size=0.03),
        # evaluation of a trained, denser scene: image and depth map with the
        # anti-aliasing filter, forward only, default tile
        _view("depth_eval", n=500_000, scene="room", width=1752, height=1168, backward=False, antialias=True,
              depth=True, size=0.04),
        # many views of mixed resolution in one captured graph
        _view("views16_graph", n=500_000, scene="room", views=16, width=0, height=0, tile=8, via="graph"),
        # the optimisation loop at scale: 3M octahedra, 8 views, L1, Adam, one
        # captured graph replayed on new poses and targets
        {"name": "train_graph", "task": "train", "kind": "octa", "n": 3_000_000, "scene": "room", "views": 8,
         "width": 1920, "height": 1080, "tile": 8, "sh_degree": 3, "via": "graph", "loss": "l1", "size": 0.02},
        # the ordinary training loop: one odd-sized view per step, L1 + SSIM,
        # Adam and densification statistics, launched call by call
        {"name": "train_eager", "task": "train", "kind": "octa", "n": 300_000, "scene": "room", "views": 1,
         "width": 1237, "height": 822, "tile": 16, "sh_degree": 3, "via": "eager", "loss": "l1_ssim",
         "size": 0.03},
        # the photometric loss of a batch
        {"name": "loss_ssim", "task": "loss", "views": 4, "width": 1920, "height": 1080},
        # population steps on a million primitives with their Adam moments
        {"name": "mcmc_step", "task": "mcmc", "kind": "octa", "n": 1_000_000, "sh_degree": 3, "grow": 0.05},
        {"name": "densify_step", "task": "densify", "kind": "octa", "n": 1_000_000, "sh_degree": 3},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    task = rng.choice(["render", "render", "render", "render", "train", "train", "loss", "mcmc", "densify"])
    kind = rng.choice(["octa", "octa", "tetra"])
    if task == "loss":
        return {"task": task, "views": rng.randint(1, 4), "width": _log_int(rng, 64, 1920),
                "height": _log_int(rng, 64, 1080)}
    if task == "mcmc":
        return {"task": task, "kind": "octa", "n": _log_int(rng, 10_000, 1_000_000),
                "sh_degree": rng.randint(0, 3), "grow": 0.05}
    if task == "densify":
        return {"task": task, "kind": kind, "n": _log_int(rng, 10_000, 1_000_000), "sh_degree": rng.randint(0, 3)}
    if task == "train":
        n = _log_int(rng, 20_000, 1_000_000)
        via = rng.choice(["graph", "eager"])
        return {"task": task, "kind": kind, "n": n, "scene": "room", "views": rng.randint(1, 4),
                "width": _log_int(rng, 320, 1920), "height": _log_int(rng, 240, 1080),
                "tile": rng.choice([8, 16]), "sh_degree": rng.randint(1, 3), "via": via,
                "loss": rng.choice(["l1", "l1_ssim"]), "size": round(0.02 * (1e6 / n) ** (1 / 3), 4)}
    n = _log_int(rng, 1_000, 1_000_000)
    scene = "box" if n < 10_000 else "room"
    exact_rays = rng.random() < 0.25
    backward = rng.random() < 0.7
    via = rng.choice(["autograd", "rasterizer", "graph"]) if backward else "rasterizer"
    return _view("", task=task, kind=kind, n=n, scene=scene, views=rng.choice([1, 1, 1, 2, 5]),
                 width=_log_int(rng, 100, 1920), height=_log_int(rng, 100, 1080), tile=rng.choice([8, 8, 16, 16, 32]),
                 sh_degree=rng.choice([0, 1, 2, 3, 3, 3]), backward=backward, via=via, exact_rays=exact_rays,
                 antialias=not exact_rays and rng.random() < 0.3, depth=not backward and rng.random() < 0.5,
                 radix=rng.random() < 0.1, size=round(0.02 * (1e6 / n) ** (1 / 3), 4))


# ------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _kind(case):
    return L.TETRAHEDRON if case["kind"] == "tetra" else L.OCTAHEDRON


def _extent(n):
    return 40.0 if n > 1_500_000 else 20.0


def _scene(case, g):
    """Primitive features, float32 on the GPU."""
    n, kind = case["n"], _kind(case)
    nd = 3 if kind == L.OCTAHEDRON else 4
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    uni = lambda *s: torch.rand(*s, generator=g, device="cuda")
    if case.get("scene", "room") == "box":
        means = 2.0 * uni(n, 3) - 1.0
        dists = 0.02 * torch.exp(uni(n, nd) * math.log(5.0))
        opacity = torch.sigmoid(rnd(n))
    else:
        half, k = _extent(n) / 2, 256
        centres = (2.0 * uni(k, 3) - 1.0) * half
        rots = torch.linalg.qr(rnd(k, 3, 3).cpu())[0].to("cuda")
        s = (0.02 + 0.08 * uni(k)) * 2.0 * half
        comp = torch.randint(0, k, (n,), generator=g, device="cuda")
        local = rnd(n, 3) * torch.stack([s, s, 0.05 * s], 1)[comp]
        means = (torch.matmul(rots[comp], local[:, :, None])[:, :, 0] + centres[comp]).clamp(-half, half)
        dists = torch.exp(math.log(case.get("size", 0.02)) + 0.7 * rnd(n, nd))
        opacity = torch.sigmoid(1.5 * rnd(n))
    quats = rnd(n, 4)
    quats = quats / quats.norm(dim=1, keepdim=True)
    K = (case["sh_degree"] + 1) ** 2
    sh = 0.2 * rnd(n, K, 3)
    return {"means": means, "quats": quats, "dists": dists, "opacity": opacity, "sh": sh}


def _cameras(case, g):
    angle = float(torch.rand(1, generator=g, device="cuda")) * 2.0 * math.pi
    v = case["views"]
    if case.get("scene", "room") == "box":
        dist = 4.0
    else:
        dist = 16.0 if _extent(case["n"]) > 20.0 else 8.0
    cams = []
    for k in range(v):
        a = angle + 2.0 * math.pi * k / v
        if case["width"]:
            w, h = case["width"], case["height"]
        else:
            w, h = scenes.MULTI_VIEW_SIZES[k % len(scenes.MULTI_VIEW_SIZES)]
        pos = (dist * math.cos(a), 0.3 * math.sin(3 * a), dist * math.sin(a))
        cams.append(scenes.look_at(pos, (0.0, 0.0, 0.0), w, h))
    return cams


def _pixels(cams):
    return sum(c.width * c.height for c in cams)


def _images(cams, g):
    """Packed target images: smooth structure plus noise, in [0, 1]."""
    parts = []
    for c in cams:
        low = torch.rand(1, 3, 9, 16, generator=g, device="cuda")
        img = torch.nn.functional.interpolate(low, size=(c.height, c.width), mode="bilinear", align_corners=True)
        img = img + 0.05 * torch.randn(img.shape, generator=g, device="cuda")
        parts.append(img.clamp(0.0, 1.0).reshape(-1))
    return torch.cat(parts)


def _moments(params, scale, g):
    """Adam moments in mid-training: second moments around the square of a
    typical gradient, first moments a fraction of it."""
    m, v = {}, {}
    for k, t in params.items():
        m[k] = 0.1 * scale * torch.randn(t.shape, generator=g, device="cuda")
        v[k] = scale * scale * (0.5 + torch.rand(t.shape, generator=g, device="cuda"))
    return m, v


def _scene_scale(cams):
    return 8.0 if len(cams) == 1 else 16.0


def _groups(case, params, grads, m, v, cams):
    # the rates late in a schedule, so that the scene stays what it is
    # however often the step runs
    s = 0.01 * _scene_scale(cams)
    lr = {"means": 1.6e-4 * s, "quats": 1e-5, "dists": 1e-4 / 2.6 * s, "opacity": 2.5e-4, "sh": 2.5e-5}
    out = []
    for k in FIELDS:
        d = {"param": params[k], "exp_avg": m[k], "exp_avg_sq": v[k], "lr": lr[k]}
        if grads is not None:
            d["grad"] = grads[k]
        if k == "dists":
            d["lo"] = 1e-5
        if k == "opacity":
            d["lo"], d["hi"] = 0.0, 1.0
        if k == "sh" and case["sh_degree"] > 0:
            d["period"], d["head"], d["lr_tail"] = 3 * (case["sh_degree"] + 1) ** 2, 3, 1.25e-6
        out.append(d)
    return out


STEP0 = 1000          # optimisation steps already taken


def _inputs(case, seed):
    g = _gen(seed)
    task = case["task"]
    if task == "loss":
        cams = [scenes.look_at((8.0, 0.0, 0.0), (0.0, 0.0, 0.0), case["width"], case["height"])
                for _ in range(case["views"])]
        target = _images(cams, g)
        rgb = (target + 0.1 * torch.randn(target.shape, generator=g, device="cuda")).clamp_min(0.0)
        return {"cams": cams, "target": target, "rgb": rgb}
    out = {"params": _scene(case, g)}
    p = out["params"]
    n = case["n"]
    if task == "render":
        out["cams"] = _cameras(case, g)
        if case["backward"]:
            out["grad_rgb"] = torch.randn(3 * _pixels(out["cams"]), generator=g, device="cuda")
    elif task == "train":
        out["cams"] = _cameras(case, g)
        out["target"] = _images(out["cams"], g)
        scale = 30.0 / (3 * _pixels(out["cams"]))
        out["m"], out["v"] = _moments(p, scale, g)
    elif task == "mcmc":
        # a few percent of the primitives have faded out
        p["opacity"] = torch.where(torch.rand(n, generator=g, device="cuda") < 0.02,
                                   torch.full_like(p["opacity"], 0.003), p["opacity"]).clamp_min(0.003)
        out["m"], out["v"] = _moments(p, 1e-6, g)
        add = int(case["grow"] * n)
        words = lambda k: torch.randint(0, 2 ** 32, (k,), generator=g, dtype=torch.int64, device="cuda").to(torch.int32)
        out["rand"], out["rand_add"] = words(n + add), words(max(add, 1))
        out["normals"] = torch.randn(n + add, 3, generator=g, device="cuda")
    else:
        out["m"], out["v"] = _moments(p, 1e-6, g)
        # fixed shares, in random places: 5% cloned, 5% split, 8% transparent
        # and 2% too wide on screen (removed), the others kept
        cls = torch.zeros(n, dtype=torch.long, device="cuda")
        where, at = torch.randperm(n, generator=g, device="cuda"), 0
        for c, share in ((1, 0.05), (2, 0.05), (3, 0.08), (4, 0.02)):
            cls[where[at: at + int(share * n)]] = c
            at += int(share * n)
        uni = lambda lo, hi: lo + (hi - lo) * torch.rand(n, generator=g, device="cuda")
        p["opacity"] = torch.where(cls == 3, uni(0.0, 0.02), uni(0.05, 1.0))
        d = p["dists"].clamp(0.001, 0.09)
        p["dists"] = torch.where((cls == 2)[:, None], d + uni(0.2, 0.5)[:, None], d)
        out["count"] = torch.randint(1, 40, (n,), generator=g, dtype=torch.int32, device="cuda")
        avg = torch.where((cls == 1) | (cls == 2), uni(2e-4, 5e-4), uni(0.0, 1e-4))
        out["grad_accum"] = avg * out["count"]
        out["max_radius"] = torch.where(cls == 4, uni(21.0, 60.0), uni(0.5, 19.0))
        out["normals"] = torch.randn(n, 2, 3, generator=g, device="cuda")
    return out


# ------------------------------------------------------------------ prepare
def prepare(case, seed):
    inp = _inputs(case, seed)
    task = case["task"]
    st = {"case": case, **inp}
    if task == "loss":
        st["cams_c"] = L.cameras(inp["cams"])
        st["ws"] = torch.empty(L.linprim_loss_workspace_size(st["cams_c"]), dtype=torch.uint8, device="cuda")
        st["grad"] = torch.empty_like(inp["rgb"])
        return st
    if task in ("mcmc", "densify"):
        return st
    kind = _kind(case)
    prims = L.Prims(kind, *(inp["params"][k] for k in FIELDS), sh_degree=case["sh_degree"])
    st["prims"] = prims
    rast = Rasterizer(kind, case["n"], inp["cams"], tile=case["tile"], headroom=1.25,
                      views_resident=(task == "train" and case["via"] == "graph"),
                      radix_sort=case.get("radix", False), exact=case.get("exact_rays", False),
                      antialias=case.get("antialias", False))
    st["rast"] = rast
    if task == "render":
        if case["via"] == "autograd":
            st["leaves"] = [inp["params"][k].requires_grad_(True) for k in FIELDS]
        elif case["via"] == "graph":
            st["step"] = CapturedStep(rast, prims, BG, grad_rgb=inp["grad_rgb"])
        return st
    grads = rast.alloc_grads(prims)
    st["grads"] = grads
    groups = _groups(case, inp["params"], grads, inp["m"], inp["v"], inp["cams"])
    st["groups"] = groups
    if case["via"] == "graph":
        st["buffer"] = inp["target"].clone()
        step = CapturedStep(rast, prims, BG, target=st["buffer"], grads=grads, loss=case["loss"],
                            adam={"groups": groups, "beta1": BETA1, "beta2": BETA2, "eps": EPS})
        step.step_count = STEP0
        st["step"] = step
    else:
        st["steps"] = STEP0
        st["pop"] = PopulationControl(kind, case["sh_degree"], case["n"])
        st["loss_ws"] = torch.empty(L.linprim_loss_workspace_size(rast.cams_c), dtype=torch.uint8, device="cuda")
        st["grad_rgb"] = torch.empty_like(inp["target"])
        st["partial"] = torch.zeros((inp["target"].numel() + 1023) // 1024, device="cuda")
    return st


# ---------------------------------------------------------------------- run
def run(state):
    case = state["case"]
    task = case["task"]
    if task == "loss":
        L.linprim_loss_grad(state["rgb"], state["target"], state["cams_c"], state["ws"], state["grad"])
        return {"grad": state["grad"]}
    if task == "mcmc":
        return _run_mcmc(state)
    if task == "densify":
        return _run_densify(state)
    if task == "train":
        return _run_train(state)
    rast, prims = state["rast"], state["prims"]
    if case["via"] == "graph":
        state["step"].replay()
        rgb, T, last = state["step"].outs
        return {"rgb": rgb, "T": T, "last": last, **state["step"].grads}
    if case["via"] == "autograd":
        leaves = state["leaves"]
        for t in leaves:
            t.grad = None
        rgb = render(rast, prims.kind, *leaves, sh_degree=case["sh_degree"], bg=BG)
        rgb.backward(state["grad_rgb"])
        return {"rgb": rgb.detach(), **{k: t.grad for k, t in zip(FIELDS, leaves)}}
    if case["depth"]:
        rast.preprocess(prims)
        rast.bin_sort(prims)
        depth = torch.empty(rast.n_pixels, device="cuda")
        rgb, T, last = rast.render(prims, BG, depth=depth)
        return {"rgb": rgb, "T": T, "last": last, "depth": depth}
    rgb, T, last = rast.forward(prims, BG)
    out = {"rgb": rgb, "T": T, "last": last}
    if case["backward"]:
        out.update(rast.backward(prims, BG, T, last, state["grad_rgb"]))
    return out


def _run_train(state):
    case, rast, prims = state["case"], state["rast"], state["prims"]
    if case["via"] == "graph":
        step = state["step"]
        rast.set_views(state["cams"])
        state["buffer"].copy_(state["target"])
        step.replay()
        rgb = step.outs[0]
    else:
        rgb, T, last = rast.forward(prims, BG)
        if case["loss"] == "l1_ssim":
            L.linprim_loss_grad(rgb, state["target"], rast.cams_c, state["loss_ws"], state["grad_rgb"])
        else:
            L.linprim_l1_grad(rgb, state["target"], 1.0 / rgb.numel(), state["grad_rgb"], state["partial"])
        rast.backward(prims, BG, T, last, state["grad_rgb"], state["grads"])
        state["pop"].accumulate(rast, prims)
        state["steps"] += 1
        L.linprim_adam_step(state["groups"], BETA1, BETA2, EPS, state["steps"])
    out = {"rgb": rgb}
    for k, g in zip(FIELDS, state["groups"]):
        out["g_" + k], out["p_" + k] = state["grads"][k], g["param"]
        out["m_" + k], out["v_" + k] = g["exp_avg"], g["exp_avg_sq"]
    return out


def _run_mcmc(state):
    # growth first (new arrays), then relocation and noise in place on them:
    # the state's own arrays stay as they are
    case = state["case"]
    mc = MCMC(case["n"], case["sh_degree"])
    p, m, v = mc.add(state["params"], int(case["grow"] * case["n"]), state["m"], state["v"],
                     rand_u32=state["rand_add"])
    mc.relocate(p, m, v, rand_u32=state["rand"])
    mc.noise(p, 1e-4, normals=state["normals"])
    return {"p": p, "m": m, "v": v}


def _run_densify(state):
    case = state["case"]
    pc = PopulationControl(_kind(case), case["sh_degree"], case["n"])
    pc.grad_accum, pc.count, pc.max_radius = state["grad_accum"], state["count"], state["max_radius"]
    p, m, v = pc.densify(state["params"], 20.0, state["m"], state["v"], normals=state["normals"])
    return {"p": p, "m": m, "v": v}


# --------------------------------------------------------------------- work
def work(case):
    task = case["task"]
    if task == "loss":
        px = case["views"] * case["width"] * case["height"]
        # five windowed statistics and three adjoint maps, 22 multiply-adds each
        return {"bytes": 36 * px, "flops": 3 * px * (8 * 44 + 60)}
    nd = 4 if case["kind"] == "tetra" else 3
    words = 3 + 4 + nd + 1 + 3 * (case["sh_degree"] + 1) ** 2
    n = case["n"]
    if task == "mcmc":
        add = int(case["grow"] * n)
        # every row with its moments moved into the grown arrays, the copied
        # rows (added, and 2% relocated), randoms and noise
        rows = add + n // 50
        return {"bytes": n * 4 * 6 * words + rows * 4 * 5 * words + n * 4 * 5, "flops": 150 * n}
    if task == "densify":
        return {"bytes": n * 4 * (6 * words + 3), "flops": 20 * n}
    if case["width"]:
        px = case["views"] * case["width"] * case["height"]
    else:
        sizes = scenes.MULTI_VIEW_SIZES
        px = sum(sizes[k % len(sizes)][0] * sizes[k % len(sizes)][1] for k in range(case["views"]))
    # about six evaluated (pixel, primitive) pairs a pixel, 108 operations
    # forward and 220 backward
    if task == "train":
        return {"bytes": n * 4 * 8 * words + px * 4 * (3 + 3), "flops": px * 6 * 328 + n * (12 * words + 2000)}
    nbytes = n * 4 * words + px * 4 * (5 + (1 if case["depth"] else 0))
    flops = px * 6 * 108 + n * case["views"] * 600
    if case["backward"]:
        nbytes += n * 4 * words + px * 12
        flops += px * 6 * 220 + n * case["views"] * 1200
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------- outputs in double precision
SLABS = ((1, 1, 1), (1, 1, -1), (1, -1, 1), (-1, 1, 1))
TET = ((1, 1, 1), (1, -1, -1), (-1, 1, -1), (-1, -1, 1))


def _rotation(q):
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).reshape(-1, 3, 3)


def _sh_basis(deg, d):
    x, y, z = d.unbind(1)
    pi = math.pi
    Y = [torch.full_like(x, 0.5 * math.sqrt(1 / pi))]
    if deg >= 1:
        c = math.sqrt(3 / (4 * pi))
        Y += [-c * y, c * z, -c * x]
    if deg >= 2:
        a, b, c = 0.5 * math.sqrt(15 / pi), 0.25 * math.sqrt(5 / pi), 0.25 * math.sqrt(15 / pi)
        Y += [a * x * y, -a * y * z, b * (2 * z * z - x * x - y * y), -a * x * z, c * (x * x - y * y)]
    if deg >= 3:
        a, b = 0.25 * math.sqrt(35 / (2 * pi)), 0.5 * math.sqrt(105 / pi)
        c, d_, e = 0.25 * math.sqrt(21 / (2 * pi)), 0.25 * math.sqrt(7 / pi), 0.25 * math.sqrt(105 / pi)
        Y += [-a * y * (3 * x * x - y * y), b * x * y * z, -c * y * (4 * z * z - x * x - y * y),
              d_ * z * (2 * z * z - 3 * x * x - 3 * y * y), -c * x * (4 * z * z - x * x - y * y),
              e * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)]
    return torch.stack(Y, 1)


class _View64:
    """The rendering definition for one view: primitives that may touch a
    pixel, their planes, colour and density, in double precision."""

    def __init__(self, case, p, cam, keep=None):
        f64 = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda")
        kind, self.exact = _kind(case), case.get("exact_rays", False)
        self.kind = kind
        w2c = f64(cam.world_to_cam)
        Rw, tw = w2c[:, :3], w2c[:, 3]
        fx, fy, cx, cy = (float(v) for v in (cam.fx, cam.fy, cam.cx, cam.cy))
        near = float(torch.tensor(cam.near, dtype=torch.float32))
        if keep is not None:
            p = {k: t[keep] for k, t in p.items()}
        R = _rotation(p["quats"])
        if kind == L.OCTAHEDRON:
            off = (R * p["dists"][:, None, :]).transpose(1, 2)
        else:
            off = torch.matmul(f64(TET) / math.sqrt(3.0), R.transpose(1, 2)) * p["dists"][:, :, None]
        tc = torch.matmul(p["means"], Rw.T) + tw
        oc = torch.matmul(off, Rw.T)
        x, y, z = tc.unbind(1)
        l = tc.norm(dim=1)
        u, v = fx * x / z + cx, fy * y / z + cy
        ax = fx * (oc[..., 0] / z[:, None] - (x / z ** 2)[:, None] * oc[..., 2])
        ay = fy * (oc[..., 1] / z[:, None] - (y / z ** 2)[:, None] * oc[..., 2])
        az = (oc * tc[:, None, :]).sum(2) / l[:, None]
        if case.get("antialias", False):
            ax, ay = self._shift(ax), self._shift(ay)
        with torch.no_grad():
            ok = z > near
            if self.exact:
                co = torch.cat([tc[:, None] + oc, tc[:, None] - oc], 1) if kind == L.OCTAHEDRON else tc[:, None] + oc
                ok &= (co[..., 2] > near).all(1)
                px, py = fx * co[..., 0] / co[..., 2] + cx, fy * co[..., 1] / co[..., 2] + cy
            elif kind == L.OCTAHEDRON:
                px = torch.cat([u[:, None] + ax, u[:, None] - ax], 1)
                py = torch.cat([v[:, None] + ay, v[:, None] - ay], 1)
            else:
                px, py = u[:, None] + ax, v[:, None] + ay
            i0 = torch.ceil(px.min(1).values - 0.5).clamp_min(0.0)
            i1 = torch.floor(px.max(1).values - 0.5).clamp_max(cam.width - 1.0)
            j0 = torch.ceil(py.min(1).values - 0.5).clamp_min(0.0)
            j1 = torch.floor(py.max(1).values - 0.5).clamp_max(cam.height - 1.0)
            self.ok = ok & (i0 <= i1) & (j0 <= j1)
            self.rect = (i0, j0, i1, j1)
        self.depth_key = tc[:, 2].detach().float()
        self.centre = z if self.exact else l
        self.cam = (fx, fy, cx, cy)
        # planes n . (X - centre) <= 1 of every face, the octahedron's as slabs
        a = oc if self.exact else torch.stack([ax, ay, az], 2)
        M = a[:, :3] if kind == L.OCTAHEDRON else None
        if kind == L.OCTAHEDRON:
            n = torch.matmul(f64(SLABS), torch.linalg.inv(M.transpose(1, 2)))
        else:
            n = torch.stack([torch.linalg.inv(a[:, [k for k in range(4) if k != f]]).sum(2) for f in range(4)], 1)
        self.n, self.u, self.v, self.tc = n, u, v, tc
        campos = -torch.matmul(Rw.T, tw)
        d = p["means"] - campos
        Y = _sh_basis(case["sh_degree"], d / d.norm(dim=1, keepdim=True))
        self.rgb = ((Y[:, :, None] * p["sh"]).sum(1) + 0.5).clamp_min(0.0)
        dmin = p["dists"].detach().min(1).values
        self.sigma = -torch.log(1 - 0.99 * p["opacity"]) / (2 * dmin)

    def _shift(self, a):
        d = a.detach()
        if self.kind == L.OCTAHEDRON:
            return a + torch.where(d.abs() == d.abs().max(1, keepdim=True).values, 0.05 * d.sign(), 0.0)
        lo, hi = d.min(1, keepdim=True).values, d.max(1, keepdim=True).values
        return a + 0.05 * (d == hi) - 0.05 * (d == lo)

    def chord(self, idx, px, py):
        """Chord and entry (relative to the centre's depth) of the pixel rays."""
        n = self.n[idx]
        inf = torch.tensor(math.inf, dtype=torch.float64, device="cuda")
        if self.exact:
            fx, fy, cx, cy = self.cam
            D = torch.stack([(px - cx) / fx, (py - cy) / fy, torch.ones_like(px)], 1)
            den = (n * D[:, None]).sum(2)
            num = (n * (self.tc[idx])[:, None]).sum(2)
            zc = self.tc[idx, 2]
            scale = D.norm(dim=1)
        else:
            den = n[..., 2]
            num = -n[..., 0] * (px - self.u[idx])[:, None] - n[..., 1] * (py - self.v[idx])[:, None]
            zc, scale = 0.0, 1.0
        if self.kind == L.OCTAHEDRON:
            t1, t2 = (num - 1) / den, (num + 1) / den
            hi, lo = torch.maximum(t1, t2).min(1).values, torch.minimum(t1, t2).max(1).values
        else:
            t = (num + 1) / den
            hi = torch.where(den >= 0, t, inf).min(1).values
            lo = torch.where(den >= 0, -inf, t).max(1).values
        return (hi - lo) * scale, lo - zc, scale


def _hits(view, width):
    """(primitive, pixel x, pixel y) with a positive chord, in chunks."""
    i0, j0, i1, j1 = (r.long() for r in view.rect)
    vis = torch.nonzero(view.ok)[:, 0]
    w = (i1 - i0 + 1)[vis]
    area = w * (j1 - j0 + 1)[vis]
    out, start, ends = [], 0, torch.cumsum(area, 0)
    while start < vis.numel():
        base = int(ends[start - 1]) if start else 0
        stop = max(start + 1, int(torch.searchsorted(ends, base + 8_000_000)))
        a, ww, ii = area[start:stop], w[start:stop], vis[start:stop]
        own = torch.repeat_interleave(torch.arange(stop - start, device="cuda"), a)
        k = torch.arange(own.numel(), device="cuda") - (torch.cumsum(a, 0) - a)[own]
        x, y = i0[ii[own]] + k % ww[own], j0[ii[own]] + k // ww[own]
        c = view.chord(ii[own], x.double() + 0.5, y.double() + 0.5)[0]
        hit = c > 0
        out.append((ii[own][hit], x[hit], y[hit]))
        start = stop
    return tuple(torch.cat([o[k] for o in out]) if out else torch.zeros(0, dtype=torch.long, device="cuda")
                 for k in range(3))


def _render64(case, p, cam):
    """Image [3 H W], transmittance and depth map, differentiable in p."""
    hw = cam.width * cam.height
    with torch.no_grad():
        flat = _View64(case, {k: t.detach() for k, t in p.items()}, cam)
        idx, x, y = _hits(flat, cam.width)
        rank = torch.empty(case["n"], dtype=torch.long, device="cuda")
        rank[torch.sort(flat.depth_key, stable=True).indices] = torch.arange(case["n"], device="cuda")
        pix = y * cam.width + x
        order = torch.sort(pix * case["n"] + rank[idx]).indices
        idx, x, y, pix = idx[order], x[order], y[order], pix[order]
        del flat
        keep, idx = torch.unique(idx, return_inverse=True)
    T = torch.ones(hw, dtype=torch.float64, device="cuda")
    C = torch.zeros(3, hw, dtype=torch.float64, device="cuda")
    depth = torch.zeros(hw, dtype=torch.float64, device="cuda")
    if keep.numel():
        view = _View64(case, p, cam, keep)
        c, entry, scale = view.chord(idx, x.double() + 0.5, y.double() + 0.5)
        o = (1 - torch.exp(-view.sigma[idx] * c.clamp_min(0.0))).clamp_max(0.99)
        with torch.no_grad():
            first = torch.ones_like(pix, dtype=torch.bool)
            first[1:] = pix[1:] != pix[:-1]
            seg = torch.cumsum(first, 0) - 1
            head = torch.nonzero(first)[:, 0]

        def before(lg):
            s = torch.cumsum(lg, 0) - lg
            return s - s[head][seg]

        with torch.no_grad():
            alive = torch.exp(before(torch.log1p(-o))) > 1e-3
        o = torch.where(alive, o, torch.zeros_like(o))
        lg = torch.log1p(-o)
        Tb = torch.exp(before(lg))
        C = C.index_add(1, pix, (Tb * o)[None] * view.rgb[idx].T)
        T = torch.exp(torch.zeros(hw, dtype=torch.float64, device="cuda").index_add(0, pix, lg))
        with torch.no_grad():
            cross = (Tb >= 0.5) & (Tb * (1 - o) < 0.5)
            zc = view.centre[idx]
            depth[pix[cross]] = ((zc + entry) * scale)[cross]
    C = C + T * torch.tensor(BG, dtype=torch.float32, device="cuda").double()[:, None]
    return C.reshape(-1), T, depth


def _window():
    g = torch.exp(-(torch.arange(11, dtype=torch.float64, device="cuda") - 5) ** 2 / (2 * 1.5 ** 2))
    return g / g.sum()


def _blur(t):
    """11 x 11 Gaussian window with zero padding over [3, H, W]."""
    w = _window()
    H, W = t.shape[1:]
    a = torch.nn.functional.pad(t, (5, 5, 5, 5))
    b = sum(w[k] * a[:, :, k: k + W] for k in range(11))
    return sum(w[k] * b[:, k: k + H] for k in range(11))


def _loss_grad64(rgb, target, cams, lam=0.2):
    out, off = [], 0
    for c in cams:
        m = 3 * c.width * c.height
        x = rgb[off: off + m].double().reshape(3, c.height, c.width).detach().requires_grad_(True)
        y = target[off: off + m].double().reshape(3, c.height, c.width)
        mx, my = _blur(x), _blur(y)
        sxx, syy, sxy = _blur(x * x) - mx * mx, _blur(y * y) - my * my, _blur(x * y) - mx * my
        s = (2 * mx * my + 1e-4) * (2 * sxy + 9e-4) / ((mx * mx + my * my + 1e-4) * (sxx + syy + 9e-4))
        ((1 - lam) * (x - y).abs().mean() + lam * (1 - s.mean())).backward()
        out.append(x.grad.reshape(-1))
        off += m
    return torch.cat(out)


def _views64(case, params, cams, grad_of):
    """Images of all views and the gradients of sum(image * grad_of(view))."""
    p = {k: t.double().requires_grad_(True) for k, t in params.items()}
    rgbs, Ts, depths, off = [], [], [], 0
    for c in cams:
        C, T, depth = _render64(case, p, c)
        m = C.numel()
        if grad_of is not None:
            g = grad_of(C.detach(), off, m, c)
            (C * g).sum().backward()
        rgbs.append(C.detach())
        Ts.append(T.detach())
        depths.append(depth)
        off += m
        del C, T
    z = {k: (t.grad if t.grad is not None else torch.zeros_like(t)) for k, t in p.items()}
    return torch.cat(rgbs), torch.cat(Ts), torch.cat(depths), z


def exact(case, seed):
    inp = _inputs(case, seed)
    task = case["task"]
    if task == "loss":
        return {"grad": _loss_grad64(inp["rgb"], inp["target"], inp["cams"])}
    if task == "mcmc":
        return _exact_mcmc(case, inp)
    if task == "densify":
        return _exact_densify(case, inp)
    if task == "render":
        grad = inp.get("grad_rgb")
        fn = (lambda C, off, m, c: grad[off: off + m].double()) if grad is not None else None
        rgb, T, depth, g = _views64(case, inp["params"], inp["cams"], fn)
        if case["via"] == "autograd":
            return {"rgb": rgb, **g}
        out = {"rgb": rgb, "T": T, "last": None}
        if case["backward"]:
            out.update(g)
        elif case["depth"]:
            out["depth"] = depth
        return out
    if case["n"] > 1_500_000:
        return None          # the largest training step takes too long here
    target, total = inp["target"], inp["target"].numel()
    if case["loss"] == "l1":
        fn = lambda C, off, m, c: torch.sign(C - target[off: off + m].double()) / total
    else:
        fn = lambda C, off, m, c: _loss_grad64(C, target[off: off + m], [c])
    rgb, _, _, g = _views64(case, inp["params"], inp["cams"], fn)
    t = STEP0 + 1
    b1, b2 = (float(torch.tensor(b, dtype=torch.float32)) for b in (BETA1, BETA2))
    out = {"rgb": rgb}
    for k, grp in zip(FIELDS, _groups(case, inp["params"], None, inp["m"], inp["v"], inp["cams"])):
        m = b1 * grp["exp_avg"].double() + (1 - b1) * g[k]
        v = b2 * grp["exp_avg_sq"].double() + (1 - b2) * g[k] ** 2
        lr = torch.full_like(m, grp["lr"]).reshape(-1)
        if "period" in grp:
            lr = torch.where(torch.arange(lr.numel(), device="cuda") % grp["period"] >= grp["head"], grp["lr_tail"], lr)
        step = lr.reshape(m.shape) * (m / (1 - b1 ** t)) / (torch.sqrt(v / (1 - b2 ** t)) + EPS)
        p = (grp["param"].double() - step).clamp(grp.get("lo", -math.inf), grp.get("hi", math.inf))
        out["g_" + k], out["p_" + k], out["m_" + k], out["v_" + k] = g[k], p, m, v
    return out


def _draws(opacity, rand, count):
    w = torch.floor(opacity.double().cpu() * 2.0 ** 32).to(torch.int64)
    w[opacity.cpu() <= 0.005] = 0
    prefix = torch.cumsum(w, 0)
    total = int(prefix[-1])
    r = rand[:count].cpu().to(torch.int64) & 0xFFFFFFFF
    t = (total >> 32) * r + _mulshift(total & 0xFFFFFFFF, r)
    return torch.searchsorted(prefix, t, right=True).to("cuda")


def _mulshift(low, r):
    """(low r) >> 32 for low, r < 2^32, without overflow of 63 bits."""
    hi, lo = low >> 16, low & 0xFFFF
    return (hi * r + ((lo * r) >> 16)) >> 16


def _relocate64(p, m, v, src, target):
    c = torch.bincount(src, minlength=p["opacity"].numel())
    s = torch.nonzero(c)[:, 0]
    N = (c[s] + 1).clamp_max(51).double()
    a = p["opacity"][s]
    an = (1 - (1 - a) ** (1 / N)).clamp(0.005, 1 - 2.0 ** -23)
    # sum over i <= N, k < i of C(i-1, k) (-1)^k an^(k+1) / sqrt(k+1)
    denom = torch.zeros_like(an)
    for k in range(51):
        binom = torch.exp(torch.lgamma(N + 1) - torch.lgamma(torch.tensor(k + 2.0, dtype=torch.float64)) -
                          torch.lgamma((N - k).clamp_min(1.0)))
        denom += torch.where(N > k, (-1.0) ** k * binom * an ** (k + 1) / math.sqrt(k + 1), 0.0)
    p["dists"][s] = (p["dists"][s] * (a / denom)[:, None]).float().double()
    p["opacity"][s] = an.float().double()
    for k in FIELDS:
        m[k][s] = 0.0
        v[k][s] = 0.0
        p[k][target] = p[k][src]
        m[k][target] = 0.0
        v[k][target] = 0.0


def _exact_mcmc(case, inp):
    n, add = case["n"], int(case["grow"] * case["n"])
    grow = lambda t: torch.cat([t.double(), torch.zeros((add,) + tuple(t.shape[1:]), dtype=torch.float64,
                                                        device="cuda")])
    p, m, v = ({k: grow(t) for k, t in inp[key].items()} for key in ("params", "m", "v"))
    op = p["opacity"][:n].float()
    _relocate64(p, m, v, _draws(op, inp["rand_add"], add), torch.arange(n, n + add, device="cuda"))
    op = p["opacity"].float()
    dead = torch.nonzero(op <= 0.005)[:, 0]
    _relocate64(p, m, v, _draws(op, inp["rand"], dead.numel()), dead)
    gate = 1 / (1 + torch.exp(-100 * ((1 - p["opacity"]) - 0.995)))
    R = _rotation(p["quats"])
    e = torch.matmul(R.transpose(1, 2), inp["normals"].double()[:, :, None])[:, :, 0]
    e = torch.matmul(R, (e * (p["dists"] / 2.6) ** 2)[:, :, None])[:, :, 0]
    lr = float(torch.tensor(1e-4, dtype=torch.float32))
    p["means"] += 5e5 * lr * gate[:, None] * e
    return {"p": p, "m": m, "v": v}


def _exact_densify(case, inp):
    p, m, v = inp["params"], inp["m"], inp["v"]
    octa = _kind(case) == L.OCTAHEDRON
    dm = p["dists"].max(1).values
    size = 2.0 * dm if octa else torch.tensor(math.sqrt(2.0), device="cuda") * dm
    cnt = inp["count"]
    avg = torch.where(cnt > 0, inp["grad_accum"] / cnt.clamp_min(1).float(), 0.0)
    f32 = lambda a: float(torch.tensor(a, dtype=torch.float32))
    big = float(torch.tensor(0.4, dtype=torch.float32) * 20.0)
    cand, small = avg > f32(1.5e-4), size < float(torch.tensor(0.01, dtype=torch.float32) * 20.0)
    solid = ~(p["opacity"] < f32(0.025))
    split = cand & ~small
    keep = ~split & solid & ~(size > big) & ~(inp["max_radius"] > 20.0)
    two = split & solid & ~(size / torch.tensor(1.2, device="cuda") > big)
    clone = cand & small & solid & ~(size > big)
    n = case["n"]
    i = torch.arange(n, device="cuda")
    key = torch.cat([i[keep] * 4, i[two] * 4, i[two] * 4 + 1, i[clone] * 4 + 2])
    typ = torch.cat([torch.zeros_like(i[keep]), torch.ones_like(i[two]), torch.full_like(i[two], 2),
                     torch.full_like(i[clone], 3)])
    order = torch.sort(key, stable=True).indices
    src, typ = (key // 4)[order], typ[order]
    out = {k: t[src].double() for k, t in p.items()}
    child = (typ == 1) | (typ == 2)
    s = src[child]
    z = inp["normals"].double()[s, (typ[child] - 1)]
    if octa:
        off = torch.matmul(_rotation(p["quats"][s].double()), (p["dists"][s].double() * z)[:, :, None])[:, :, 0]
    else:
        off = 0.5 * dm[s].double()[:, None] * z
    out["means"][child] += off
    out["dists"][child] /= f32(1.2)
    mo = {k: torch.where((typ == 0).reshape([-1] + [1] * (t.dim() - 1)), t[src], 0.0) for k, t in m.items()}
    vo = {k: torch.where((typ == 0).reshape([-1] + [1] * (t.dim() - 1)), t[src], 0.0) for k, t in v.items()}
    return {"p": out, "m": mo, "v": vo}
