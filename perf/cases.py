"""Performance cases of the LoD-select + splat path, through its public Python
entry points.

A case names a seeded scene (the input generator's leaf distributions at a
stated number of leaves), a camera of a stated kind over it, an image size, a
pixel threshold and what a program does with the view:

  forward   lod_select + render: a viewer, or one request of a server
  graph     the same view replayed from a captured HIP graph: a server's slot
  autograd  render_lod + backward to dense parameter gradients: a small
            optimisation written in plain torch
  step      lod_select, render, L1 against a target, backward accumulating in
            node-indexed gradients: one training view of a larger batch
  adam      lod_select, render, L1, backward into the selection's gradients,
            Adam on the cut set: one training iteration
  batch     several views through render_lod on three streams, their gradients
            accumulated on a scatter stream, one backward for all
  pooled    parameters in host memory: cached cut, row-pool gather, render from
            the rows, L1, backward into the rows' gradients

The seed makes the scene, the camera's place, the target and the cotangent.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import scenegen
from paper_2507_01110_amd.autograd import render_lod
from paper_2507_01110_amd.lodgs import (GROUPS, AdamCut, CutCache, Frame, HostParams, RowPool, Scene, ViewGraph,
                                        grads_like, rows_like)
from scenegen import configs

# Late-schedule learning rates: the parameters of a timed scene stay where
# training left them however often a pass is repeated.
ADAM_LR = {"means": 1e-7, "log_scales": 1e-6, "quats": 1e-6, "opacity_logits": 1e-6, "sh": 1e-6}
BACKGROUND = (0.1, 0.2, 0.3)


def listed():
    """The cases, smallest first."""
    def case(name, kind, scene, leaves, camera, width, height, tau, degree=3, views=1):
        return {"name": name, "kind": kind, "scene": scene, "leaves": leaves, "camera": camera, "width": width,
                "height": height, "tau": tau, "degree": degree, "views": views}
    return [
        # a viewer on a small object: launches and latency count
        case("preview 512", "forward", "cube", 16384, "orbit", 512, 512, 1.0),
        # a small optimisation in plain torch, dense gradients
        case("autograd 512", "autograd", "cube", 16384, "orbit", 512, 512, 1.0),
        # an odd image size, degree 1, a training iteration on a small scene
        case("iteration 333x171", "adam", "ground", 60001, "oblique", 333, 171, 1.0, degree=1),
        # the smallest request class of the server, from its captured graph
        case("request 360p", "graph", "city", 500_000, "oblique", 640, 360, 1.0),
        # out-of-core training view whose cut is already pooled
        case("pooled 720p", "pooled", "city", 250_000, "oblique", 1280, 720, 1.0),
        # an ordinary full-HD view
        case("view 1080p", "forward", "ground", 1_000_000, "oblique", 1920, 1080, 1.0),
        # full-HD training views at the two ends of an aerial-to-street path
        case("step 1080p aerial", "step", "city", 4_000_000, "aerial", 1920, 1080, 2.0),
        case("step 1080p street", "step", "city", 6_000_000, "street", 1920, 1080, 0.5),
        # a full-HD training iteration with the optimiser
        case("iteration 1080p", "adam", "ground", 2_000_000, "oblique", 1920, 1080, 1.0),
        # the largest request class of the server
        case("view 4k street", "forward", "city", 4_000_000, "street", 3840, 2160, 1.0),
        # a batch of full-HD views over the whole path, gradients accumulated
        case("batch 8x1080p", "batch", "city", 1_000_000, "path", 1920, 1080, 1.0, views=8),
    ]


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(["forward", "forward", "step", "step", "adam", "graph", "autograd", "batch", "pooled"])
    logu = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    scene = rng.choice(["cube", "ground", "city", "city"])
    top = {"autograd": 200_000, "pooled": 250_000, "batch": 300_000}.get(kind, 4_000_000)
    leaves = logu(4096, min(top, (50_000 if kind == "batch" else 200_000) if scene == "cube" else 4_000_000))
    if kind == "forward":
        width, height = rng.choice([(640, 360), (1280, 720), (1920, 1080), (3840, 2160),
                                    (logu(64, 1920), logu(64, 1080))])
    elif rng.random() < 0.5:
        width, height = rng.choice([(512, 512), (640, 360), (1280, 720), (1920, 1080)])
    else:
        width, height = logu(64, 1920), logu(64, 1080)
    camera = "orbit" if scene == "cube" else rng.choice(["aerial", "oblique", "street"])
    if kind == "batch":
        camera = "orbit" if scene == "cube" else "path"
    return {"kind": kind, "scene": scene, "leaves": leaves, "camera": camera, "width": width, "height": height,
            "tau": round(math.exp(rng.uniform(math.log(0.5), math.log(2.0))), 3),
            "degree": rng.choice([0, 1, 2, 3, 3, 3]), "views": rng.randint(2, 6) if kind == "batch" else 1}


# ------------------------------------------------------------------ inputs
def extent(case):
    """Half extent of the scene in metres: the leaf densities of the workload
    recipes (16,384 in a 20 m cube, 8 and about 3 per square metre)."""
    n = case["leaves"]
    if case["scene"] == "cube":
        return 10.0 * (n / 16384.0) ** (1.0 / 3.0)
    return 0.5 * math.sqrt(n / (8.0 if case["scene"] == "ground" else 3.125))


def make_tree(case, seed):
    n, ext, deg = case["leaves"], extent(case), case["degree"]
    if case["scene"] == "cube":
        spec = configs.tiny_spec(n=n, seed=seed, sh_degree=deg)
        spec.half_extent = ext
    elif case["scene"] == "ground":
        spec = configs.medium_spec(n=n, seed=seed, sh_degree=deg)
        spec.half_extent, spec.n_boxes = ext, max(4, n // 10_000)
    else:
        spec = configs.city_spec(n=n, seed=seed, half_extent=ext, n_boxes=max(4, n // 2500), sh_degree=deg)
    return scenegen.build_tree(spec)


def make_cameras(case, seed):
    """The views' cameras: the kind's pose with a seeded place and heading."""
    rng = np.random.default_rng(np.random.PCG64(seed))
    w, h, ext = case["width"], case["height"], extent(case)
    cams = []
    for b in range(case["views"]):
        if case["camera"] == "orbit":
            a = rng.uniform(0.0, 2.0 * math.pi)
            p = (3.0 * ext * math.sin(a), ext * rng.uniform(-0.5, 0.5), 3.0 * ext * math.cos(a))
            cams.append(scenegen.camera_look_at(p, (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), w, h))
            continue
        # from high over a corner, looking down, to eye height in the middle
        s = {"aerial": 0.0, "oblique": 0.6, "street": 1.0}.get(case["camera"], b / max(1, case["views"] - 1))
        alt = 0.8 * ext * (1.8 / (0.8 * ext)) ** s
        xy = -0.5 * ext * (1.0 - s) + rng.uniform(-0.02, 0.02, 2) * ext
        yaw = math.radians(45.0 + rng.uniform(-10.0, 10.0))
        cams.append(scenegen.camera_yaw_pitch((xy[0], xy[1], alt), yaw, math.radians(-60.0 * (1.0 - s)), w, h))
    return cams


def make_images(case, seed, device):
    """Targets of the L1 loss, or (autograd) the loss's derivative by the image."""
    g = torch.Generator().manual_seed(seed)
    shape = (case["views"], case["height"], case["width"], 3)
    if case["kind"] == "autograd":
        return (torch.randn(shape, generator=g) / (case["height"] * case["width"])).to(device)
    return torch.rand(shape, generator=g).to(device)


def max_instances(case):
    """Splat-tile pairs that a frame holds."""
    tiles = ((case["width"] + 15) // 16) * ((case["height"] + 15) // 16)
    return (1 << 20) + 12 * case["leaves"] + 64 * tiles


def prepare(case, seed):
    tree = make_tree(case, seed)
    scene = Scene(tree)
    kind, w, h = case["kind"], case["width"], case["height"]
    st = {"kind": kind, "scene": scene, "cams": make_cameras(case, seed + 1), "tau": case["tau"]}
    frames = [Frame(scene, scene.n_nodes, max_instances(case), w, h) for _ in range(case["views"])]
    st["frames"], st["frame"] = frames, frames[0]
    if kind not in ("forward", "graph"):
        st["images"] = make_images(case, seed + 2, scene.device)
    if kind == "graph":
        st["stream"] = torch.cuda.Stream()
        with torch.cuda.stream(st["stream"]):
            st["graph"] = ViewGraph(frames[0], st["cams"][0], st["tau"], st["stream"], bg=BACKGROUND)
    if kind in ("step", "batch"):
        st["grads"] = grads_like(scene)
    if kind == "batch":
        for t in scene.params.values():
            t.requires_grad_(True)
        st["streams"], st["scatter"] = [torch.cuda.Stream() for _ in range(3)], torch.cuda.Stream()
    if kind == "autograd":
        for t in scene.params.values():
            t.requires_grad_(True)
    if kind in ("adam", "pooled"):
        st["sel"] = grads_like(scene, scene.n_nodes)
    if kind == "adam":
        st["opt"] = AdamCut(scene.params, scene.sh_degree, lr=ADAM_LR)
    if kind == "pooled":
        st["cache"] = CutCache(scene, scene.n_nodes, 0.8, 1.25)
        st["host"] = HostParams.from_scene(scene)
        st["pool"] = RowPool(st["cache"], st["host"], scene.n_nodes)
        st["rows"] = rows_like(scene.sh_degree, scene.n_nodes)
    return st


# ------------------------------------------------------------------ a pass
def run(st):
    kind, f, cam, tau = st["kind"], st["frame"], st["cams"][0], st["tau"]
    if kind == "forward":
        f.lod_select(cam, tau)
        return {"idx": f.idx, "count": f.count, "image": f.render(cam, bg=BACKGROUND)}
    if kind == "graph":
        img = st["graph"].launch(cam, tau)
        return {"idx": f.idx, "count": f.count, "image": img}
    if kind == "autograd":
        img = render_lod(f, cam, tau, bg=BACKGROUND)
        params = [f.scene.params[k] for k in GROUPS]
        return {"image": img, "grads": dict(zip(GROUPS, torch.autograd.grad(img, params, st["images"][0])))}
    if kind == "batch":
        main = torch.cuda.current_stream()
        losses = []
        for b, (fb, cb) in enumerate(zip(st["frames"], st["cams"])):
            s = st["streams"][b % len(st["streams"])]
            s.wait_stream(main)
            with torch.cuda.stream(s):
                img = render_lod(fb, cb, tau, bg=BACKGROUND, accumulate_into=st["grads"],
                                 scatter_stream=st["scatter"])
                losses.append((img - st["images"][b]).abs().mean())
        for s in st["streams"]:
            main.wait_stream(s)
        losses = torch.stack(losses)
        losses.sum().backward()
        main.wait_stream(st["scatter"])
        return {"losses": losses.detach(), "grads": st["grads"]}
    if kind == "pooled":
        f.lod_select(cam, tau, cache=st["cache"])
        st["pool"].gather(f.idx, f.count, st["rows"])
        img = f.render_rows(cam, st["rows"], bg=BACKGROUND)
    else:
        f.lod_select(cam, tau)
        img = f.render(cam, bg=BACKGROUND)
    dL = f.l1_loss(img, st["images"][0])
    if kind == "step":
        f.backward(dL, nodes=st["grads"])
        return {"image": img, "dL": dL, "grads": st["grads"]}
    f.backward(dL, sel=st["sel"])
    if kind == "pooled":
        return {"idx": f.idx, "count": f.count, "image": img, "dL": dL, "grads": st["sel"]}
    opt = st["opt"]
    opt.step(st["sel"], f.idx, f.count)
    return {"image": img, "params": opt.params, "exp_avg": opt.exp_avg, "exp_avg_sq": opt.exp_avg_sq}


# ------------------------------------------------------------------ work
# Shares of a scene's nodes that are selected, and of those drawn, splat-tile
# pairs for each drawn splat at 1080p and contributing pixels for each pair, by
# camera: counted on views of the listed cases, rounded.
VIEW_COUNTS = {"orbit": (0.5, 1.0, 2.5, 15.0), "aerial": (0.06, 0.6, 3.7, 12.0), "oblique": (0.1, 0.2, 4.7, 45.0),
               "street": (0.13, 0.65, 2.2, 30.0), "path": (0.14, 0.3, 4.0, 35.0)}


def work(case):
    """Bytes and operations of a pass: the selected nodes' geometry and the
    drawn nodes' coefficients read once, the image written; backward: the
    image's derivative and the drawn nodes' parameters read, their gradients
    written (accumulating: read too; with Adam: both moments and the
    parameters read and written).  43 operations for each contribution of a
    splat to a pixel, 88 in the backward."""
    sel, drawn, pairs, hits = VIEW_COUNTS[case["camera"]]
    coef = 3 * (case["degree"] + 1) ** 2
    row = 4.0 * (11 + coef)
    n_sel = 2.0 * case["leaves"] * sel
    n_drawn = n_sel * drawn
    pix = case["width"] * case["height"]
    n_pairs = n_drawn * (1.0 + (pairs - 1.0) * math.sqrt(pix / (1920.0 * 1080.0)))
    out = 12.0 * pix
    b = n_sel * (4 + 44) + n_drawn * 4 * coef + out
    f = 43.0 * n_pairs * hits
    kind = case["kind"]
    if kind not in ("forward", "graph"):
        b += 2 * out + n_drawn * row + {"step": 2 * n_drawn, "batch": 2 * n_drawn, "adam": 6 * n_sel}.get(kind, n_sel) * row
        f += 88.0 * n_pairs * hits
    if kind == "autograd":
        b += 2.0 * case["leaves"] * row  # the dense gradients' other rows
    if kind == "pooled":
        b += n_sel * row
    return {"bytes": b * case["views"], "flops": f * case["views"]}


# ------------------------------------------------------------------ the results in 64 bits
def layout64(tree):
    """The hierarchy's layout in plain numpy: (perm, r_min, r_max, rho, upper,
    SPT index) by layout position; upper nodes in preorder, then the SPTs."""
    n, left, right = tree.n_nodes, tree.left.astype(np.int64), tree.right.astype(np.int64)
    s = np.exp(tree.log_scales.astype(np.float64))
    g = np.sqrt(s[:, 0] * s[:, 1] + s[:, 0] * s[:, 2] + s[:, 1] * s[:, 2]).astype(np.float32)
    rho = (3.0 * s.max(axis=1)).astype(np.float32)
    ls = tree.log_scales.astype(np.float64)
    cuts = (left < 0) | ((ls[:, 0] + ls[:, 1]) + ls[:, 2] < tree.log_volume_threshold)
    levels = [np.array([tree.root], np.int64)]
    while True:
        inner = levels[-1][left[levels[-1]] >= 0]
        if not inner.size:
            break
        levels.append(np.concatenate([left[inner], right[inner]]))
    size = np.ones(n, np.int64)
    for lev in reversed(levels):
        inner = lev[left[lev] >= 0]
        size[inner] += size[left[inner]] + size[right[inner]]
    pre = np.zeros(n, np.int64)
    spt = np.full(n, -1, np.int64)  # the SPT's root, -1 for an upper node
    parent = np.full(n, -1, np.int64)
    r_max = np.full(n, np.inf, np.float32)
    for lev in levels:
        own = lev[(spt[lev] < 0) & cuts[lev]]
        spt[own] = own
        inner = lev[left[lev] >= 0]
        below = np.minimum(r_max[inner], g[inner])
        for child, first in ((left[inner], pre[inner] + 1), (right[inner], pre[inner] + 1 + size[left[inner]])):
            pre[child], parent[child] = first, inner
            spt[child] = spt[inner]
            r_max[child] = np.where(spt[inner] >= 0, below, np.inf)
    r_min = np.where((left < 0) & (spt >= 0), np.float32(0.0), g)
    rank = np.where(spt >= 0, pre[np.maximum(spt, 0)], -1)
    perm = np.lexsort((np.arange(n), -r_min, -r_max, rank))
    n_up = int((spt < 0).sum())
    perm[:n_up] = perm[:n_up][np.argsort(pre[perm[:n_up]])]
    return perm, r_min, r_max, rho, spt, parent, levels


def cut64(tree, lay, cam, tau):
    """Selected tree nodes of a view, in layout order (32-bit tests, as the
    cut is defined)."""
    perm, r_min, r_max, rho, spt, parent, levels = lay
    f32 = np.float32
    R, t, pos = cam.R.astype(f32).reshape(9), cam.t.astype(f32), cam.pos.astype(f32)
    fx, fy, cx, cy = f32(cam.fx), f32(cam.fy), f32(cam.cx), f32(cam.cy)
    k = f32(tau) / fx

    def tests(u):
        m = tree.means[u]
        d = m - pos
        X = np.sqrt((d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2]) * k
        c = [((R[3 * r] * m[:, 0] + R[3 * r + 1] * m[:, 1]) + R[3 * r + 2] * m[:, 2]) + t[r] for r in range(3)]
        culled = c[2] + rho[u] < f32(cam.z_near)
        hl, hr, ht, hb = cx / fx, (f32(cam.width) - cx) / fx, cy / fy, (f32(cam.height) - cy) / fy
        norm = lambda a: np.sqrt(f32(1.0) + a * a)
        culled |= c[0] - hr * c[2] > rho[u] * norm(hr)
        culled |= -c[0] - hl * c[2] > rho[u] * norm(hl)
        culled |= c[1] - hb * c[2] > rho[u] * norm(hb)
        culled |= -c[1] - ht * c[2] > rho[u] * norm(ht)
        return X, culled

    n = tree.n_nodes
    descends, chosen = np.zeros(n, bool), np.zeros(n, bool)
    root_X = np.full(n, np.nan, f32)
    for lev in levels:
        u = lev[(spt[lev] < 0) | (spt[lev] == lev)]
        u = u[(parent[u] < 0) | descends[parent[u]]]
        if not u.size:
            break
        X, culled = tests(u)
        upper = spt[u] < 0
        fine = r_min[u] <= X
        chosen[u[upper & ~culled & fine]] = True
        descends[u[upper & ~culled & ~fine]] = True
        seen = ~upper & ~culled
        root_X[u[seen]] = X[seen]
    X = np.where(spt >= 0, root_X[np.maximum(spt, 0)], np.nan)
    with np.errstate(invalid="ignore"):
        chosen |= (spt >= 0) & (r_max > X) & (r_min <= X)
    return perm[chosen[perm]]


def sh64(deg, d):
    """Real spherical harmonics up to degree 3 at unit directions [n, 3]."""
    x, y, z = d.unbind(1)
    Y = [torch.full_like(x, 0.5 / math.sqrt(math.pi))]
    if deg > 0:
        c = math.sqrt(3.0 / (4.0 * math.pi))
        Y += [-c * y, c * z, -c * x]
    if deg > 1:
        c = math.sqrt(15.0 / (4.0 * math.pi))
        Y += [c * x * y, -c * y * z, math.sqrt(5.0 / (16.0 * math.pi)) * (2 * z * z - x * x - y * y), -c * x * z,
              0.5 * c * (x * x - y * y)]
    if deg > 2:
        a, b, c = math.sqrt(35.0 / (32.0 * math.pi)), math.sqrt(105.0 / (4.0 * math.pi)), math.sqrt(21.0 / (32.0 * math.pi))
        Y += [-a * y * (3 * x * x - y * y), b * x * y * z, -c * y * (4 * z * z - x * x - y * y),
              math.sqrt(7.0 / (16.0 * math.pi)) * z * (2 * z * z - 3 * x * x - 3 * y * y),
              -c * x * (4 * z * z - x * x - y * y), 0.5 * b * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)]
    return torch.stack(Y, 1)


def project64(p, deg, cam):
    """(depth, mean, covariance A B C, opacity, colour) of nodes in 64 bits."""
    dev = p["means"].device
    R = torch.from_numpy(cam.R.astype(np.float64).reshape(3, 3)).to(dev)
    t, pos = (torch.from_numpy(a.astype(np.float64)).to(dev) for a in (cam.t, cam.pos))
    c = p["means"] @ R.T + t
    z = c[:, 2]
    q = p["quats"] / p["quats"].norm(dim=1, keepdim=True)
    w, x, y, zq = q.unbind(1)
    rot = torch.stack([1 - 2 * (y * y + zq * zq), 2 * (x * y - w * zq), 2 * (x * zq + w * y),
                       2 * (x * y + w * zq), 1 - 2 * (x * x + zq * zq), 2 * (y * zq - w * x),
                       2 * (x * zq - w * y), 2 * (y * zq + w * x), 1 - 2 * (x * x + y * y)], 1).reshape(-1, 3, 3)
    M = rot * p["log_scales"].exp()[:, None, :]
    u, v = c[:, 0] / z, c[:, 1] / z
    T0 = (cam.fx / z)[:, None] * (R[0] - u[:, None] * R[2])
    T1 = (cam.fy / z)[:, None] * (R[1] - v[:, None] * R[2])
    M0, M1 = ((M * a[:, :, None]).sum(1) for a in (T0, T1))  # rows of T M
    A, B, C = (M0 * M0).sum(1) + 0.3, (M0 * M1).sum(1), (M1 * M1).sum(1) + 0.3
    d = p["means"] - pos
    Y = sh64(deg, d / d.norm(dim=1, keepdim=True))
    rgb = ((p["sh"] * Y[:, :, None]).sum(1) + 0.5).clamp(min=0.0)
    return z, torch.stack([cam.fx * u + cam.cx, cam.fy * v + cam.cy], 1), A, B, C, p["opacity_logits"].sigmoid(), rgb


def view64(par, deg, cam, target=None, cot=None):
    """Image of the nodes with parameters par (64 bits, blend ties in row
    order) and, given a target of the L1 loss or the image's derivative, that
    derivative and the parameters' gradients."""
    dev, W, H = par["means"].device, cam.width, cam.height
    bg = torch.tensor(BACKGROUND, dtype=torch.float32).double().to(dev)
    with torch.no_grad():
        z, mean, A, B, C, _, _ = project64(par, deg, cam)
        det = A * C - B * B
        mid = 0.5 * (A + C)
        rad = torch.ceil(3.0 * (mid + (mid * mid - det).clamp(min=0.1).sqrt()).sqrt())
        tx, ty = (W + 15) // 16, (H + 15) // 16
        edge = lambda v, hi: torch.floor(v).clamp(0, hi).nan_to_num(0.0).long()
        x0, x1 = edge((mean[:, 0] - rad) / 16, tx), edge((mean[:, 0] + rad) / 16 + 1, tx)
        y0, y1 = edge((mean[:, 1] - rad) / 16, ty), edge((mean[:, 1] + rad) / 16 + 1, ty)
        keep = (z > cam.z_near) & (det > 0) & (x1 > x0) & (y1 > y0)
        at = torch.nonzero(keep).reshape(-1)
        at = at[torch.sort(z[at].float(), stable=True).indices]
        x0, x1, y0, y1 = (v[at] for v in (x0, x1, y0, y1))
        num = (x1 - x0) * (y1 - y0)
        own = torch.repeat_interleave(torch.arange(at.numel(), device=dev), num)
        l = torch.arange(own.numel(), device=dev) - (num.cumsum(0) - num)[own]
        tile = (y0[own] + l // (x1 - x0)[own]) * tx + x0[own] + l % (x1 - x0)[own]
        tile, o = torch.sort(tile, stable=True)
        own = own[o]
        count = torch.bincount(tile, minlength=tx * ty)
        first = count.cumsum(0) - count
    need = target is not None or cot is not None
    drawn = {k: v[at].detach().requires_grad_(need) for k, v in par.items()}
    _, mean, A, B, C, opac, rgb = project64(drawn, deg, cam)
    det = A * C - B * B
    splat = torch.cat([mean, torch.stack([C / det, -B / det, A / det, opac], 1), rgb], 1)
    image = torch.zeros(H, W, 3, dtype=torch.float64, device=dev)
    dimage = torch.zeros_like(image) if need else None
    dsplat = torch.zeros_like(splat)
    with torch.no_grad():
        sp = splat.detach()
        order = torch.sort(count, descending=True).indices
        counts = count[order].cpu().numpy()
        lane = torch.arange(256, device=dev)
        a = 0
        while a < tx * ty:
            k = max(1, int(counts[a]))
            b = min(tx * ty, a + max(1, (1 << 24) // (256 * k)))
            tiles = order[a:b]
            a = b
            px, py = (tiles % tx)[:, None] * 16 + lane % 16, (tiles // tx)[:, None] * 16 + lane // 16
            inside = (px < W) & (py < H)
            slot = torch.arange(k, device=dev)
            valid = slot < count[tiles][:, None]
            who = own[(first[tiles][:, None] + slot).clamp(max=max(0, own.numel() - 1))] if own.numel() else None
            if who is None:
                color, fin = torch.zeros(len(tiles), 256, 3, dtype=torch.float64, device=dev), 1.0
                color = color + bg
            else:
                mx, my, ca, cb, cc, op, cr, cg, cbl = (v[:, None, :] for v in sp[who].unbind(2))
                dx, dy = px[:, :, None] + 0.5 - mx, py[:, :, None] + 0.5 - my
                e = torch.exp(-0.5 * (ca * dx * dx + cc * dy * dy) - cb * dx * dy)
                alpha = (op * e).clamp(max=0.99)
                hit = valid[:, None, :] & (alpha >= 1.0 / 255.0)
                keep_T = torch.where(hit, 1.0 - alpha, 1.0)
                P = keep_T.cumprod(2)
                con = hit & (P >= 1e-4)
                T = P / keep_T
                w = torch.where(con, alpha * T, 0.0)
                fin = torch.where(con, P, 1.0).amin(2)
                color = torch.stack([(w * v).sum(2) for v in (cr, cg, cbl)], 2) + fin[:, :, None] * bg
            image[py[inside], px[inside]] = color[inside]
            if not need or who is None:
                if need:
                    dimage[py[inside], px[inside]] = _dimage(color, target, cot, px, py, inside, W, H)[inside]
                continue
            G = _dimage(color, target, cot, px, py, inside, W, H)
            dimage[py[inside], px[inside]] = G[inside]
            gc = G[:, :, 0:1] * cr + G[:, :, 1:2] * cg + G[:, :, 2:3] * cbl
            behind = (w * gc).sum(2, keepdim=True) + (fin * (G @ bg))[:, :, None] - (w * gc).cumsum(2)
            dalpha = torch.where(con, T * gc - behind / (1.0 - alpha), 0.0)
            dalpha = torch.where(op * e <= 0.99, dalpha, 0.0)
            dpow = dalpha * alpha
            sx, sy = (dpow * dx).sum(1), (dpow * dy).sum(1)
            parts = [ca[:, 0] * sx + cb[:, 0] * sy, cb[:, 0] * sx + cc[:, 0] * sy, -0.5 * (dpow * dx * dx).sum(1),
                     -(dpow * dx * dy).sum(1), -0.5 * (dpow * dy * dy).sum(1), (dalpha * e).sum(1)]
            parts += [(w * G[:, :, c:c + 1]).sum(1) for c in range(3)]
            dsplat.index_add_(0, who[valid], torch.stack(parts, 2)[valid])
    if not need:
        return image, None, None
    got = torch.autograd.grad(splat, [drawn[k] for k in GROUPS], dsplat)
    grads = {k: torch.zeros_like(par[k]).index_copy_(0, at, g) for k, g in zip(GROUPS, got)}
    return image, dimage, grads


def _dimage(color, target, cot, px, py, inside, W, H):
    x, y = px.clamp(max=W - 1), py.clamp(max=H - 1)
    g = cot[y, x] if cot is not None else torch.sign(color - target[y, x]) / (3.0 * W * H)
    return torch.where(inside[:, :, None], g, 0.0)


def exact(case, seed):
    device = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    tree = make_tree(case, seed)
    cams = make_cameras(case, seed + 1)
    lay = layout64(tree)
    perm, n, kind = lay[0], tree.n_nodes, case["kind"]
    place = np.empty(n, np.int64)
    place[perm] = np.arange(n)
    nodes = {"means": tree.means, "log_scales": tree.log_scales, "quats": tree.quats,
             "opacity_logits": tree.opacity_logits, "sh": tree.sh.reshape(n, -1, 3)}
    images = None if kind in ("forward", "graph") else make_images(case, seed + 2, device).double()
    dense = lambda rows=n: {k: torch.zeros((rows,) + v.shape[1:], dtype=torch.float64, device=device)
                            for k, v in nodes.items()}
    total, losses = dense() if kind in ("autograd", "step", "batch") else None, []
    for b, cam in enumerate(cams):
        ids = cut64(tree, lay, cam, case["tau"])
        par = {k: torch.from_numpy(v[ids]).to(device).double() for k, v in nodes.items()}
        img = None if images is None else images[b]
        auto = kind == "autograd"
        image, dL, grads = view64(par, case["degree"], cam, None if auto else img, img if auto else None)
        at = torch.from_numpy(place[ids]).to(device)
        if total is not None:
            for k in GROUPS:
                total[k].index_add_(0, at, grads[k])
            losses.append((image - images[b]).abs().mean())
    if kind in ("forward", "graph"):
        return {"idx": None, "count": None, "image": image}
    if kind == "autograd":
        return {"image": image, "grads": total}
    if kind == "batch":
        return {"losses": torch.stack(losses), "grads": total}
    if kind == "step":
        return {"image": image, "dL": dL, "grads": total}
    if kind == "pooled":
        sel = dense()
        for k in GROUPS:
            sel[k][:len(ids)] = grads[k]
        return {"idx": None, "count": None, "image": image, "dL": dL, "grads": sel}
    params = {k: torch.from_numpy(np.take(v, perm, axis=0)).to(device).double() for k, v in nodes.items()}
    m, v = dense(), dense()
    for k in GROUPS:
        g = grads[k]
        m[k][at], v[k][at] = 0.1 * g, 0.001 * g * g
        params[k][at] -= ADAM_LR[k] * g / (g.abs() + 1e-15)
    return {"image": image, "params": params, "exp_avg": m, "exp_avg_sq": v}
