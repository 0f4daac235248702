"""The workloads whose speed this repository tracks, each one pass through the public entry points.

A case is a dict of plain values; "op" says which entry points it goes through:

* step       one SGD iteration (ipt_loss_grad, with the L1 regulariser where it is used, and ipt_sgd_step): what
             `optimize` repeats hundreds of times.  With a guide, also the refill of the cached proposal.
* render     the colour estimate alone (ipt_render, or ipt_render_static for callers without a workspace): target
             images and previews.
* autograd   the differentiable image and its vector-Jacobian product (`ipt.render` under torch.autograd).
* rays       a batch of closest-hit queries (ipt_trace_rays): coverage and the pixels' triangles.
* build      a scene from host arrays (BVH and layouts) and a few first queries on it.
* guide_grad one training batch of the learned proposal (ipt_guide_loss_grad).
* guide_eval a batch of its mixtures (ipt_guide_eval).

Scenes are the repository's own workloads at their own sizes, cut to fewer or resized views where a case says so.
"""
import functools
import math

import numpy as np
import torch

from paper_1903_07145_amd import ipt, scenes

GUIDE_CELLS = {"cornell": 20000, "room": 200000, "apartment": 1180000}
TRIANGLES = {"cornell": 36, "room": 49284, "apartment": 500582, "office_floor": 2001228}
VIEWS = {"cornell": 1, "room": 4, "apartment": 16, "office_floor": 30}
ADAM = dict(lr=1e-2, beta1=0.9, beta2=0.999, eps=1e-8)


def _step(name, scene, views, width, height, spp, depth, rr, mis=2, material="ggx", guide="none", pixels=0, grad_spp=0,
          loss=0, emissive=False):
    c = dict(op="step", scene=scene, views=views, width=width, height=height, spp=spp, depth=depth, rr=rr, mis=mis,
             material=material, guide=guide, pixels=pixels, grad_spp=grad_spp or spp, loss=loss, emissive=emissive)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest scene at its own size: 16 thousand paths, where latency and launches count
        _step("step_cornell", "cornell", 1, 64, 64, 4, 3, -1),
        # the paper's own optimisation setting: a few pixels, many colour paths, one gradient path, every segment
        # of the apartment an emitter, L1 loss and regulariser
        _step("step_pixel_batch", "apartment", 16, 640, 480, 512, 7, 3, pixels=8, grad_spp=1, loss=1, emissive=True),
        # one room at its own size: the middle of the range
        _step("step_room", "room", 4, 320, 240, 16, 5, -1),
        # the benchmark's default workload
        _step("step_apartment", "apartment", 16, 640, 480, 8, 7, 3),
        # the Disney material model, half of the apartment's views
        _step("step_apartment_disney", "apartment", 8, 640, 480, 4, 7, 3, material="disney"),
        # the learned proposal from its cached rows, refilled each iteration
        _step("step_room_guided", "room", 4, 320, 240, 8, 5, -1, guide="cached"),
        # target images of the largest scene: every view, a few samples per pass
        dict(name="render_office_floor", op="render", scene="office_floor", views=30, width=640, height=480, spp=2,
             depth=8, rr=3, mis=2, static=False, profile=0),
        # a preview without a workspace: odd sizes, the power heuristic and the cosine emission profile
        dict(name="render_static_odd", op="render", scene="apartment", views=1, width=333, height=251, spp=5, depth=6,
             rr=2, mis=3, static=True, profile=1),
        # forward and backward through torch.autograd on an odd image, light sampling only
        dict(name="autograd_room_odd", op="autograd", scene="room", views=2, width=211, height=157, spp=6, depth=4,
             rr=-1, mis=1),
        # coverage: one query per pixel of every view
        dict(name="rays_apartment", op="rays", scene="apartment", n=4915200),
        # a new scene, as each refinement round makes one
        dict(name="build_room", op="build", scene="room", n=4099),
        # a training batch of the proposal at the optimiser's size
        dict(name="guide_grad_16384", op="guide_grad", n=16384, segments=128),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["step", "step", "step", "render", "autograd", "rays", "build", "guide_grad", "guide_eval"])
    if op == "guide_grad":
        return dict(op=op, n=_log(rng, 1000, 100000), segments=rng.choice([8, 32, 128, 256]))
    if op == "guide_eval":
        return dict(op=op, n=_log(rng, 1000, 2000000), segments=rng.choice([8, 32, 128, 256]), mode=0)
    scene = rng.choice(["cornell", "room", "apartment"])
    if op == "rays":
        return dict(op=op, scene=scene, n=_log(rng, 1000, 4900000))
    if op == "build":
        return dict(op=op, scene=scene, n=_log(rng, 1000, 5000))
    views = rng.randint(1, VIEWS[scene])
    paths = _log(rng, 10000, 12000000)
    spp = min(64, _log(rng, 1, 32))
    width = max(16, min(1024, int(math.sqrt(paths / spp / views * rng.uniform(0.8, 1.6)))))
    height = max(16, min(1024, int(paths / spp / views / width)))
    depth, rr, mis = rng.randint(2, 8), rng.choice([-1, 2, 3]), rng.choice([0, 2, 2, 2, 3])
    if op == "render":
        return dict(op=op, scene=scene, views=views, width=width, height=height, spp=spp, depth=depth, rr=rr, mis=mis,
                    static=False, profile=rng.randint(0, 1))
    if op == "autograd":
        return dict(op=op, scene=scene, views=views, width=width, height=height, spp=spp, depth=depth, rr=rr, mis=mis)
    kind = rng.choice(["plain", "plain", "plain", "disney", "cached", "pixels"])
    if kind == "pixels":
        n = _log(rng, 8, 512)
        return _step(None, scene, views, 320, 240, _log(rng, 8, 1024), depth, rr, pixels=n, grad_spp=rng.randint(1, 64),
                     loss=1, emissive=bool(rng.randint(0, 1)))
    return _step(None, scene, views, width, height, spp, depth, rr, mis=mis,
                 material="disney" if kind == "disney" else "ggx", guide="cached" if kind == "cached" else "none")


@functools.lru_cache(maxsize=None)
def _scene(name, material="ggx", emissive=False):
    """The workload's host arrays (geometry, true parameters, ranges)."""
    sc = scenes.WORKLOADS[name]()
    if material == "disney":
        sc = scenes.disney(sc, seed=11)
    return scenes.all_emissive(sc) if emissive else sc


def _cams(sc, views, width, height):
    c = sc["cams"]
    return dict(cam_to_world=c["cam_to_world"][:views], fov_y=c["fov_y"][:views], width=width, height=height)


def _dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), device="cuda")


def _rays(sc, n, seed):
    """Rays through random points of random views' images."""
    g = np.random.default_rng(seed)
    c = sc["cams"]
    c2w = np.asarray(c["cam_to_world"], np.float64)
    v = np.sort(g.integers(0, c2w.shape[0], n))
    t = np.tan(0.5 * np.asarray(c["fov_y"], np.float64))[v]
    d = np.stack([(2 * g.random(n) - 1) * t * c["width"] / c["height"], (2 * g.random(n) - 1) * t, -np.ones(n)], 1)
    d = np.einsum("nij,nj->ni", c2w[v, :3, :3], d)
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    return c2w[v, :3, 3].astype(np.float32), d.astype(np.float32)


def _guide_weights(segments, seed):
    """Weights of a proposal after some training: He-normal layers, lobes of moderate width."""
    g = np.random.default_rng(seed)
    parts = []
    for fan_in, fan_out, gain in ((25, 64, 1.0), (64, 64, 1.0), (64, 64, 1.0), (64, 64, 1.0), (64, 40, 2.0)):
        parts += [g.normal(0, gain * np.sqrt(2.0 / fan_in), fan_in * fan_out), g.normal(0, 0.05, fan_out)]
    return np.concatenate(parts + [g.normal(0, 0.3, 16 * segments)]).astype(np.float32)


def _unit(g, n):
    v = g.normal(size=(n, 3))
    return v / np.linalg.norm(v, axis=1, keepdims=True)


def _records(n, segments, seed):
    """Training records in the ring's layout: features, segment, direction, weight."""
    g = np.random.default_rng(seed)
    r = np.zeros((n, 16), np.float32)
    r[:, 0:3] = g.uniform(-1, 1, (n, 3))
    r[:, 3] = g.integers(0, segments, n).astype(np.int32).view(np.float32)
    r[:, 4:7] = _unit(g, n)
    r[:, 7] = g.uniform(0.1, 2.0, n)
    r[:, 8:11] = _unit(g, n)
    r[:, 12:15] = _unit(g, n)
    return r


def _bare_guide(case, seed):
    """A proposal on a scene with the case's number of segments."""
    s = case["segments"]
    v, f = scenes.random_soup(max(64, s), seed=1)
    g = ipt.Scene(v, f, np.arange(len(f), dtype=np.int32) % s, s, np.zeros(0, np.int32))
    gd = ipt.Guide(g, seed=1, batch=16384, ring_capacity=1 << 15)
    gd.set_weights(_guide_weights(s, seed))
    return gd


def prepare(case, seed):
    op = case["op"]
    if op == "guide_grad":
        return dict(op=op, guide=_bare_guide(case, seed), rec=_dev(_records(case["n"], case["segments"], seed)))
    if op == "guide_eval":
        r = _records(case["n"], case["segments"], seed)
        return dict(op=op, guide=_bare_guide(case, seed), mode=case["mode"],
                    feat=_dev(np.concatenate([r[:, 0:3], r[:, 4:7], r[:, 8:11]], 1)),
                    seg=_dev(r[:, 3].copy().view(np.int32)))
    sc = _scene(case["scene"], case.get("material", "ggx"), case.get("emissive", False))
    if op in ("rays", "build"):
        o, d = _rays(sc, case["n"], seed)
        s = dict(op=op, o=_dev(o), d=_dev(d), sc=sc)
        if op == "rays":
            s["scene"] = ipt.Scene.from_dict(sc)
        return s
    g = ipt.Scene.from_dict(sc)
    dc = ipt.make_cameras(_cams(sc, case["views"], case["width"], case["height"]))
    npix = case["views"] * case["width"] * case["height"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    params = _dev(scenes.init_theta(sc, "uniform", seed=seed))
    kw = dict(seed=seed, iteration=3, max_depth=case["depth"], rr_depth=case["rr"], mis=case["mis"],
              emission_profile=case.get("profile", 0))
    s = dict(op=op, scene=g, dc=dc, params=params)
    if op == "render":
        s["opts"] = ipt.render_opts(stream_tag=1, spp=case["spp"], **kw)
        s["static"] = case["static"]
    elif op == "autograd":
        s["params"] = params.requires_grad_()
        s["color"] = ipt.render_opts(stream_tag=1, spp=case["spp"], **kw)
        s["grad"] = ipt.render_opts(stream_tag=2, spp=case["spp"], **kw)
        s["w"] = torch.randn((npix, 3), generator=gen, device="cuda") / npix
    else:
        pix = torch.randint(0, npix, (case["pixels"],), generator=gen, device="cuda") if case["pixels"] else None
        n = case["pixels"] or npix
        # target: the true parameters' image, a few samples per pixel
        s["target"] = g.render(dc, _dev(sc["params"]), ipt.render_opts(
            stream_tag=0, spp=4, pixel_list=pix, **dict(kw, seed=seed + 1)))
        if case["guide"] == "cached":
            gd = ipt.Guide(g, seed=7, batch=16384, ring_capacity=1 << 21,
                           record_stride=max(1, (n * case["spp"] * 3) // (1 << 20)))
            gd.set_weights(_guide_weights(g.num_segments, seed))
            v, f = sc["verts"][sc["tris"]].astype(np.float64), GUIDE_CELLS[case["scene"]]
            area = 0.5 * np.linalg.norm(np.cross(v[:, 1] - v[:, 0], v[:, 2] - v[:, 0]), axis=1)
            gd.cache_build(float(area.sum() / f))
            kw.update(guide=gd, guide_mix=0.5, guide_cached=1)
            s["guide"] = gd
        s["color"] = ipt.render_opts(stream_tag=1, spp=case["spp"], pixel_list=pix, **kw)
        s["grad"] = ipt.render_opts(stream_tag=2, spp=case["grad_spp"], pixel_list=pix, **kw)
        s["loss_kind"] = case["loss"]
        s["scale"], s["lo"], s["hi"] = _dev(sc["scale"]), _dev(sc["lo"]), _dev(sc["hi"])
        s["trainable"] = _dev(sc["trainable"])
        if case["emissive"]:
            w = np.zeros(g.P, np.float32)
            w[7 * g.num_segments:] = 1e-3 / sc["scale"][7 * g.num_segments:]
            s["l1"] = _dev(w)
        # parameters and Adam moments in the middle of a run; a pass steps a copy of them
        s["start"] = torch.stack([params, 1e-3 * torch.randn(g.P, generator=gen, device="cuda"),
                                  1e-4 * torch.rand(g.P, generator=gen, device="cuda") + 1e-5])
        s["at"] = torch.empty_like(s["start"])
        s["image"] = torch.empty((n, 3), device="cuda")
        # the workspace of a run is sized once, for the pass that needs most
        for o in (s["color"], s["grad"]):
            g.workspace(dc, o)
    return s


def run(s):
    op = s["op"]
    if op == "guide_grad":
        loss, grad = s["guide"].loss_grad(s["rec"])
        return dict(loss=loss, grad=grad)
    if op == "guide_eval":
        return s["guide"].eval(s["feat"], s["seg"], mode=s["mode"])
    if op in ("rays", "build"):
        g = s["scene"] if op == "rays" else ipt.Scene.from_dict(s["sc"])
        tri, tuv = g.trace_rays(s["o"], s["d"])
        if op == "build":
            s["scene"] = g   # the queries run on it after the call returns
        return dict(tri=tri, tuv=tuv)
    g, dc = s["scene"], s["dc"]
    if op == "render":
        return (g.render_static if s["static"] else g.render)(dc, s["params"], s["opts"])
    if op == "autograd":
        img = ipt.render(g, dc, s["params"], s["color"], s["grad"])
        return dict(image=img.detach(), grad=torch.autograd.grad(img, s["params"], s["w"])[0])
    if "guide" in s:
        s["guide"].cache_build(s["guide"].cell_area)
    at = s["at"].copy_(s["start"])
    loss, grad = g.loss_grad(dc, at[0], s["target"], s["color"], s["grad"], s["loss_kind"], image=s["image"])
    if "l1" in s:
        ipt.l1_reg(at[0], grad, s["l1"], loss)
    ipt.sgd_step(at[0], grad, at[1], at[2], 10, scale=s["scale"], lo=s["lo"], hi=s["hi"], trainable=s["trainable"],
                 **ADAM)
    return dict(loss=loss, grad=grad, image=s["image"], params=at[0], m=at[1], v=at[2])


def work(case):
    """Inputs and outputs once; per ray one descent of a four-way tree (a visit tests four boxes, about 60 operations)
    and two triangle tests; per path vertex about 300 operations of shading.  About half of a path's vertices are
    reached, each with a light sample's ray and a continuation."""
    op = case["op"]
    if op in ("guide_grad", "guide_eval"):
        n, net = case["n"], 2 * (25 * 64 + 3 * 64 * 64 + 64 * 40)
        params = 4 * (16744 + 16 * case["segments"])
        if op == "guide_grad":
            return {"bytes": 64 * n + 2 * params, "flops": 3 * net * n}
        return {"bytes": (36 + 4 + 160) * n + params, "flops": net * n}
    tris = TRIANGLES[case["scene"]]
    ray = (math.log(tris, 4) + 2) * 60 + 2 * 60
    if op in ("rays", "build"):
        n = case["n"]
        build = tris * math.log2(tris) * 60 if op == "build" else 0.0
        return {"bytes": 48 * tris * (3 if op == "build" else 1) + (24 + 16) * n, "flops": ray * n + build}
    pix = case.get("pixels") or case["views"] * case["width"] * case["height"]
    colour = pix * case["spp"]
    grad = pix * case.get("grad_spp", case["spp"]) if op != "render" else 0
    per_path = 0.5 * (case["depth"] + 1) * (2 * ray + 300)
    return {"bytes": 48 * tris + 12 * pix * (1 if op == "render" else 3), "flops": (colour + 1.3 * grad) * per_path}


def _exact_hits(sc, o, d):
    """Nearest triangle of every ray by testing all of them (Moeller and Trumbore) in 64 bits."""
    v = torch.as_tensor(sc["verts"][sc["tris"]], device="cuda", dtype=torch.float64)
    o, d = (torch.as_tensor(x, device="cuda", dtype=torch.float64) for x in (o, d))
    e1, e2 = v[:, 1] - v[:, 0], v[:, 2] - v[:, 0]
    best = torch.full((len(o),), math.inf, device="cuda", dtype=torch.float64)
    uv = torch.zeros((len(o), 2), device="cuda", dtype=torch.float64)
    for a in range(0, len(v), 4096):
        for b in range(0, len(o), 4096):
            E1, E2, D = e1[None, a:a + 4096], e2[None, a:a + 4096], d[b:b + 4096, None]
            p = torch.linalg.cross(D.expand(-1, E2.shape[1], -1), E2.expand(D.shape[0], -1, -1))
            det = (p * E1).sum(-1)
            s = o[b:b + 4096, None] - v[None, a:a + 4096, 0]
            u = (p * s).sum(-1) / det
            q = torch.linalg.cross(s, E1.expand(D.shape[0], -1, -1))
            w = (q * D).sum(-1) / det
            t = (q * E2).sum(-1) / det
            t = torch.where((u >= 0) & (w >= 0) & (u + w <= 1) & (t > 0), t, math.inf)
            near, at = t.min(1)
            closer = near < best[b:b + 4096]
            pick = torch.stack([u.gather(1, at[:, None])[:, 0], w.gather(1, at[:, None])[:, 0]], 1)
            uv[b:b + 4096] = torch.where(closer[:, None], pick, uv[b:b + 4096])
            best[b:b + 4096] = torch.where(closer, near, best[b:b + 4096])
    return torch.where(best.isfinite()[:, None], torch.cat([best[:, None], uv], 1), 0.0)


def _exact_mixture(w, feat, seg):
    """Network and mixture (mu, kappa, weight per lobe) of the proposal in 64 bits."""
    off, layers = 0, []
    for i, j in ((25, 64), (64, 64), (64, 64), (64, 64), (64, 40)):
        layers.append((w[off:off + i * j].reshape(i, j), w[off + i * j:off + i * j + j]))
        off += i * j + j
    x = torch.cat([feat, w[off:].reshape(-1, 16)[seg]], 1)
    for k, (m, b) in enumerate(layers):
        x = x @ m + b
        x = x.relu() if k < 4 else x
    y = x.reshape(-1, 8, 5)
    kappa = (torch.nn.functional.softplus(y[..., 3]) + 0.01).clamp(max=1e4)
    return y[..., :3] / y[..., :3].norm(dim=-1, keepdim=True), kappa, torch.softmax(y[..., 4], -1)


def exact(case, seed):
    """In 64 bits: hits of the ray batches that all triangles can be tested for, and the proposal's outputs, loss and
    gradient.  The Monte Carlo estimates have none: a path in 64 bits takes another turn wherever two events are
    nearly tied, and is another sample from there on."""
    op = case["op"]
    if op in ("guide_grad", "guide_eval"):
        s = case["segments"]
        w = torch.as_tensor(_guide_weights(s, seed), device="cuda", dtype=torch.float64).requires_grad_()
        rec = _records(case["n"], s, seed)
        seg = torch.as_tensor(rec[:, 3].copy().view(np.int32), device="cuda").long()
        r = torch.as_tensor(rec, device="cuda", dtype=torch.float64)
        feat = torch.cat([r[:, 0:3], r[:, 4:7], r[:, 8:11]], 1)
        if op == "guide_eval":
            with torch.no_grad():
                mu, kappa, weight = _exact_mixture(w, feat, seg)
                return torch.cat([mu, kappa[..., None], weight[..., None]], -1).reshape(-1, 40)
        mu, kappa, weight = _exact_mixture(w, feat, seg)
        c = (mu * r[:, None, 12:15]).sum(-1)
        lp = kappa.log() - math.log(2 * math.pi) - (-torch.expm1(-2 * kappa)).log() + kappa * (c - 1)
        loss = -(r[:, 7] * (weight * lp.exp()).sum(-1).log()).sum() / r[:, 7].sum()
        return dict(loss=loss.detach().reshape(1), grad=torch.autograd.grad(loss, w)[0])
    if op in ("rays", "build") and case["n"] * TRIANGLES[case["scene"]] <= 1 << 31:
        sc = _scene(case["scene"])
        return dict(tri=None, tuv=_exact_hits(sc, *_rays(sc, case["n"], seed)))
    return None
