"""Path streams against the per-lane state machine: a pass that asks for path
hashes runs as the state machine, the same pass without them as streams.  Both
do the same arithmetic, so images agree bit for bit and gradients up to the
order of their float64 sums (1e-6 of the norm).  Sizes at the edges of the
streams' tiles (256 paths) and groups (8 tiles), a pixel list with invalid
entries, and a scratch that forces several batches."""
import ctypes

import numpy as np
import pytest
import torch

from _gpu import banner
from paper_1903_07145_amd import ipt, scenes

pytestmark = pytest.mark.gpu


def _scene(name, material, storage=ipt.PARAMS_AUTO):
    sc = getattr(scenes, name)()
    if material == "disney":
        sc = scenes.disney(sc, seed=3)
    return sc, ipt.Scene.from_dict(sc, param_storage=storage)


def _cams(sc, w, h):
    c = sc["cams"]
    return ipt.make_cameras(dict(cam_to_world=c["cam_to_world"][:1], fov_y=c["fov_y"][:1], width=w, height=h))


def _both(g, dc, p, kw, pix=None, sampling=None):
    """(image, gradient) as streams and as the state machine."""
    n = (dc["width"] * dc["height"] if pix is None else pix.numel())
    w = torch.randn((n, 3), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    out = []
    for machine in (False, True):
        h = torch.zeros(n * kw["spp"], dtype=torch.int64, device="cuda") if machine else None
        o = ipt.render_opts(pixel_list=pix, debug_path_hash=h, **kw)
        out.append((g.render(dc, p, o, sampling_params=sampling), g.render_grad(dc, p, w, o, sampling_params=sampling)))
    torch.cuda.synchronize()
    assert h.ne(0).any()
    return out


def _check(a, b):
    assert torch.equal(a[0].view(torch.int32), b[0].view(torch.int32))
    ga, gb = a[1].double(), b[1].double()
    assert (ga - gb).norm() <= 1e-6 * gb.norm() + 1e-30


@pytest.mark.parametrize("w,h,spp", [(1, 1, 1), (5, 51, 1), (16, 16, 1), (257, 1, 1), (64, 32, 1), (23, 89, 1),
                                     (61, 67, 5)])
def test_sizes_at_tile_and_group_edges(w, h, spp):
    banner("streams against the state machine: %d x %d pixels, %d spp" % (w, h, spp))
    sc, g = _scene("cornell", "ggx")
    p = torch.as_tensor(sc["params"], device="cuda")
    _check(*_both(g, _cams(sc, w, h), p, dict(seed=9, spp=spp, max_depth=4, mis=2)))


@pytest.mark.parametrize("material", ["ggx", "disney"])
@pytest.mark.parametrize("storage", [ipt.PARAMS_AUTO, ipt.PARAMS_GLOBAL])
@pytest.mark.parametrize("guided", [False, True])
def test_kernel_variants(material, storage, guided):
    banner("streams against the state machine: %s, storage %d, cached proposal %d" % (material, storage, guided))
    sc, g = _scene("room", material, storage)
    dc = _cams(sc, 90, 61)
    p = torch.as_tensor(scenes.init_theta(sc, "uniform", seed=3), device="cuda")
    q = torch.as_tensor(scenes.init_theta(sc, "uniform", seed=4), device="cuda")
    kw = dict(seed=4, spp=3)
    if guided:
        gd = ipt.Guide(g, seed=2, batch=64, ring_capacity=1 << 16)
        gd.cache_build(1e-2)
        kw.update(guide=gd, guide_mix=0.5, guide_cached=1)
    for mis, rr, prof, depth, sp in ((2, 2, 0, 5, None), (3, -1, 1, 16, None), (0, 1, 0, 1, q), (1, -1, 1, 3, q)):
        _check(*_both(g, dc, p, dict(kw, mis=mis, rr_depth=rr, emission_profile=prof, max_depth=depth), sampling=sp))


def test_pixel_list_with_invalid_entries():
    banner("streams against the state machine: pixel list with invalid entries")
    sc, g = _scene("room", "ggx")
    dc = _cams(sc, 64, 48)
    rng = np.random.default_rng(2)
    pix = rng.integers(0, 64 * 48, 700)
    pix[::7] = -1
    pix[3::50] = 64 * 48
    pix = torch.as_tensor(pix, device="cuda")
    p = torch.as_tensor(sc["params"], device="cuda")
    a, b = _both(g, dc, p, dict(seed=4, spp=9, max_depth=4, mis=2), pix=pix)
    _check(a, b)
    assert (a[0][::7] == 0).all()


def test_scratch_for_several_batches():
    banner("streams in several batches")
    sc, g = _scene("cornell", "ggx")
    dc = _cams(sc, 700, 411)
    p = torch.as_tensor(sc["params"], device="cuda")
    o = ipt.render_opts(seed=5, spp=9, max_depth=3, mis=2)   # 2.6 M paths
    whole = g.render(dc, p, o)
    mn, full = g.workspace_query(dc, o)
    paths = 700 * 411 * 9
    # all but the scratch of 1.5 M paths (224 B each) and of the checkpoints
    need = full - (paths - 1500000) * 224 - paths * 4 * 48
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    img = torch.empty_like(whole)
    C = ipt._cams_struct(dc)
    ipt._check(ipt.lib().ipt_render(g.handle, ctypes.byref(C), ipt._ptr(p), None, ctypes.byref(o), ipt._ptr(img),
                                    ipt._ptr(ws), need, ipt._stream()))
    assert torch.equal(whole, img)
    w = torch.randn_like(whole)
    grad = g.render_grad(dc, p, w, o)
    half = g.render_grad(dc, p, w, o, workspace_bytes=mn + (full - mn) // 2)   # checkpoints in chunks
    assert (grad.double() - half.double()).norm() <= 1e-6 * grad.double().norm()
