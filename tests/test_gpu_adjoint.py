"""The adjoint with a guide, a vertex per lane: one path to several chunks of
paths, one vertex to the longest paths, roulette at the first vertex, other
sampling parameters, masks, the smallest workspace, against the sum of calls for
every fifth pixel, whose tiles hold other paths: the same float32 vertices in other
float64 sums, each rounded to float32 once (1e-6 of the norm)."""
import numpy as np
import pytest
import torch

from _gpu import banner
from paper_1903_07145_amd import ipt, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,spp,depth,rr,small", [
    (1, 1, 1, 1, -1, False), (1, 1, 3, 16, -1, True), (9, 7, 1, 1, 1, False), (13, 5, 1, 16, 1, False),
    (64, 3, 4, 3, 2, True), (3, 1, 512, 5, -1, False), (61, 43, 5, 16, -1, False), (90, 71, 2, 6, 3, True)])
def test_adjoint_edges(w, h, spp, depth, rr, small):
    banner("adjoint %d x %d, %d spp, depth %d, rr %d, small %d" % (w, h, spp, depth, rr, small))
    sc = scenes.cornell()
    g = ipt.Scene.from_dict(sc)
    c = sc["cams"]
    dc = ipt.make_cameras(dict(cam_to_world=c["cam_to_world"][:1], fov_y=c["fov_y"][:1], width=w, height=h))
    p = torch.as_tensor(sc["params"], device="cuda")
    q = torch.as_tensor(scenes.init_theta(sc, "uniform", seed=4), device="cuda")
    gd = ipt.Guide(g, seed=2, batch=64, ring_capacity=1 << 16)
    gd.cache_build(1e-2)
    kw = dict(seed=8, spp=spp, max_depth=depth, rr_depth=rr, mis=2, guide=gd, guide_mix=0.5, guide_cached=1)
    n = w * h
    wt = torch.randn((n, 3), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    mask = torch.as_tensor((np.random.default_rng(5).random((n, spp)) < 0.7).astype(np.uint8), device="cuda")

    def grad(sampling, m, pix=None):
        sel = slice(None) if pix is None else pix
        o = ipt.render_opts(path_mask=None if m is None else m[sel].reshape(-1).contiguous(), pixel_list=pix, **kw)
        nb = g.workspace_query(dc, o)[0] if small else None
        return g.render_grad(dc, p, wt[sel].contiguous(), o, sampling_params=sampling, workspace_bytes=nb).double()

    for sampling, m in ((None, None), (q, None), (None, mask)):
        a = grad(sampling, m)
        assert torch.isfinite(a).all()
        parts = sum(grad(sampling, m, torch.arange(i, n, 5, device="cuda")) for i in range(min(5, n)))
        assert (a - parts).norm() <= 1e-6 * a.norm()
