"""The adjoint with a guide against the float64 oracle where the other guided parity tests
do not go: Russian roulette from the first vertex (whose factor is formed anew, the later
ones' come from the records), from the second one, and sampling parameters of their own
(the roulette sees the weights at these).  Paths whose events agree and whose gradient is
well conditioned; gradients at 1e-3 of max(|g|, 1e-2 rms g), the bar of the other gradient
parity tests."""
import math

import numpy as np
import pytest

import _guide
from _gpu import banner, both, check_mismatches, gpu_grad, gpu_render, mask_report, oracle_opts
from paper_1903_07145_amd import ipt, scenes

pytestmark = pytest.mark.gpu

GRAD_REL = 1e-3


@pytest.fixture(scope="module")
def room():
    sc = scenes.room()
    g, o = both(sc)
    return sc, g, o, ipt.make_cameras(sc["cams"])


@pytest.mark.parametrize("cached", [0, 1])
@pytest.mark.parametrize("rr,own_sampling", [(0, False), (1, False), (2, False), (-1, True), (1, True), (2, True)])
def test_guided_gradient(room, rr, own_sampling, cached):
    label = "guided gradient, roulette from %d, own sampling parameters %d, cached %d" % (rr, own_sampling, cached)
    banner(label)
    sc, g, o, dc = room
    lo, inv = _guide.box(sc["verts"])
    w = _guide.random_weights(sc["num_segments"], seed=22, out_gain=3.0, kappa_bias=1.0)
    gd = ipt.Guide(g)
    gd.set_weights(w)
    okw = dict(guide_w=w, guide_mix=0.5, bb_lo=lo, bb_inv=inv)
    if cached:
        okw["guide_cell_area"] = 0.05
        gd.cache_build(0.05, mode=1)
    n = dc["num_views"] * dc["width"] * dc["height"]
    pix = np.sort(np.random.default_rng(3).choice(n, size=800, replace=False)).astype(np.int64)
    kw = dict(seed=47, stream_tag=2, iteration=1, spp=4, max_depth=4, rr_depth=rr, mis=2)
    gkw = dict(kw, guide=gd, guide_mix=0.5, guide_cached=cached, guide_fp32=1 - cached)
    sp = scenes.init_theta(sc, "uniform", seed=4) if own_sampling else None
    wt = np.random.default_rng(7).normal(size=(pix.size, 3))
    _, h = gpu_render(g, dc, sc["params"], gkw, pixel_list=pix, sampling_params=sp)
    r = o.run(sc["cams"], sc["params"], sampling_params=sp, pixel_list=pix, w=wt, want_hash=True, want_margin=True,
              want_cond=True, **oracle_opts(kw), **okw)
    check_mismatches(h, r, 3, label=label, depth=kw["max_depth"])
    m = mask_report(h, r, gcond=r["gcond"], label=label)["tight_g"]
    assert m.mean() > 0.7
    got = gpu_grad(g, dc, sc["params"], wt, gkw, pixel_list=pix, mask=m, sampling_params=sp)
    want = o.run(sc["cams"], sc["params"], sampling_params=sp, pixel_list=pix, w=wt, path_mask=m.astype(np.uint8),
                 want_grad=True, **oracle_opts(kw), **okw)["grad"]
    rms = math.sqrt(np.mean(want ** 2))
    err = np.abs(got - want) / np.maximum(np.abs(want), 1e-2 * rms)
    print("gradient over %d paths: rel err p50 %.2e max %.2e" % (m.sum(), np.median(err), err.max()))
    assert err.max() <= GRAD_REL
