"""Passes of one path run as the state machine, larger ones as streams: the same image
bit for bit, and gradients up to the order of their float64 sums (1e-6 of the norm), on
both sides of the line.  The kernels' own ray counter tells which ran: for a pixel that
does not exist the state machine traces nothing, streams a placeholder."""
import pytest
import torch

from _gpu import banner
from paper_1903_07145_amd import ipt, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pixels,spp", [([1290], 1), ([1290], 2), ([1290, 2100], 1), ([-1], 1), ([-1, 1290], 1)])
def test_few_paths(pixels, spp):
    banner("few paths: pixels %s, %d spp" % (pixels, spp))
    sc = scenes.cornell()
    g = ipt.Scene.from_dict(sc)
    dc = ipt.make_cameras(sc["cams"])
    p = torch.as_tensor(sc["params"], device="cuda")
    pix = torch.tensor(pixels, device="cuda")
    w = torch.randn((len(pixels), 3), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    out = []
    for machine in (False, True):
        h = torch.zeros(len(pixels) * spp, dtype=torch.int64, device="cuda") if machine else None
        o = ipt.render_opts(seed=9, spp=spp, max_depth=6, pixel_list=pix, debug_path_hash=h)
        out.append((g.render(dc, p, o), g.render_static(dc, p, o), g.render_grad(dc, p, w, o)))
    a, b = out
    for x, y in zip(a[:2], b[:2]):
        assert torch.equal(x.view(torch.int32), y.view(torch.int32))
    assert (a[2].double() - b[2].double()).norm() <= 1e-6 * b[2].double().norm()


def test_one_path_runs_as_the_state_machine():
    banner("one path, a pixel that does not exist")
    sc = scenes.cornell()
    g = ipt.Scene.from_dict(sc)
    dc = ipt.make_cameras(sc["cams"])
    p = torch.as_tensor(sc["params"], device="cuda")
    rays = []
    for n in (1, 2):
        pix = torch.full((n,), -1, dtype=torch.int64, device="cuda")
        g.profile_reset()
        g.profile(True)
        img = g.render(dc, p, ipt.render_opts(seed=9, spp=1, max_depth=6, pixel_list=pix))
        torch.cuda.synchronize()
        g.profile(False)
        assert (img == 0).all()
        rays.append(g.profile_read(0)["rays"])
    assert rays == [0, 2]
