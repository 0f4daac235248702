"""The light table and the colour sums by many blocks.

* The table of more lights than one block tabulates, at the edges of its 1024
  runs: the lights that the paths pick are the oracle's, which sums in float64
  (a path's hash covers the index; it may differ where u times the total falls on
  an entry to rounding, n 2^-24 of the picks at most, and on near-tied hits).
* Sums of 128 and more units per pixel: float32 sums of n terms in order agree
  with the float64 sum to n 2^-24.
"""
import numpy as np
import pytest
import torch

from _gpu import banner
from paper_1903_07145_amd import ipt, scenes

pytestmark = pytest.mark.gpu


def _pixel(w, h):
    return ipt.make_cameras(dict(cam_to_world=scenes.look_at([0.0, 0.0, 4.0], [0.0, 0.0, 0.0])[None],
                                 fov_y=np.array([0.9], np.float32), width=w, height=h))


def _lit_soup(n, S=8):
    v, f = scenes.random_soup(n, seed=1)
    e = np.arange(S, dtype=np.int32)
    g = ipt.Scene(v, f, np.arange(n, dtype=np.int32) % S, S, e)
    rng = np.random.default_rng(3)
    return g, v, f, rng.uniform(0.2, 0.9, g.P).astype(np.float32)


@pytest.mark.parametrize("n", [8192, 8193, 9217, 20000])
def test_light_table_of_many_blocks(n):
    banner("light table: %d lights" % n)
    from oracle import oracle
    g, v, f, p = _lit_soup(n)
    dc = _pixel(24, 16)
    kw = dict(seed=3, stream_tag=1, iteration=2, spp=4, max_depth=1, rr_depth=-1, mis=1)
    L = torch.empty((24 * 16 * 4, 3), device="cuda")
    h = torch.zeros(24 * 16 * 4, dtype=torch.int64, device="cuda")
    g.render(dc, torch.as_tensor(p, device="cuda"), ipt.render_opts(debug_path_hash=h, debug_path_radiance=L, **kw))
    o = oracle.Scene(v, f, np.arange(n, dtype=np.int32) % 8, 8, np.arange(8, dtype=np.int32), None)
    r = o.run(dict(cam_to_world=dc["c2w"].cpu().numpy().reshape(-1, 4, 4), fov_y=dc["fov"].cpu().numpy(), width=24,
                   height=16), p.astype(np.float64), want_hash=True, **kw)
    same = h.cpu().numpy().view(np.uint64) == r["hash"].reshape(-1)
    print("paths with the oracle's events: %.4f" % same.mean())
    # a light index differs only where u * total falls on a table entry to rounding
    assert same.mean() > 0.98


@pytest.mark.parametrize("spp", [127, 128, 129, 512])
def test_long_colour_sums(spp):
    banner("colour sums of %d units" % spp)
    sc = scenes.cornell()
    g = ipt.Scene.from_dict(sc)
    dc = ipt.make_cameras(dict(sc["cams"], width=11, height=1))
    p = torch.as_tensor(sc["params"], device="cuda")
    L = torch.empty((11 * spp, 3), device="cuda")
    img = g.render(dc, p, ipt.render_opts(seed=5, spp=spp, max_depth=3, debug_path_radiance=L))
    want = L.double().reshape(11, spp, 3).mean(1)
    assert ((img.double() - want).abs() <= (spp + 2) * 2.0 ** -24 * L.double().abs().reshape(11, spp, 3).mean(1)).all()
