"""GPU builds at the edges of the subtrees that one wave finishes (64 triangles)
and of the prefix sum over the leaves (blocks of 1024): the host builder's tree,
and the hits of a search over every triangle."""
import numpy as np
import pytest
import torch

from _gpu import banner, dev
from paper_1903_07145_amd import ipt, scenes

pytestmark = pytest.mark.gpu


def _scene(n, same_centre):
    v, f = scenes.random_soup(n, seed=n)
    if same_centre:   # boxes around one centre, exactly: the median cut
        s = (1.0 + np.arange(n, dtype=np.float32)) / 1024.0
        v = np.stack([np.stack([-s, -s, s], 1), np.stack([s, -s, -s], 1), np.stack([0 * s, s, 0 * s], 1)], 1)
        v = v.reshape(-1, 3).astype(np.float32)
    return dict(verts=v, normals=None, tris=f, tri_seg=np.zeros(n, np.int32), num_segments=1,
                emitter_seg=np.zeros(0, np.int32))


@pytest.mark.parametrize("same_centre", [False, True])
@pytest.mark.parametrize("n", [3, 63, 64, 65, 127, 129, 1023, 1026, 2049])
def test_build_edges(n, same_centre):
    banner("BVH build: %d triangles%s" % (n, ", one centre" if same_centre else ""))
    sc = _scene(n, same_centre)
    gg = ipt.Scene.from_dict(sc, bvh_builder=ipt.BVH_GPU)
    if not same_centre:   # median cuts follow the order inside a node, which the builders keep differently
        ig, ih = gg.info(), ipt.Scene.from_dict(sc, bvh_builder=ipt.BVH_HOST).info()
        assert (ig["num_nodes"], ig["bvh_depth"]) == (ih["num_nodes"], ih["bvh_depth"])
        assert abs(ig["sah_cost"] - ih["sah_cost"]) <= 1e-9 * ih["sah_cost"]   # float64 sums in another order
    rng = np.random.default_rng(n)
    lo, hi = sc["verts"].min(axis=0), sc["verts"].max(axis=0)
    org = rng.uniform(lo - 0.1, hi + 0.1, size=(4096, 3))
    d = rng.normal(size=(4096, 3))
    o, d = dev(org), dev(d / np.linalg.norm(d, axis=1, keepdims=True))
    for a, b in zip(gg.trace_rays(o, d), gg.trace_rays(o, d, brute_force=True)):
        assert torch.equal(a, b)
