"""The cell sizes that the ray kernel reads from a quantized node (x and y as the upper
halves of two floats in word 10, z as a float in word 11) are 2^(e + 24) for the node's
exponents e, exactly, up to the largest coordinates that a scene may have (1e12): the
bounds that other tests derive from the exponents hold for the ray kernel's planes too."""
import numpy as np
import pytest

from paper_1903_07145_amd import scenes
from test_host_bvh_wide import CASES, _build, harness  # noqa: F401


def _soup(n, seed, scale, stretch=(1.0, 1.0, 1.0)):
    v, f = scenes.random_soup(n, seed=seed)
    v = v.astype(np.float64) / np.abs(v).max() * np.asarray(stretch) * scale
    return v.astype(np.float32), f


SCENES = dict(CASES, **{
    "largest coordinates": lambda: _soup(3000, 8, 1e12),
    "one long axis": lambda: _soup(3000, 9, 1e12, (1.0, 1e-12, 1e-24)),
    "flat": lambda: _soup(3000, 10, 1.0, (1.0, 0.0, 1.0)),
    "tiny": lambda: _soup(3000, 11, 1e-30),
    "a point": lambda: _soup(5, 12, 0.0),
    "far from the origin": lambda: (lambda v, f: (v + np.float32(9e11), f))(*_soup(3000, 13, 1e11)),
})


@pytest.mark.parametrize("case", list(SCENES))
def test_cell_sizes(harness, case):  # noqa: F811
    verts, tris = SCENES[case]()
    nodes, _, _ = _build(harness, verts, tris, 1)
    w = nodes.view(np.uint32)
    e = np.stack([((w[:, 3] >> (8 * a)) & 0xFF).astype(np.int64) - 127 for a in range(3)], axis=1)
    size = np.stack([w[:, 10] & np.uint32(0xFFFF0000), w[:, 10] << np.uint32(16), w[:, 11]], axis=1)
    size = np.ascontiguousarray(size).view(np.float32)
    assert np.isfinite(size).all()
    assert np.array_equal(size.astype(np.float64), np.ldexp(1.0, e + 24))
