"""`Scene.loss_grad` sizes its workspace for both passes: with more colour samples than
gradient samples (the paper's setting: 512 and 1) the colour pass's lists need more than
the gradient's query asks for.  Without a GPU: the library's calls are stand-ins."""
import types

import pytest

from paper_1903_07145_amd import ipt

RECORD, LIST = 48, 224   # bytes of a vertex record and of a path's lists


class _Bytes:
    def __init__(self, n):
        self.n = n

    def numel(self):
        return self.n


def _query(dcams, o):
    """A workspace query of the library's form: fixed part, vertex records, lists."""
    paths = o.num_pixels * o.spp
    return 1000, 1000 + paths * ((o.max_depth + 1) * RECORD + LIST)


@pytest.fixture
def scene(monkeypatch):
    g = ipt.Scene.__new__(ipt.Scene)
    g.handle, g._ws, g.P, g.passed = None, None, 7, []
    g.workspace_query = _query
    torch = types.SimpleNamespace(uint8=None, float32=None, cuda=types.SimpleNamespace(empty_cache=lambda: None),
                                  empty=lambda n, **k: _Bytes(n))
    monkeypatch.setattr(ipt, "torch", torch)
    monkeypatch.setattr(ipt, "_ptr", lambda t: None)
    monkeypatch.setattr(ipt, "_stream", lambda: None)
    monkeypatch.setattr(ipt, "_cams_struct", lambda d: ipt.Cameras())
    monkeypatch.setattr(ipt, "lib", lambda: types.SimpleNamespace(
        ipt_loss_grad=lambda *a: g.passed.append(a[-2]) or ipt.IPT_OK))
    return g


def _opts(pixels, spp, depth):
    o = ipt.RenderOpts()
    o.num_pixels, o.spp, o.max_depth = pixels, spp, depth
    return o


@pytest.mark.parametrize("colour,grad", [(512, 1), (64, 8), (8, 8), (4, 16)])
def test_workspace_covers_both_passes(scene, colour, grad):
    co, go = _opts(8, colour, 7), _opts(8, grad, 7)
    scene.loss_grad(None, None, None, co, go)
    lists = 1000 + 8 * colour * LIST                      # the colour pass: no vertex records
    assert scene.passed[0] >= max(lists, _query(None, go)[1])
    assert scene.passed[0] <= max(lists + 8 * colour * 2 * RECORD, _query(None, go)[1])
    assert co.max_depth == 7 and co.spp == colour         # the caller's options stay as they are
