"""Training batches of several launches (more than 16384 records): every record's
input gradient is added to the embedding of its own segment.  One segment occurs
only beyond the first launch, so its 16 entries are the gradient of those records
alone; they are held to the oracle that rounds to bfloat16 where the kernel does,
at the bound of the single-launch batches (1e-2 of the block's norm)."""
import numpy as np
import pytest
import torch

import _guide
from _gpu import banner
from oracle import guide_ref
from paper_1903_07145_amd import ipt, scenes

pytestmark = pytest.mark.gpu

BF16_REL = 1e-2
LAUNCH = 16384   # records of one launch


@pytest.mark.parametrize("n", [LAUNCH, LAUNCH + 1, LAUNCH + 64, 40000])
def test_embedding_gradient_of_later_launches(n):
    banner("embedding gradient, batch of %d records" % n)
    S = 5
    v, f = scenes.random_soup(64, seed=1)
    g = ipt.Scene(v, f, np.arange(64, dtype=np.int32) % S, S, np.zeros(0, np.int32))
    w = _guide.random_weights(S, seed=12, out_gain=2.0)
    gd = ipt.Guide(g)
    gd.set_weights(w)
    rec = _guide.random_records(n, S, seed=n)
    seg = np.random.default_rng(n).integers(0, S - 1, n).astype(np.int32)
    late = max(1, min(n - LAUNCH, n // 8))   # the last records (of a single launch too) have the last segment
    seg[n - late:] = S - 1
    rec[:, 3] = seg.view(np.float32)
    loss, grad = gd.loss_grad(rec)
    torch.cuda.synchronize()
    want_loss, want = guide_ref.loss_grad_mfma(w, rec)[:2]
    assert abs(float(loss.cpu()) - want_loss) <= BF16_REL * abs(want_loss)
    grad = grad.cpu().numpy().astype(np.float64)
    a, b = grad[guide_ref.N_NET:].reshape(S, 16), want[guide_ref.N_NET:].reshape(S, 16)
    for s in range(S):
        rel = np.linalg.norm(a[s] - b[s]) / np.linalg.norm(b[s])
        print("segment %d |g| %.3e rel %.2e" % (s, np.linalg.norm(b[s]), rel))
        assert rel <= BF16_REL, (s, rel)
