"""Self-gravity at the sizes where its kernels change: a pair and a full group of 64
particles and one more, a tile of the sort (2,048) and one more, the last set whose groups
are walked by four wavefronts (1,792 groups) and the first by one, and the last whose sort
finds its tiles' starts without a scan (256 tiles) and the first with one.

As for the large sets, a sum of a few thousand terms in another order than the oracle's:
1e-12 of the largest acceleration."""
import numpy as np
import pytest
import torch

from oracle import native

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_1604_03290_amd")

G = 6.674e-11


@pytest.mark.parametrize("n", [2, 64, 65, 2048, 2049, 114688, 114689, 524288, 524289])
def test_sampled_bodies_match_oracle(n):
    rng = np.random.default_rng(n)
    pos, m = rng.normal(size=(3, n)), rng.uniform(1.0, 2.0, n)
    out = P.sph_gravity(torch.as_tensor(pos).cuda(), torch.as_tensor(m).cuda(), G, 0.7, 0.01, count=True)
    assert P.workspace_status(out["_ws"]) == 0
    idx = np.sort(rng.choice(n, min(n, 128), replace=False))
    ref = native.gravity(pos, m, G, 0.7, 0.01, targets=idx)
    assert out["nodes"] == ref["nodes"]
    ok = ~ref["tie"]
    assert ok.mean() >= 0.98
    cnt, acc = out["count"].cpu().numpy()[idx], out["acc"].cpu().numpy()[:, idx]
    assert np.array_equal(cnt[ok], ref["count"][ok])
    assert np.abs(acc[:, ok] - ref["acc"][:, ok]).max() <= 1e-12 * np.abs(ref["acc"]).max()
