"""fs_cache_reorder where sources or heads exceed one launch's grid (65535 in
each of its two outer dimensions, sources counted once per tensor)."""
import numpy as np
import pytest
import torch

from paper_2106_04718_amd import api

from _gpu import device, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,both", [(32768, 1, True), (32767, 1, True), (65536, 1, False), (1, 65536, True),
                                      (2, 70001, False)])
def test_more_sources_or_heads_than_a_launch_takes(B, H, both):
    k, T, t, D = 2, 3, 2, 4
    rng = np.random.default_rng(B + H)
    K = rng.standard_normal((B * k, H, T, D)).astype(np.float32)
    V = K + 1.0
    parent = rng.integers(0, k, size=B * k).astype(np.int32)
    say(f"[reorder grid] B={B} H={H} both={both}")
    gK, gV = torch.from_numpy(K).to(device()), torch.from_numpy(V).to(device())
    api.cache_reorder(gK, gV if both else None, torch.from_numpy(parent).to(device()), k, t)
    torch.cuda.synchronize()
    # the definition, by numpy indexing
    src = (np.arange(B * k) // k) * k + parent
    for got, x, moved in ((gK, K, True), (gV, V, both)):
        want = x.copy()
        if moved:
            want[:, :, :t] = x[src][:, :, :t]
        assert np.array_equal(got.cpu().numpy(), want)
