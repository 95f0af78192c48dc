"""The split cache's two walks: generated tokens walked a beam per wave or
spread over all waves as tasks; and beams attended in groups on the vector tile
(fp32, and D = 16).  The two walks meet where the rule changes between them
(one tile, three tiles); groups have remainders at odd beam counts.  Every
decomposition gives the same bits, a beam's bits do not depend on how many
beams there are, and all match the oracle.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2106_04718_amd import api, workloads

from _gpu import assert_attn_close, bits, say, to_dev
from test_gpu_shared_tiles import table

pytestmark = pytest.mark.gpu

PATHS = ("split", "whole1", "whole2", "whole4")


def draw(rng, dtype, *shape):
    x = rng.standard_normal(shape).astype(np.float32)
    return x if dtype == "f32" else workloads.f32_to_bf16_bits(x)


# rows of a tile: 8 KiB of keys
@pytest.mark.parametrize("dtype,D", [("f32", 16), ("f32", 32), ("f32", 64), ("f32", 128), ("bf16", 16), ("bf16", 32),
                                     ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("k", [3, 4, 5, 6, 7, 8])
def test_both_walks_at_their_edges(dtype, D, k):
    B, H, tile = 2, 2, 8192 // (D * (4 if dtype == "f32" else 2))
    rng = np.random.default_rng(100 * D + k)
    for N, t in ((0, 1), (3, tile), (5 * tile + 1, tile + 1), (tile, 3 * tile), (2, 3 * tile + 1)):
        T = t + 2
        q, Kp, Vp = draw(rng, dtype, B, k, H, D), draw(rng, dtype, B, H, N, D), draw(rng, dtype, B, H, N, D)
        Kt, Vt = draw(rng, dtype, B * k, H, T, D), draw(rng, dtype, B * k, H, T, D)
        plen = np.array([N, N // 2], np.int32)
        anc = table(B, k, T, t, rng, True)
        Kg, Vg = oracle.gather_generated(Kt, anc, k, t), oracle.gather_generated(Vt, anc, k, t)
        dev = [to_dev(x) for x in (q, Kp, Vp, plen)]
        base = None
        for path in PATHS:
            say(f"[beam waves] {dtype} D={D} k={k} N={N} t={t} path={path}")
            with api.attn_path(path):
                ind = api.beam_prefix_attn(*dev, to_dev(Kt), to_dev(Vt), t, anc=to_dev(anc))
                direct = api.beam_prefix_attn(*dev, to_dev(Kg), to_dev(Vg), t)
            torch.cuda.synchronize()
            base = bits(direct) if base is None else base
            assert np.array_equal(bits(ind), base), (path, N, t)
            assert np.array_equal(bits(direct), base), (path, N, t)
        assert_attn_close(direct, oracle.prefix_attn(q, Kp, Vp, plen, Kg, Vg, t), f"{dtype} D={D} k={k} N={N} t={t}")


@pytest.mark.parametrize("D", [16, 32, 64, 128])
def test_groups_of_beams_give_each_beam_its_bits(D):
    # one beam alone against its place among up to eight, in every decomposition
    B, H, S = 2, 3, 5 * (2048 // D) + 3
    rng = np.random.default_rng(D)
    q = rng.standard_normal((B, 8, H, D)).astype(np.float32)
    K, V = (rng.standard_normal((B, H, S, D)).astype(np.float32) for _ in range(2))
    ln = np.array([S, S // 2], np.int32)
    for path in PATHS:
        with api.attn_path(path):
            alone = [bits(api.beam_cross_attn(to_dev(q[:, i:i + 1]), to_dev(K), to_dev(V), to_dev(ln)))
                     for i in range(8)]
            for k in (5, 6, 7, 8):
                say(f"[beam groups] D={D} k={k} path={path}")
                got = bits(api.beam_cross_attn(to_dev(q[:, :k]), to_dev(K), to_dev(V), to_dev(ln)))
                for i in range(k):
                    assert np.array_equal(got[:, i], alone[i][:, 0]), (path, k, i)
