"""fs_beam_select over the sizes of its slice windows: every number of loads a
thread takes, at the edges where it changes, from rows that start at each
offset from 16 bytes; few and many records per merger; heavy masks and equal
logits in each.  Against the oracle, with the tolerance of the other tests of
the call (a few roundings of an fp32 log-normaliser).
"""
import numpy as np
import pytest
import torch

from paper_2106_04718_amd import api

import test_gpu_select
from _gpu import device, say
from test_gpu_select import check, random_case

pytestmark = pytest.mark.gpu


# a window of one slice is V + 3 positions at most, 2048 per load
@pytest.mark.parametrize("loads", range(1, 9))
def test_each_window_size_at_its_edges(loads):
    for V in (2048 * loads - 5, 2048 * loads - 4, 2048 * loads - 3, 2048 * (loads - 1) + 9):
        with api.select_slices(1):
            d = random_case(2, 3, V, 20, seed=loads * 10 + V % 7)
            check(d, 3, 6, 3, 20, f"one slice, V={V}")
            d = random_case(2, 3, V, 12, seed=V, neg_inf=0.999)     # a few finite logits per row
            check(d, 3, 5, 2, 12, f"one slice, V={V}, mostly -inf")
            d["logits"][:] = np.where(np.isinf(d["logits"]), -np.inf, np.float32(0.5))   # and those equal
            check(d, 3, 5, 2, 12, f"one slice, V={V}, equal")


MASKS = (-1e4, -1e9, -1e10, -1e30, float(np.finfo(np.float32).min))


@pytest.mark.parametrize("loads", range(1, 9))
def test_finite_mask_values(loads):
    # whole lanes, and whole waves, of one mask value beside ordinary logits:
    # a lane's own maximum is then the mask value, whose product with log2 e
    # rounds by more than the exponent's range (or overflows)
    V = 2048 * loads - 3
    rng = np.random.default_rng(loads)
    for mask in MASKS:
        for what, share in (("90 %", 0.9), ("99.9 %", 0.999), ("a run", 0.0)):
            d = random_case(2, 3, V, 12, seed=loads)
            if share:
                d["logits"][rng.random(d["logits"].shape) < share] = mask
            else:
                d["logits"][:, V // 8:] = mask
            d["logits"][:, 1:9] = np.linspace(0.0, 1.0, 8, dtype=np.float32)   # picks that are no mask value
            with api.select_slices(1):
                check(d, 3, 6, 2, 12, f"one slice, V={V}, {what} {mask}")


def test_rows_of_one_finite_value():
    # every logit of a row the same: the normaliser is that value plus log V,
    # held in fp32, so a score is off by its rounding at that value's size
    dev = device()
    V = 5003
    for x in MASKS + (0.0, 1e30):
        lg = torch.full((6, V), x, device=dev)
        bs = torch.tensor([-1.0, -2.0, -3.0, -1.5, -1.5, -1.5], device=dev)
        say(f"[select parity] rows of {x}")
        s, i, v = (o.cpu().numpy() for o in api.beam_select(lg, bs, 3, 6))
        assert np.isfinite(s).all()
        want = bs.cpu().numpy().reshape(2, 3)[np.arange(2)[:, None], i] - np.log(V)
        assert np.all(np.abs(s - want) <= 1e-5 * (1 + np.abs(want)) + np.spacing(np.float32(abs(x)))), x
        for b in range(2):
            assert len({(int(p), int(w)) for p, w in zip(i[b], v[b])}) == 6 and v[b].min() >= 0 and v[b].max() < V


def test_nan_beside_masked_logits_reaches_the_scores():
    # a NaN logit must not pass for a masked one: the row has no normaliser, so
    # none of its scores is a number, whatever the other logits of its lane are
    dev = device()
    V = 4099
    for rest in (-np.inf, 0.5):
        for at in (1000, 1003, 4098):
            lg = torch.full((2, V), rest, device=dev)
            lg[:, 960:1100:20] = 1.0       # ordinary logits in the lanes about it
            lg[:, 4060:4096:20] = 1.0
            lg[0, at] = float("nan")
            say(f"[select parity] NaN at {at}, rest {rest}")
            s = api.beam_select(lg, torch.zeros(2, device=dev), 1, 4)[0].cpu().numpy()
            assert not np.isfinite(s[0]).any() and np.isfinite(s[1]).all(), (at, rest, s)


def test_common_offset_costs_nothing():
    # scores that spread little about a large common value reach the same few
    # candidates as the same scores about 0: not the c rounds over every value
    # that equal logits need (2.5 times as long at these sizes)
    dev = device()
    B, k, V, c = 32, 4, 50264, 8
    g = torch.Generator(device=dev).manual_seed(5)
    x = torch.randn(B * k, V, device=dev, generator=g)
    bs = torch.zeros(B * k, device=dev)
    out = (torch.empty(B, c, device=dev), torch.empty(B, c, dtype=torch.int32, device=dev),
           torch.empty(B, c, dtype=torch.int32, device=dev))
    ws = api.new_workspace(api.beam_select_workspace_bytes(B, k, V, c), dev)

    def time_of(lg):
        best = float("inf")
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(20):
                api.beam_select(lg, bs, k, c, out=out, workspace=ws)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    ref = time_of(x)
    for off in (4e3, 1e4, -1e4, 1e5):
        say(f"[select time] offset {off}")
        assert time_of(x + off) < 1.5 * ref, off


@pytest.mark.parametrize("offset", [0.0, 4e3, 1e4, -1e4])
@pytest.mark.parametrize("step", [0.0, 2.0 ** -10, 2.0 ** -8, 1.0])
def test_offset_logits_of_few_values(offset, step, monkeypatch):
    # ties, and values that the threshold's first bits do not tell apart, around
    # the counts at which the threshold is finished and at which the exact path runs
    # (the fp32 normaliser is off by one rounding at the logits' size)
    size = np.spacing(np.float32(abs(offset) + 300 * step))
    monkeypatch.setattr(test_gpu_select, "tol", lambda v: 1e-5 * (1.0 + np.abs(v)) + size)
    for V, seed in ((4099, 1), (16381, 2)):
        d = random_case(2, 2, V, 12, seed=seed)
        d["logits"] = (np.float32(offset) + np.float32(step) * np.floor(d["logits"] * 64)).astype(np.float32)
        with api.select_slices(1):
            check(d, 2, 8, 2, 12, f"V={V}, offset {offset}, steps of {step}")


@pytest.mark.parametrize("k,slices,c", [(1, 64, 8), (1, 65, 8), (2, 33, 4), (4, 16, 16), (5, 13, 8), (16, 4, 16),
                                        (1, 1, 16), (3, 22, 15)])
def test_records_of_a_merger(k, slices, c):
    # up to 64 records are pruned by every wave on its own, more through LDS
    with api.select_slices(slices):
        d = random_case(3, k, 5003 + slices, 30, seed=k * 100 + slices)
        check(d, k, c, 2, 30, f"k={k} slices={slices} c={c}")


def test_threshold_between_close_values():
    # values that differ only below the threshold's leading 20 bits, of both
    # signs: more candidates are collected, the picks stay the same
    dev = device()
    rng = np.random.default_rng(3)
    for sign in (1.0, -1.0):
        x = np.float32(sign) * (np.float32(4.0) + rng.permutation(6000).astype(np.float32) * np.float32(4.8e-7))
        lg = torch.from_numpy(x[None]).to(dev)
        say(f"[select threshold] sign={sign}")
        s, i, v = api.beam_select(lg, torch.zeros(1, device=dev), 1, 16)
        torch.cuda.synchronize()
        # equal values after the subtraction of the normaliser resolve to the smaller index
        sc = s.cpu().numpy()[0]
        assert np.all(np.diff(sc) <= 0)
        got = x[v.cpu().numpy()[0]]
        want = np.sort(x)[::-1][:16]
        assert np.all(np.abs(got - want) <= np.spacing(np.float32(12.7)))   # one rounding of x - lse, lse < 12.71
