"""The native argument checks of the tensor front end against the general path
in Python: the same outputs, or the same error, for plain calls and for every
form that only one of them could take (other strides, types, devices, sizes,
number types, leading dimensions, missing buffers)."""
import numpy as np
import pytest
import torch

from paper_2106_04718_amd import api

from _gpu import device, say

pytestmark = pytest.mark.gpu

B, k, H, S, D, T, V, LD = 2, 3, 2, 70, 64, 20, 101, 12


class General:
    """Stands in for the native module: declines every call."""

    def __getattr__(self, name):
        return lambda *a: None


def inputs():
    dev = device()
    g = torch.Generator(device=dev).manual_seed(7)
    r = lambda *s, dt=torch.bfloat16: torch.randn(*s, device=dev, dtype=dt, generator=g)
    i = lambda hi, *s: torch.randint(0, hi, s, device=dev, dtype=torch.int32, generator=g)
    ws = lambda n: api.new_workspace(n, dev)
    return dict(
        q=r(B, k, H, D), K=r(B, H, S, D), V=r(B, H, S, D), ln=torch.tensor([70, 33], dtype=torch.int32, device=dev),
        Kt=r(B * k, H, T, D), Vt=r(B * k, H, T, D), out=r(B, k, H, D), tok=i(6, B * k, LD), anc=i(k, B * k, T),
        lg=r(B * k, V, dt=torch.float32), bs=r(B * k, dt=torch.float32), par=i(k, B * k),
        so=(r(B, 4, dt=torch.float32), i(9, B, 4), i(9, B, 4)),
        wx=ws(api.beam_cross_attn_workspace_bytes(B, k, H, S, D)),
        wp=ws(api.beam_prefix_attn_workspace_bytes(B, k, H, S, T, D)), wsel=ws(api.beam_select_workspace_bytes(B, k, V, 4)))


def raw(t):
    """A tensor's bytes (and its type and shape)."""
    c = t.detach().cpu().contiguous()
    return str(t.dtype), tuple(t.shape), c.view(torch.uint8).numpy().tobytes() if c.numel() else b""


def sealed(x):
    """A tensor whose data pointer torch refuses to give (it throws)."""
    x = x.clone()
    torch._C._set_throw_on_mutable_data_ptr(x)
    return x


def wide(x):
    """The same values with a leading dimension past the columns."""
    return torch.cat([x, x], dim=1)[:, :x.shape[1]]


CALLS = {
    "cross": lambda x: api.beam_cross_attn(x["q"], x["K"], x["V"], x["ln"], out=x["out"], workspace=x["wx"]),
    "step": lambda x: api.beam_decode_step(x["q"], x["K"], x["V"], x["ln"], x["tok"], x.get("n", 2), x["lg"],
                                           t=x.get("t"), out=x["out"], workspace=x["wx"]),
    "prefix": lambda x: api.beam_prefix_attn(x["q"], x["K"], x["V"], x["ln"], x["Kt"], x["Vt"], x.get("t", 9),
                                             out=x["out"], workspace=x["wp"]),
    "table": lambda x: api.beam_prefix_attn(x["q"], x["K"], x["V"], x["ln"], x["Kt"], x["Vt"], x.get("t", 9),
                                            out=x["out"], workspace=x["wp"], anc=x["anc"]),
    "ngram": lambda x: api.ngram_block(x["tok"], x.get("n", 2), x["lg"], t=x.get("t")),
    "select": lambda x: api.beam_select(x["lg"], x["bs"], x.get("k", k), 4, tokens=x["tok"], n=x.get("n", 2),
                                        t=x.get("t"), out=x["so"], workspace=x["wsel"]),
    "reorder": lambda x: api.cache_reorder(x["Kt"], x["Vt"], x["par"], x.get("k", k), x.get("t")),
    "ancestry": lambda x: api.ancestry_step(x["anc"], x["par"], x.get("k", k), x.get("t", 5)),
}

CHANGES = {
    "plain": {},
    "t": dict(t=7), "t over": dict(t=10_000), "t negative": dict(t=-1), "t numpy": dict(t=np.int64(7)),
    "t huge": dict(t=1 << 40), "n 0": dict(n=0), "n -1": dict(n=-1), "n numpy": dict(n=np.int32(3)),
    "k 2": dict(k=2), "k 4": dict(k=4), "k numpy": dict(k=np.int64(3)),
    "tok ld": lambda x: dict(tok=wide(x["tok"])), "tok columns": lambda x: dict(tok=x["tok"].t().contiguous().t()),
    "tok int64": lambda x: dict(tok=x["tok"].long()), "tok cpu": lambda x: dict(tok=x["tok"].cpu()),
    "tok none": dict(tok=None), "tok rows": lambda x: dict(tok=x["tok"][:5]),
    "anc ld": lambda x: dict(anc=wide(x["anc"])), "anc rows": lambda x: dict(anc=x["anc"][:5].contiguous()),
    "q strided": lambda x: dict(q=x["q"].transpose(1, 2).contiguous().transpose(1, 2)),
    "q f32": lambda x: dict(q=x["q"].float()), "q parameter": lambda x: dict(q=torch.nn.Parameter(x["q"])),
    "sealed": lambda x: dict(q=sealed(x["q"]), tok=sealed(x["tok"]), par=sealed(x["par"])),
    "K 3d": lambda x: dict(K=x["K"][0]), "K cut": lambda x: dict(K=x["K"][:, :, :60].contiguous()),
    "len int64": lambda x: dict(ln=x["ln"].long()), "len 3": lambda x: dict(ln=x["ln"].repeat(2)[:3]),
    "out f32": lambda x: dict(out=x["out"].float()), "out none": dict(out=None), "so two": lambda x: dict(so=x["so"][:2]),
    "so shape": lambda x: dict(so=(x["so"][0][:, :3].contiguous(),) + x["so"][1:]),
    "small workspace": lambda x: dict(wx=x["wx"][:16], wp=x["wp"][:16], wsel=x["wsel"][:16]),
    "workspace none": dict(wx=None, wp=None, wsel=None), "V none": dict(V=None, Vt=None),
    "lg f16": lambda x: dict(lg=x["lg"].half()), "lg strided": lambda x: dict(lg=wide(x["lg"])),
    "bs 2d": lambda x: dict(bs=x["bs"][None]), "par int64": lambda x: dict(par=x["par"].long()),
    "aliased out": lambda x: dict(out=x["q"]), "no sources": lambda x: {
        key: (x[key][:0] if key != "so" else tuple(o[:0] for o in x["so"]))
        for key in ("q", "K", "V", "ln", "Kt", "Vt", "out", "tok", "anc", "lg", "bs", "par", "so")},
}


def outcome(call, change):
    x = inputs()
    x.update(change(x) if callable(change) else change)
    try:
        r = CALLS[call](x)
        torch.cuda.synchronize()
    except Exception as e:  # noqa: BLE001 - both paths have to raise the same
        return type(e).__name__, str(e).split("0x")[0]   # addresses differ between allocations
    seen = [r] if isinstance(r, torch.Tensor) else list(r) if r is not None else []
    seen += [x["lg"], x["Kt"], x["Vt"], x["anc"]]
    return [raw(t) if t is not None else None for t in seen]


@pytest.mark.parametrize("call", CALLS)
def test_native_checks_take_and_refuse_what_the_general_path_does(call, monkeypatch):
    for name, change in CHANGES.items():
        say(f"[front] {call}: {name}")
        monkeypatch.setattr(api, "_fast", None)
        a = outcome(call, change)
        monkeypatch.setattr(api, "_fast", General())
        b = outcome(call, change)
        assert type(a) is type(b), (call, name, a if isinstance(a, tuple) else "", b if isinstance(b, tuple) else "")
        if isinstance(a, tuple):
            assert a == b, (call, name)
        else:
            assert a == b, (call, name)


class Spy:
    """The native module, with what each call returned."""

    def __init__(self, native):
        self.native, self.seen = native, []

    def __getattr__(self, name):
        def call(*a):
            r = getattr(self.native, name)(*a)
            self.seen.append(r)
            return r
        return call


# forms that the native module leaves to the general path, by call
DECLINED = {
    "cross": ["q strided", "sealed"], "step": ["t numpy", "q strided", "tok cpu", "tok columns", "sealed"],
    "prefix": ["t numpy", "q strided", "sealed"], "table": ["t numpy", "q strided", "sealed"],
    "ngram": ["t numpy", "tok cpu", "tok columns", "sealed"], "select": ["t numpy", "tok cpu", "tok columns", "sealed"],
    "reorder": ["t numpy", "k numpy", "sealed"], "ancestry": ["t numpy", "k numpy", "sealed"],
}


@pytest.mark.parametrize("call", CALLS)
def test_the_native_module_takes_the_plain_call_and_leaves_the_others(call, monkeypatch):
    for name in ["plain", *DECLINED[call]]:
        say(f"[front] {call}: {name}")
        spy = Spy(api._load_fast())
        monkeypatch.setattr(api, "_fast", spy)
        outcome(call, CHANGES[name])
        assert spy.seen == [0 if name == "plain" else None], name
