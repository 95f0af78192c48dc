"""The decode-step work measured for speed: cases, their inputs, one pass through
the public entry points, and what each pass cannot do without.

Every case is a part of one beam-search generation step as a serving or
evaluation loop runs it, with the buffers such a loop keeps (outputs and
zero-filled workspaces) made beforehand:

  step    ``beam_decode_step``: one layer's encoder-decoder attention with the
          step's no-repeat-n-gram scan in the same launch.
  cross   ``beam_cross_attn``: a layer's encoder-decoder attention alone.
  prefix  ``beam_prefix_attn``: self-attention over a split cache (shared prompt
          plus each beam's generated tokens), rows read directly or through an
          ancestry table; with N = 0 the self-attention of a decoder that has
          no prompt.
  select  ``beam_select``: log-softmax, bans and the best candidates per source.
  token   one whole generated token of a small decoder: the selection, the cache
          maintenance (rows moved, or the ancestry table), then every layer's
          self-attention and encoder-decoder attention.

Sizes are those of the workload configurations (BART, T5, ProphetNet and GPT2
shaped) and generic ones around them.
"""
import math

import numpy as np
import torch

from paper_2106_04718_amd import api

DEV = "cuda"
DT = {"bf16": torch.bfloat16, "f32": torch.float32}
ESIZE = {"bf16": 2, "f32": 4}


def listed():
    return [
        # One interactive request: 16 (source, head) rows, so latency and
        # launches count, not bandwidth.
        dict(name="step_one", kind="step", B=1, k=4, H=16, D=64, S=1024, lo=400, hi=1024, dtype="bf16",
             t=61, n=3, V=50264),
        # The BART-large-shaped summarisation step (the benchmark's default).
        dict(name="step_bart", kind="step", B=32, k=4, H=16, D=64, S=1024, lo=400, hi=1024, dtype="bf16",
             t=140, n=3, V=50264),
        # The T5-base-shaped translation step: more, shorter rows.
        dict(name="step_t5", kind="step", B=64, k=4, H=12, D=64, S=512, lo=128, hi=512, dtype="bf16",
             t=200, n=3, V=32128),
        # The large batch that de-duplication makes possible: the largest call.
        dict(name="step_large", kind="step", B=320, k=4, H=16, D=64, S=1024, lo=256, hi=1024, dtype="bf16",
             t=140, n=3, V=50264),
        # The same layer in single precision, as an accuracy run uses it.
        dict(name="step_f32", kind="step", B=32, k=4, H=16, D=64, S=1024, lo=400, hi=1024, dtype="f32",
             t=140, n=3, V=50264),
        # Wide heads, the widest beam, an odd source length.
        dict(name="cross_wide", kind="cross", B=24, k=8, H=16, D=128, S=777, lo=129, hi=777, dtype="bf16"),
        # GPT2-shaped decoder-only summarisation: a long shared prompt, few
        # generated tokens per beam.
        dict(name="prefix_gpt2", kind="prefix", B=16, k=4, H=12, D=64, N=1024, lo=400, hi=1024, T=140, t=64,
             dtype="bf16", table=False),
        # A long generation (the ProphetNet-shaped history of 512 tokens, beam
        # 5) behind a short prompt, cache maintained by the ancestry table.
        dict(name="prefix_long", kind="prefix", B=32, k=5, H=16, D=64, N=300, lo=75, hi=300, T=512, t=509,
             dtype="bf16", table=True),
        # The decoder self-attention of the BART-shaped step: no prompt, every
        # key is a generated token.
        dict(name="self_bart", kind="prefix", B=32, k=4, H=16, D=64, N=0, lo=0, hi=0, T=140, t=140, dtype="bf16",
             table=True),
        # The selection of the BART-shaped step, and of the large batch.
        dict(name="select_bart", kind="select", B=32, k=4, V=50264, t=140, n=3),
        dict(name="select_large", kind="select", B=320, k=4, V=50264, t=140, n=3),
        # One generated token of a small T5-base-shaped batch over six layers.
        dict(name="token_small", kind="token", B=4, k=4, H=12, D=64, S=512, lo=128, hi=512, T=64, t=37, n=3,
             V=32128, layers=6, maintain="reorder", dtype="bf16"),
    ]


MAX_KV_BYTES = 2 * 320 * 16 * 1024 * 64 * 2   # K and V of the largest listed step


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "cross", "prefix", "prefix", "select", "token"])
    k = rng.choice([1, 2, 3, 4, 4, 4, 5, 5, 6, 8])
    H = rng.choice([8, 12, 16])
    n = rng.choice([2, 3, 3, 4])
    V = rng.choice([30522, 32128, 50257, 50264])
    if kind == "select":
        return dict(kind=kind, B=_log_int(rng, 1, 320), k=min(k, 5) if rng.random() < 0.8 else k, V=V,
                    t=_log_int(rng, 1, 512), n=n)
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    D = rng.choice([64, 64, 64, 128])
    if kind == "token":
        S = _log_int(rng, 64, 512)
        t = _log_int(rng, 1, 140)
        return dict(kind=kind, B=_log_int(rng, 1, 16), k=min(k, 5), H=H, D=64, S=S, lo=max(1, S // 4), hi=S,
                    T=t + rng.randint(1, 32), t=t, n=n, V=V, layers=rng.randint(2, 6),
                    maintain=rng.choice(["reorder", "table"]), dtype="bf16")
    if kind == "prefix":
        N = 0 if rng.random() < 0.25 else _log_int(rng, 32, 2048)
        t = _log_int(rng, 1, 512)
        case = dict(kind=kind, B=_log_int(rng, 1, 64), k=k, H=H, D=D, N=N, lo=min(N, max(1, N // 4)), hi=N,
                    T=t + rng.randint(0, 64), t=t, dtype=dtype, table=rng.random() < 0.5)
    else:
        S = _log_int(rng, 64, 2048)
        case = dict(kind=kind, B=_log_int(rng, 1, 320), k=k, H=H, D=D, S=S, lo=max(1, S // 4), hi=S, dtype=dtype)
        if kind == "step":
            case.update(t=_log_int(rng, 1, 512), n=n, V=V)
    # never more than the largest listed call: fewer sources instead
    keys = case.get("S", case.get("N", 0)) + case["k"] * case.get("T", 0)
    per_source = 2 * H * keys * D * ESIZE[dtype]
    case["B"] = max(1, min(case["B"], MAX_KV_BYTES // 2 // per_source))
    return case


# ---- inputs -------------------------------------------------------------------

def _lengths(case, seed):
    """Valid keys per source, uniform over [lo, hi] (right padding)."""
    r = np.random.default_rng([seed, 1])
    return r.integers(case["lo"], case["hi"] + 1, size=case["B"]).astype(np.int32)


def _ancestry(case, seed, steps):
    """The table that `steps` selection steps leave: at each, hypothesis j of a
    source continues beam floor(k u^2) (the better beams more often), so old
    tokens mostly have one ancestor and recent ones differ.  [B*k, T] int32."""
    B, k = case["B"], case["k"]
    r = np.random.default_rng([seed, 2])
    par = np.floor(k * r.random((max(steps, 1), B, k)) ** 2).astype(np.int32)
    cur = np.tile(np.arange(k, dtype=np.int32), (B, 1))
    anc = np.tile(cur[:, :, None], (1, 1, case["T"]))
    for tau in range(steps - 1, -1, -1):       # back from the last step
        anc[:, :, tau] = cur
        cur = np.take_along_axis(par[tau], cur, axis=1)
    return anc.reshape(B * k, case["T"])


def _tokens(case, g, rows):
    """Zipf(1.1) history ids, one earlier copy of the last n - 1 tokens where it
    fits (text repeats some n-grams; independent draws hardly do)."""
    V, t, n = case["V"], case["t"], case["n"]
    p = torch.arange(1, V + 1, device=DEV, dtype=torch.float64) ** -1.1
    cdf = torch.cumsum(p / p.sum(), 0)
    u = torch.rand(rows, t, device=DEV, dtype=torch.float64, generator=g)
    tok = torch.searchsorted(cdf, u).clamp_(max=V - 1).to(torch.int32)
    hi = t - 2 * n + 2
    if n > 1 and hi >= 0:
        at = torch.randint(0, hi + 1, (rows, 1), device=DEV, generator=g)
        idx = at + torch.arange(n - 1, device=DEV)[None, :]
        tok.scatter_(1, idx, tok[:, t - n + 1:].clone())
    return tok.contiguous()


def _logits(case, g, rows):
    """A language model's scores: a broad body, a few likely tokens per row, and
    one id the caller has masked."""
    V = case["V"]
    x = torch.randn(rows, V, device=DEV, generator=g)
    x.mul_(2.0)
    top = torch.randint(0, V, (rows, 6), device=DEV, generator=g)
    x.scatter_add_(1, top, 6.0 + 2.0 * torch.randn(rows, 6, device=DEV, generator=g))
    x[:, 1] = -math.inf
    return x


def _randn(g, dtype, *shape):
    return torch.randn(*shape, device=DEV, dtype=DT[dtype], generator=g)


def _select_state(case, g, s):
    B, k = case["B"], case["k"]
    s["logits"] = _logits(case, g, B * k)
    s["tokens"] = _tokens(case, g, B * k)
    bs = -2.0 * torch.randn(B, k, device=DEV, generator=g).abs() - 10.0
    s["beam_scores"] = bs.sort(dim=1, descending=True).values.reshape(-1).contiguous()
    c = 2 * k
    s["sel_out"] = (torch.empty(B, c, device=DEV), torch.empty(B, c, dtype=torch.int32, device=DEV),
                    torch.empty(B, c, dtype=torch.int32, device=DEV))
    s["sel_ws"] = api.new_workspace(api.beam_select_workspace_bytes(B, k, case["V"], c), DEV)


def prepare(case, seed):
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    kind, B, k = case["kind"], case["B"], case["k"]
    s = {"case": case}
    if kind == "select":
        _select_state(case, g, s)
        return s
    H, D, dt = case["H"], case["D"], case["dtype"]
    s["len"] = torch.from_numpy(_lengths(case, seed)).to(DEV)
    if kind in ("step", "cross"):
        S = case["S"]
        s["q"] = _randn(g, dt, B, k, H, D)
        s["K"], s["V"] = _randn(g, dt, B, H, S, D), _randn(g, dt, B, H, S, D)
        s["out"] = torch.empty_like(s["q"])
        s["ws"] = api.new_workspace(api.beam_cross_attn_workspace_bytes(B, k, H, S, D, DT[dt]), DEV)
        if kind == "step":
            s["tokens"], s["logits"] = _tokens(case, g, B * k), _logits(case, g, B * k)
        return s
    T, t = case["T"], case["t"]
    if kind == "prefix":
        N = case["N"]
        s["q"] = _randn(g, dt, B, k, H, D)
        s["Kp"], s["Vp"] = _randn(g, dt, B, H, N, D), _randn(g, dt, B, H, N, D)
        s["Kt"], s["Vt"] = _randn(g, dt, B * k, H, T, D), _randn(g, dt, B * k, H, T, D)
        s["anc"] = torch.from_numpy(_ancestry(case, seed, t)).to(DEV) if case["table"] else None
        s["out"] = torch.empty_like(s["q"])
        s["ws"] = api.new_workspace(api.beam_prefix_attn_workspace_bytes(B, k, H, N, T, D, DT[dt]), DEV)
        return s
    # token
    _select_state(case, g, s)
    S = case["S"]
    s["layers"] = []
    for _ in range(case["layers"]):
        s["layers"].append(dict(
            q1=_randn(g, dt, B, k, H, D), q2=_randn(g, dt, B, k, H, D),
            Kt=_randn(g, dt, B * k, H, T, D), Vt=_randn(g, dt, B * k, H, T, D),
            K=_randn(g, dt, B, H, S, D), V=_randn(g, dt, B, H, S, D),
            o1=torch.empty(B, k, H, D, dtype=DT[dt], device=DEV), o2=torch.empty(B, k, H, D, dtype=DT[dt], device=DEV)))
    r = np.random.default_rng([seed, 3])
    s["parent"] = torch.from_numpy(np.floor(k * r.random(B * k) ** 2).astype(np.int32)).to(DEV)
    s["anc"] = torch.from_numpy(_ancestry(case, seed, t)).to(DEV) if case["maintain"] == "table" else None
    s["Kp"] = torch.empty(B, H, 0, D, dtype=DT[dt], device=DEV)
    s["plen"] = torch.zeros(B, dtype=torch.int32, device=DEV)
    s["ws1"] = api.new_workspace(api.beam_prefix_attn_workspace_bytes(B, k, H, 0, T, D, DT[dt]), DEV)
    s["ws2"] = api.new_workspace(api.beam_cross_attn_workspace_bytes(B, k, H, S, D, DT[dt]), DEV)
    return s


# ---- one pass -----------------------------------------------------------------

def run(s):
    case = s["case"]
    kind, k = case["kind"], case["k"]
    if kind == "step":
        out = api.beam_decode_step(s["q"], s["K"], s["V"], s["len"], s["tokens"], case["n"], s["logits"],
                                   out=s["out"], workspace=s["ws"])
        return {"out": out, "logits": s["logits"]}
    if kind == "cross":
        return {"out": api.beam_cross_attn(s["q"], s["K"], s["V"], s["len"], out=s["out"], workspace=s["ws"])}
    if kind == "prefix":
        return {"out": api.beam_prefix_attn(s["q"], s["Kp"], s["Vp"], s["len"], s["Kt"], s["Vt"], case["t"],
                                            out=s["out"], workspace=s["ws"], anc=s["anc"])}
    scores, beam, token = api.beam_select(s["logits"], s["beam_scores"], k, 2 * k, tokens=s["tokens"], n=case["n"],
                                          out=s["sel_out"], workspace=s["sel_ws"])
    got = {"scores": scores, "beam": beam, "token": token}
    if kind == "select":
        return got
    t = case["t"]
    if s["anc"] is not None:
        got["anc"] = api.ancestry_step(s["anc"], s["parent"], k, t)
    for i, L in enumerate(s["layers"]):
        if s["anc"] is None:
            api.cache_reorder(L["Kt"], L["Vt"], s["parent"], k, t)
            got["K%d" % i], got["V%d" % i] = L["Kt"], L["Vt"]
        got["self%d" % i] = api.beam_prefix_attn(L["q1"], s["Kp"], s["Kp"], s["plen"], L["Kt"], L["Vt"], t + 1,
                                                 out=L["o1"], workspace=s["ws1"], anc=s["anc"])
        got["cross%d" % i] = api.beam_cross_attn(L["q2"], L["K"], L["V"], s["len"], out=L["o2"], workspace=s["ws2"])
    return got


# ---- what a pass cannot do without --------------------------------------------

def _attn_work(case, keys, own_keys):
    """keys read for all k beams at once, own_keys (distinct rows over the
    beams) of the generated tokens; each dotted and accumulated once per beam."""
    B, k, H, D, es = case["B"], case["k"], case["H"], case["D"], ESIZE[case["dtype"]]
    by = 2 * (keys + own_keys) * H * D * es + 2 * B * k * H * D * es + 4 * B
    return by, 4 * D * H * k * keys


def _distinct(case, t, table):
    """Generated rows of one pass, each counted once (a table shares them)."""
    B, k = case["B"], case["k"]
    if not table:
        return B * k * t
    anc = _ancestry(case, 0, t)[:, :t].reshape(B, k, t)
    return int(sum((anc == i).any(axis=1).sum() for i in range(k)))


def work(case):
    kind, B, k = case["kind"], case["B"], case["k"]
    rows = B * k
    if kind in ("step", "cross"):
        by, fl = _attn_work(case, B * (case["lo"] + case["hi"]) // 2, 0)
        if kind == "step":
            by += rows * case["t"] * 4
        return {"bytes": by, "flops": fl}
    if kind == "prefix":
        t = case["t"]
        by, fl = _attn_work(case, B * (case["lo"] + case["hi"]) // 2, _distinct(case, t, case["table"]))
        return {"bytes": by + (rows * t * 4 if case["table"] else 0), "flops": fl + 4 * case["D"] * case["H"] * rows * t}
    by = rows * case["V"] * 4 + rows * case["t"] * 4 + rows * 4 + B * 2 * k * 12
    fl = 2 * rows * case["V"]
    if kind == "token":
        t, es = case["t"], ESIZE[case["dtype"]]
        table = case["maintain"] == "table"
        x, f = _attn_work(case, B * (case["lo"] + case["hi"]) // 2, 0)
        y, _ = _attn_work(case, 0, _distinct(case, t + 1, table))
        # moved rows: about half of the beams continue another beam
        z = 0 if table else 2 * 2 * (rows // 2) * case["H"] * t * case["D"] * es
        by += case["layers"] * (x + y + z) + (2 * rows * t * 4 if table else 0)
        fl += case["layers"] * (f + 4 * case["D"] * case["H"] * rows * (t + 1))
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # About four times the error measured against exact(): bf16 outputs and
    # probabilities are rounded to 8 bits (2.1e-3), single-precision sums over
    # a thousand keys (1.8e-7), scores less a log-sum-exp (3e-8).  Whole values
    # differ where two candidates score the same to the last bits.
    if case["kind"] == "select":
        return {"rel": 2e-7, "max": 2e-6, "differ": 2e-3}
    if case["kind"] == "token":
        return {"rel": 8e-3, "max": 4e-2, "differ": 2e-3}
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 1e-5}
    return {"rel": 8e-3, "max": 4e-2}


# ---- the same in 64 bits --------------------------------------------------------

def _attend(q, K, V, valid):
    """softmax(q K^T / sqrt(D)) V over the valid keys, in 64 bits; q [B,H,k,D],
    K, V [B,H,J,D], valid [B,1,1,J]; a row without keys is zero."""
    D = q.shape[-1]
    if K.shape[2] == 0:
        return torch.zeros_like(q)
    sc = torch.matmul(q, K.transpose(-1, -2).contiguous()) / math.sqrt(D)
    sc = sc.masked_fill(~valid, -math.inf)
    p = torch.softmax(sc, dim=-1)
    p = torch.where(valid, p, torch.zeros_like(p))
    return torch.matmul(p, V)


def _cross(q, K, V, length):
    out = []
    S = K.shape[2]
    j = torch.arange(S, device=DEV)
    for b0 in range(0, q.shape[0], 16):
        b = slice(b0, b0 + 16)
        valid = (j[None, :] < length[b, None])[:, None, None, :]
        o = _attend(q[b].double().permute(0, 2, 1, 3).contiguous(), K[b].double(), V[b].double(), valid)
        out.append(o.permute(0, 2, 1, 3).contiguous())
    return torch.cat(out)


def _prefix(q, Kp, Vp, length, Kt, Vt, t, anc):
    B, k, H, D = q.shape
    N, T = Kp.shape[2], Kt.shape[2]
    out = torch.empty(B, k, H, D, dtype=torch.float64, device=DEV)
    j = torch.arange(N + t, device=DEV)
    for b in range(B):
        valid = ((j < length[b]) | (j >= N))[None, None, None, :]
        blk_k, blk_v = (x[b * k:(b + 1) * k, :, :t].double() for x in (Kt, Vt))       # [k, H, t, D]
        if anc is not None:
            a = anc[b * k:(b + 1) * k, :t].long()[:, None, :, None].expand(k, H, t, D)
            blk_k, blk_v = torch.gather(blk_k, 0, a), torch.gather(blk_v, 0, a)
        kk = torch.cat([Kp[b].double()[None].expand(k, H, N, D), blk_k], dim=2)
        vv = torch.cat([Vp[b].double()[None].expand(k, H, N, D), blk_v], dim=2)
        out[b] = _attend(q[b].double()[:, :, None, :].contiguous(), kk, vv, valid)[:, :, 0]
    return out


def _banned(tokens, t, n):
    """(row, id) of Algorithm 1's bans."""
    if t < n:
        z = torch.zeros(0, dtype=torch.long, device=DEV)
        return z, z
    w = tokens[:, :t].unfold(1, n, 1)
    hit = (w[:, :, :n - 1] == tokens[:, None, t - n + 1:t]).all(-1)
    r, j = hit.nonzero(as_tuple=True)
    return r, w[r, j, n - 1].long()


def _select(s):
    case = s["case"]
    B, k, V = case["B"], case["k"], case["V"]
    r, v = _banned(s["tokens"], case["t"], case["n"])
    scores = []
    for b in range(B):
        x = s["logits"][b * k:(b + 1) * k].double()
        x = x - torch.logsumexp(x, dim=1, keepdim=True) + s["beam_scores"][b * k:(b + 1) * k].double()[:, None]
        mine = (r // k == b).nonzero(as_tuple=True)[0]
        x[r[mine] - b * k, v[mine]] = -math.inf
        scores.append(x.reshape(-1).topk(2 * k).values)
    return torch.stack(scores)


def exact(case, seed):
    s = prepare(case, seed)
    kind = case["kind"]
    if kind in ("step", "cross"):
        got = {"out": _cross(s["q"], s["K"], s["V"], s["len"])}
        if kind == "step":
            r, v = _banned(s["tokens"], case["t"], case["n"])
            s["logits"][r, v] = -math.inf
            got["logits"] = s["logits"]
        return got
    if kind == "prefix":
        return {"out": _prefix(s["q"], s["Kp"], s["Vp"], s["len"], s["Kt"], s["Vt"], case["t"], s["anc"])}
    got = {"scores": _select(s), "beam": None, "token": None}
    if kind == "select":
        return got
    k, t = case["k"], case["t"]
    rows = torch.arange(case["B"] * k, device=DEV)
    old = (rows // k) * k + s["parent"].long()
    anc = s["anc"]
    if anc is not None:
        anc[:, :t] = anc[old, :t].clone()
        anc[:, t] = (rows % k).to(torch.int32)
        got["anc"] = None
    for i, L in enumerate(s["layers"]):
        if anc is None:
            for x, name in ((L["Kt"], "K"), (L["Vt"], "V")):
                x[:, :, :t] = x[old, :, :t].clone()
                got["%s%d" % (name, i)] = x
        got["self%d" % i] = _prefix(L["q1"], s["Kp"], s["Kp"], s["plen"], L["Kt"], L["Vt"], t + 1, anc)
        got["cross%d" % i] = _cross(L["q2"], L["K"], L["V"], s["len"])
    return got
