"""Performance cases of the mLSTM entry points: what is timed, on which inputs, and what the results have to be.

A case is a dict of plain values.  ``entry`` names the public entry points that one pass goes through:

* ``step`` / ``layer_step``: one generation step from a state (C, n, m), cell only or with NORM and output gate;
* ``fwd`` / ``layer_fwd``: a prompt, from a given or a zero state, with the final state as a result;
* ``train`` / ``layer_train``: forward and backward; ``keep`` says whether the backward call is handed the forward
  call's workspace or recomputes the gates and chunk states (the memory-saving choice).

The program that is imagined around a pass owns its output tensors and workspaces, as ``bench.py`` does, and has the
inputs on the GPU.  Shapes and gate distributions are those of ``workloads.py``, the tests and the benchmark's sweeps:
8 heads of 256 / 512 (the 7B head shape), 4096 columns in all split over heads of 32 to 1024, sequences from a few
hundred steps to 32768, the chunk sizes 64 to 512.
"""
from __future__ import annotations

import math

import torch

import paper_2503_14376_amd as tfla
from paper_2503_14376_amd.binding import BWD, FWD

EPS = 1e-6
NORM_EPS = 1e-6


def _case(name, entry, B, NH, T, dqk, dhv, chunk=256, variant="exp", dtype="bf16", state=False, keep=True, f_mean=3.0,
          norm="rms", softcap=15.0):
    return {"name": name, "entry": entry, "B": B, "NH": NH, "T": T, "dqk": dqk, "dhv": dhv, "chunk": chunk,
            "variant": variant, "dtype": dtype, "state": state, "keep": keep, "f_mean": f_mean, "norm": norm,
            "softcap": softcap}


def listed():
    return [
        # one sequence generating with the 7B head shape: the smallest call, repeated once per layer and token
        _case("generate_one", "layer_step", 1, 8, 1, 256, 512, state=True),
        # a serving batch of 32 sequences generating together: the state traffic of App. F
        _case("generate_batch", "step", 32, 8, 1, 256, 512, state=True),
        # a prompt of ordinary, odd length through one layer of the 7B head shape
        _case("prompt_ragged", "layer_fwd", 1, 8, 1000, 256, 512, chunk=128, norm="layer"),
        # a long document, continued from an earlier state (long-context configuration)
        _case("prompt_long", "fwd", 1, 8, 32768, 256, 512, chunk=512, state=True, f_mean=5.0),
        # the headline training step of the kernels
        _case("train_7b", "train", 2, 8, 8192, 256, 512),
        # the same head shape with the sigmoid input gate, one sequence, states recomputed in the backward pass
        _case("train_sig_recompute", "train", 1, 8, 8192, 256, 512, variant="sig", keep=False),
        # a whole layer of that shape on a batch of sequences that do not fill their last chunk
        _case("layer_ragged", "layer_train", 2, 8, 4000, 256, 512, norm="layer"),
        # many narrow heads (4096 columns as 64 heads of 64) in a layer
        _case("layer_heads_64", "layer_train", 4, 64, 2048, 64, 64),
        # the wide end of the head-dimension sweep (4096 columns as 4 heads of 1024)
        _case("train_heads_1024", "train", 4, 4, 4096, 1024, 1024),
        # head dimensions between the kernels' widths, odd length, initial state and upstream state gradient
        _case("train_odd_heads", "train", 2, 16, 3000, 96, 192, chunk=128, state=True),
        # single precision: the smallest training call, and an ordinary one
        _case("train_f32_small", "train", 1, 1, 256, 64, 64, chunk=64, dtype="f32"),
        _case("train_f32", "train", 2, 8, 1024, 128, 256, chunk=64, dtype="f32", variant="sig", state=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _odd(rng, x, share=0.5):
    """x, or (with the given probability) a nearby length that is no multiple of anything."""
    return max(1, x - rng.randrange(1, max(2, x // 8))) if rng.random() < share else x


def _cost(c):
    """A rough time of one pass in seconds (not a floor): keeps drawn cases below the largest listed one."""
    w = work(c)
    return w["bytes"] / 2.5e12 + w["flops"] / (2.0e13 if c["dtype"] == "f32" else 4.0e14)


# the head shapes of the configurations, the head-dimension sweep and the tests
_SHAPES = [(8, 256, 512), (8, 128, 128), (128, 32, 32), (64, 64, 64), (32, 128, 128), (16, 256, 256), (8, 512, 512),
           (4, 1024, 1024), (16, 96, 192), (4, 192, 80), (8, 64, 128), (4, 512, 256)]


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        entry = rng.choice(["step", "layer_step", "fwd", "layer_fwd", "train", "train", "layer_train"])
        NH, dqk, dhv = rng.choice(_SHAPES)
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        c = _case("", entry, 1, NH, 1, dqk, dhv, variant=rng.choice(["exp", "exp", "sig"]), dtype=dtype,
                  state=rng.random() < 0.4, keep=rng.random() < 0.7, norm=rng.choice(["rms", "layer"]),
                  f_mean=rng.choice([3.0, 3.0, 5.0]))
        del c["name"]
        if "step" in entry:
            if dqk % 64 or dhv % 64:
                continue
            c["B"], c["state"] = _log_int(rng, 1, 64), True
        else:
            c["B"] = _log_int(rng, 1, 8)
            c["chunk"] = rng.choice([64, 128, 256, 256, 512])
            c["T"] = _odd(rng, _log_int(rng, 128, 16384))
        if dtype == "f32" and max(dqk, dhv) > 512:
            continue
        if _cost(c) <= most:
            return c


def _variant(c):
    return tfla.EXP if c["variant"] == "exp" else tfla.SIG


def _inputs(c, seed):
    """Every tensor that the program has before the call: N(0, 1) activations, gate pre-activations as the configurations
    name them (in a layer twice as wide, so that the soft-cap bends them), states of a sequence under way."""
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 11)
    B, NH, T, dqk, dhv = c["B"], c["NH"], c["T"], c["dqk"], c["dhv"]
    td = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    lead = (B, NH) if "step" in c["entry"] else (B, NH, T)

    def normal(*shape, dtype=torch.float32, mean=0.0, std=1.0):
        return (torch.randn(shape, generator=g, device="cuda") * std + mean).to(dtype)

    layer = "layer" in c["entry"]
    gs = 2.0 if layer else 1.0
    t = {"q": normal(*lead, dqk, dtype=td), "k": normal(*lead, dqk, dtype=td), "v": normal(*lead, dhv, dtype=td),
         "i_pre": normal(*lead, std=gs), "f_pre": normal(*lead, mean=c["f_mean"] * gs, std=gs)}
    if layer:
        t["o_pre"] = normal(*lead, dhv, dtype=td)
        t["gamma"] = normal(NH, dhv, mean=1.0, std=0.1)
        t["beta"] = normal(NH, dhv, std=0.1)
    if c["state"]:
        t["C0"], t["n0"] = normal(B, NH, dqk, dhv, std=0.1), normal(B, NH, dqk, std=0.1)
        t["m0"] = torch.zeros((B, NH), device="cuda")
    if "train" in c["entry"]:
        t["dH"] = normal(*lead, dhv, dtype=td)
        if c["state"]:
            t["dCn"] = normal(B, NH, dqk, dhv, std=0.1)
    return t


def prepare(case, seed):
    c, t = dict(case), _inputs(case, seed)
    s = {"c": c, "t": t, "fo": {}, "bo": {}, "fw": None, "bw": None}
    B, NH, T, dqk, dhv = c["B"], c["NH"], c["T"], c["dqk"], c["dhv"]
    f32 = dict(dtype=torch.float32, device="cuda")
    new = torch.empty_like
    if "step" in c["entry"]:
        s["fo"] = {"h": new(t["v"]), "C": new(t["C0"]), "n": new(t["n0"]), "m": new(t["m0"])}
        if c["entry"] == "layer_step":
            s["fo"]["y"] = new(t["v"])
        return s
    wsb = tfla.layer_workspace_bytes if "layer" in c["entry"] else tfla.workspace_bytes
    dims = (B, NH, T, dqk, dhv, c["chunk"], _variant(c), tfla.BF16 if c["dtype"] == "bf16" else tfla.F32)
    s["fw"] = torch.empty(wsb(FWD, *dims), dtype=torch.uint8, device="cuda")
    s["fo"] = {"H": new(t["v"]), "Cn": torch.empty((B, NH, dqk, dhv), **f32), "nn": torch.empty((B, NH, dqk), **f32),
               "mn": torch.empty((B, NH), **f32), "n_out": new(t["i_pre"]), "m_out": new(t["i_pre"])}
    if "layer" in c["entry"]:
        s["fo"]["Y"] = new(t["v"])
    if "train" in c["entry"]:
        s["bw"] = torch.empty(wsb(BWD, *dims), dtype=torch.uint8, device="cuda")
        s["bo"] = {"dq": new(t["q"]), "dk": new(t["k"]), "dv": new(t["v"]), "d_i_pre": new(t["i_pre"]),
                   "d_f_pre": new(t["f_pre"])}
        if c["state"]:
            s["bo"]["dC0"] = new(t["C0"])
        if "layer" in c["entry"]:
            s["bo"].update(do_pre=new(t["v"]), dgamma=new(t["gamma"]), dbeta=new(t["beta"]))
    return s


def _without_workspace(o):
    return {k: v for k, v in o.items() if k != "workspace"}


def run(state):
    c, t = state["c"], state["t"]
    entry = c["entry"]
    kw = dict(variant=_variant(c), eps=EPS)
    layer = {}
    if "layer" in entry:
        kw.update(gate_softcap=c["softcap"], norm_kind=tfla.NORM_RMS if c["norm"] == "rms" else tfla.NORM_LAYER,
                  norm_eps=NORM_EPS)
        layer = dict(o_pre=t["o_pre"], gamma=t["gamma"], beta=t["beta"])
    qkv = (t["q"], t["k"], t["v"], t["i_pre"], t["f_pre"])
    if "step" in entry:
        call = tfla.mlstm_layer_step if layer else tfla.mlstm_step
        return call(*qkv, t["C0"], t["n0"], t["m0"], **layer, **kw, out=state["fo"])
    kw["chunk"] = c["chunk"]
    st = dict(C0=t.get("C0"), n0=t.get("n0"), m0=t.get("m0"))
    call = tfla.mlstm_layer_fwd if layer else tfla.mlstm_fwd
    f = call(*qkv, **layer, **st, **kw, workspace=state["fw"], out=state["fo"])
    out = _without_workspace(f)
    if "train" in entry:
        st.update(n_out=f["n_out"], m_out=f["m_out"], dCn=t.get("dCn"), want_dC0=c["state"], out=state["bo"],
                  workspace=state["bw"], fwd_workspace=f["workspace"] if c["keep"] else None)
        if layer:
            g = tfla.mlstm_layer_bwd(*qkv, f["H"], t["dH"], **layer, **st, **kw)
        else:
            g = tfla.mlstm_bwd(*qkv, t["dH"], **st, **kw)
        out.update(_without_workspace(g))
    return out


def work(case):
    """Bytes: inputs and results once.  Operations: the matrix products of the chunkwise form (App. F.1 with half of the
    causal square counted) and, for a generation step, of the recurrence."""
    c = case
    es = 2 if c["dtype"] == "bf16" else 4
    BH, T, dqk, dhv = c["B"] * c["NH"], c["T"], c["dqk"], c["dhv"]
    tok = BH * T
    layer, train = "layer" in c["entry"], "train" in c["entry"]
    state = BH * (dqk * dhv + dqk + 1) * 4
    row_qk, row_v = dqk * es, dhv * es
    gates = 8
    if "step" in c["entry"]:
        per = 2 * row_qk + 2 * row_v + gates + (2 * row_v if layer else 0)
        return {"bytes": tok * per + 2 * state, "flops": BH * 5 * dqk * dhv}
    L = min(c["chunk"], T)
    # forward: q, k, v, gates in; h, the two per-step scalars and the final state out
    per = 2 * row_qk + 2 * row_v + gates + 8 + (2 * row_v if layer else 0)
    b = tok * per + state * (2 if c["state"] else 1)
    f = tok * (4 * dqk * dhv + L * (dqk + dhv))
    if train:
        # backward: the same inputs and the upstream gradient again; dq, dk, dv and the gate gradients out
        per = 2 * (2 * row_qk + row_v) + row_v + gates + 8 + 8 + (3 * row_v if layer else 0)
        b += tok * per + (state * 3 if c["state"] else 0)
        f += tok * (8 * dqk * dhv + L * (3 * dqk + 2 * dhv))
    return {"bytes": b, "flops": f}


def tolerance(case):
    """About four times the distance from the 64-bit results that was measured over the ranges (2-norm; largest
    element).  bf16: 1.5e-3 to 2.9e-3 for activations and their gradients (the rounding of the results and of the weights
    and states as matrix operands), 6e-3 for the forget gate's gradient, a cumulative sum of differences that cancel, and
    1.2e-2 for it behind a norm; single elements are further off where the normaliser is near its lower bound.  fp32:
    4e-7 for most, 9e-6 for the forget gate's gradient of a long sequence, 4e-5 for h with such normalisers."""
    c = case
    layer, train = "layer" in c["entry"], "train" in c["entry"]
    if c["dtype"] == "f32":
        return {"rel": 1.5e-4 if c["variant"] == "exp" else 4e-5, "max": 2e-2 if c["variant"] == "exp" else 1e-3}
    if "step" in c["entry"]:
        return {"rel": 1e-2, "max": 3e-2}
    if not train:
        return {"rel": 1.2e-2, "max": 0.9}
    return {"rel": 3e-2, "max": 0.99} if layer else {"rel": 2.4e-2, "max": 0.9}


# ---- 64-bit results, from the definitions -------------------------------------------------------------------------


def _norm(x, gamma, beta, kind):
    if kind == "layer":
        x = x - x.mean(-1, keepdim=True)
    x = x / torch.sqrt((x * x).mean(-1, keepdim=True) + NORM_EPS) * gamma[None, :, None, :]
    return x + beta[None, :, None, :] if kind == "layer" else x


def _cell(c, q, k, v, i, f, C, n, m, block):
    """The recurrence in blocks of `block` steps on (G, T, .) tensors; the max states and the denominators are constants
    for the gradient.  Returns H, the last state and the per-step normaliser and max state."""
    is_exp = c["variant"] == "exp"
    T = q.shape[1]
    q = q / math.sqrt(q.shape[-1])
    fb = torch.nn.functional.logsigmoid(f)
    ib = i if is_exp else torch.nn.functional.logsigmoid(i)
    hs, ns, ms = [], [], []
    for t0 in range(0, T, block):
        t1 = min(T, t0 + block)
        qq, kk, vv, ii = q[:, t0:t1], k[:, t0:t1], v[:, t0:t1], ib[:, t0:t1]
        b = torch.cumsum(fb[:, t0:t1], 1)
        low = torch.ones(t1 - t0, t1 - t0, dtype=torch.bool, device=q.device).tril()
        D = (b[:, :, None] - b[:, None, :] + ii[:, None, :]).masked_fill(~low, -math.inf)
        if is_exp:
            mt = torch.maximum(b + m[:, None], D.amax(2)).detach()
        else:
            mt = torch.zeros_like(b)
        W = torch.exp(D - mt[:, :, None]) * (qq @ kk.transpose(1, 2))
        sc = torch.exp(b + m[:, None] - mt)[:, :, None]
        num = W @ vv + sc * (qq @ C)
        m1 = mt[:, -1].detach()
        decay = torch.exp(b[:, -1] + m - m1)
        ks = torch.exp(b[:, -1:] - b + ii - m1[:, None])[:, :, None] * kk
        if is_exp:
            nq = (W.sum(2) + (sc * (qq @ n[:, :, None]))[:, :, 0]).detach()
            num = num / (torch.maximum(nq.abs(), torch.exp(-mt)) + EPS)[:, :, None]
            ns.append(nq)
            n = decay[:, None] * n + ks.detach().sum(1)
            n = n.detach()
        else:
            ns.append(torch.zeros_like(b).detach())
        hs.append(num)
        ms.append(mt)
        C = decay[:, None, None] * C + ks.transpose(1, 2) @ vv
        m = m1 if is_exp else m
    return torch.cat(hs, 1), C, n, m, torch.cat(ns, 1), torch.cat(ms, 1)


def exact(case, seed):
    c = case
    t = {k: x.double() for k, x in _inputs(c, seed).items()}
    entry = c["entry"]
    layer, train, step = "layer" in entry, "train" in entry, "step" in entry
    B, NH, T, dqk, dhv = c["B"], c["NH"], c["T"], c["dqk"], c["dhv"]
    if step:
        for k in ("q", "k", "v", "o_pre"):
            if k in t:
                t[k] = t[k][:, :, None]
        t["i_pre"], t["f_pre"] = t["i_pre"][:, :, None], t["f_pre"][:, :, None]
    BH = B * NH
    state = [t[k] if k in t else torch.zeros((B, NH) + s, dtype=torch.float64, device="cuda")
             for k, s in (("C0", (dqk, dhv)), ("n0", (dqk,)), ("m0", ()))]
    if c["variant"] != "exp":
        state[1], state[2] = torch.zeros_like(state[1]), torch.zeros_like(state[2])
    block = max(16, min(128, T))
    # heads in groups that keep the graph of a group to a few GB
    per = T * (block * 8 + 2 * dqk + 6 * dhv) * 8 + (T // block + 1) * dqk * dhv * 32
    group = max(1, min(NH, int(12e9 / per)))
    parts = []
    for b in range(B):
        for h0 in range(0, NH, group):
            hs = slice(h0, min(NH, h0 + group))
            leaf = {k: t[k][b, hs].clone().requires_grad_(train) for k in ("q", "k", "v", "i_pre", "f_pre", "o_pre") if k in t}
            leaf["C0"] = state[0][b, hs].clone().requires_grad_(train)
            if layer:
                leaf["gamma"], leaf["beta"] = (t[k][hs].clone().requires_grad_(train) for k in ("gamma", "beta"))
            with torch.set_grad_enabled(train):
                i, f = leaf["i_pre"], leaf["f_pre"]
                if layer:
                    i, f = (c["softcap"] * torch.tanh(x / c["softcap"]) for x in (i, f))
                H, Cn, nn, mn, no, mo = _cell(c, leaf["q"], leaf["k"], leaf["v"], i, f, leaf["C0"], state[1][b, hs],
                                              state[2][b, hs], block)
                y = H
                if layer:
                    y = torch.sigmoid(leaf["o_pre"]) * _norm(H[None], leaf["gamma"], leaf["beta"], c["norm"])[0]
                o = {"H": H, "Cn": Cn, "nn": nn, "mn": mn, "n_out": no, "m_out": mo}
                if layer:
                    o["Y"] = y
                o = {k: x.detach() for k, x in o.items()}
                if train:
                    loss = (y * t["dH"][b, hs]).sum()
                    if "dCn" in t:
                        loss = loss + (Cn * t["dCn"][b, hs]).sum()
                    loss.backward()
                    names = {"q": "dq", "k": "dk", "v": "dv", "i_pre": "d_i_pre", "f_pre": "d_f_pre", "o_pre": "do_pre",
                             "gamma": "dgamma", "beta": "dbeta"}
                    if c["state"]:
                        names["C0"] = "dC0"
                    for k, g in names.items():
                        if k in leaf:
                            o[g] = leaf[k].grad if leaf[k].grad is not None else torch.zeros_like(leaf[k])
            parts.append((b, o))
    out = {}
    for key in parts[0][1]:
        rows = [torch.cat([o[key] for bb, o in parts if bb == b]) for b in range(B)]
        out[key] = sum(rows) if key in ("dgamma", "dbeta") else torch.stack(rows)
    if step:
        r = {"h": out["H"][:, :, 0], "C": out["Cn"], "n": out["nn"], "m": out["mn"]}
        if layer:
            r["y"] = out["Y"][:, :, 0]
        return r
    return out
