"""The calls whose speed is measured: what one speculation round of a serving
program asks of the library, through its Python entry points.

A case is a plain dict; "kind" names the entry point, the rest its sizes:

  attn      wf_verify_attn / wf_verify_attn_tree of one layer
  prefill   wf_kv_only_prefill (layers == 1) / wf_kv_only_prefill_layers
  lmhead    wf_lmhead_accept_entropy / _accept_tree / _accept_route_neural,
            over LM-head weights or over given logits
  forward   wf_drafter_forward: a drafter layer over a few tokens
  catchup   wf_drafter_catchup: the lazy catch-up of a drafter switch
  step_f32  the fp32 verify step: prefill, attention and LM head of one layer

Workspaces, outputs and tiled weights are made once in prepare(), as a
serving loop makes them once.  Inputs follow the distributions of the
repository's synthetic workloads: layer inputs and final hidden states
N(0, 1), weights N(0, 0.02), queries and cached K/V N(0, 0.02 sqrt(hidden)).
"""
import math

import torch

import paper_2606_07710_amd as wf

BF16, F32, F64 = torch.bfloat16, torch.float32, torch.float64
DEV = "cuda"
VOCAB = 151936


# ---- the cases ---------------------------------------------------------------

def _attn(name, gamma, ctx, hq=32, hkv=8, dh=128, tree=False):
    return {"name": name, "kind": "attn", "gamma": gamma, "ctx": ctx, "hq": hq,
            "hkv": hkv, "dh": dh, "tree": tree}


def _prefill(name, n, layers=1, d=4096, hkv=8, dh=128, start=4096, tiled=True):
    return {"name": name, "kind": "prefill", "n": n, "layers": layers, "d": d,
            "hkv": hkv, "dh": dh, "start": start, "tiled": tiled}


def _lmhead(name, gamma, d, vocab=VOCAB, tiled=True, accept="chain", source="weights"):
    return {"name": name, "kind": "lmhead", "gamma": gamma, "d": d, "vocab": vocab,
            "tiled": tiled, "accept": accept, "source": source}


def _drafter(name, kind, n, pos, d=4096, hq=32, hkv=8, dh=128, inter=12288, tiled=True):
    return {"name": name, "kind": kind, "n": n, "pos": pos, "d": d, "hq": hq, "hkv": hkv,
            "dh": dh, "inter": inter, "tiled": tiled}


def listed():
    return [
        # a short chat: an autoregressive chain of 8 over about a thousand
        # tokens (8B attention shapes) -- the smallest attention calls
        _attn("attn-chain8-1k", 8, 1003),
        # a long document: the diffusion drafter's block of 16 over 32K tokens
        _attn("attn-block16-32k", 16, 32768),
        # an EAGLE-3-shaped draft tree (root and 60 nodes) over 8K tokens
        _attn("attn-tree61-8k", 61, 8192, tree=True),
        # the largest attention: 32B shapes, 64K tokens
        _attn("attn-block16-64k-32b", 16, 65536, hq=64),
        # one round's tokens appended to a layer's cache (every round, each layer)
        _prefill("prefill-16", 16),
        # a long backlog of one layer: a thousand tokens since the last switch
        _prefill("prefill-1k", 1013, tiled=False),
        # the typical switch backlog (80-90 tokens) through all 36 layers
        _prefill("prefill-80-36layers", 80, layers=36),
        # the LM head of a block of 16: the round's largest single call
        _lmhead("lmhead-block16", 16, 4096),
        # the LM head of a draft tree on the 2560-wide model, weights as loaded
        _lmhead("lmhead-tree61-2560", 61, 2560, tiled=False, accept="tree"),
        # a drafter layer over a block of 16 tokens
        _drafter("forward-16", "forward", 16, 4096),
        # a drafter switch: 80 backlog tokens on a cache of 4096 rows
        _drafter("catchup-80", "catchup", 80, 4096),
        # the whole fp32 step at the repository's smallest configuration
        {"name": "step-f32-tiny", "kind": "step_f32", "hidden": 512, "hq": 8, "hkv": 2,
         "dh": 64, "ctx": 256, "gamma": 8, "n": 4, "vocab": 4096},
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, even over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("attn", "attn", "attn", "prefill", "prefill", "lmhead", "lmhead",
                       "forward", "catchup", "step_f32"))
    if kind == "attn":
        hq, hkv, dh = rng.choice(((32, 8, 128), (32, 8, 128), (64, 8, 128), (24, 8, 128),
                                  (16, 8, 128), (32, 8, 64)))
        gamma = _log(rng, 1, 64)
        c = _attn("", gamma, _log(rng, 100, 65536), hq, hkv, dh,
                  tree=gamma > 4 and rng.random() < 0.4)
    elif kind == "prefill":
        d, hkv, dh = rng.choice(((4096, 8, 128), (4096, 8, 128), (5120, 8, 128),
                                 (2560, 8, 128), (2048, 8, 64)))
        many = rng.random() < 0.35
        c = _prefill("", _log(rng, 1, 200 if many else 4096), rng.randint(2, 36) if many else 1,
                     d, hkv, dh, _log(rng, 1, 32768) - 1, rng.random() < 0.6)
    elif kind == "lmhead":
        d = rng.choice((4096, 4096, 5120, 2560, 2880))
        accept = rng.choice(("chain", "chain", "tree", "neural"))
        if accept == "neural" and d == 2880:      # its d/8 units are no multiple of 16
            accept = "chain"
        gamma = _log(rng, 1, 64)
        given = accept != "neural" and rng.random() < 0.2
        fits = d % 512 == 0 and (accept != "neural" or (gamma <= 16 and d >= 4096))
        c = _lmhead("", gamma, d, _log(rng, 32000, VOCAB if d <= 4096 else 120000),
                    not given and fits and rng.random() < 0.6, accept,
                    "logits" if given else "weights")
    elif kind in ("forward", "catchup"):
        d, hq, inter = rng.choice(((4096, 32, 12288), (4096, 32, 14336), (2560, 32, 9728),
                                   (5120, 64, 8192)))
        n = _log(rng, 1, 64) if kind == "forward" else _log(rng, 1, 2048)
        c = _drafter("", kind, n, _log(rng, 1, 16384) - 1, d, hq, 8, 128, inter,
                     rng.random() < 0.6)
    else:
        hkv = rng.choice((2, 4))
        c = {"name": "", "kind": kind, "hidden": 128 * rng.randint(2, 8),
             "hq": hkv * rng.choice((1, 2, 4)), "hkv": hkv, "dh": rng.choice((64, 128)),
             "ctx": _log(rng, 16, 1024), "gamma": _log(rng, 1, 16), "n": _log(rng, 1, 16),
             "vocab": _log(rng, 500, 8000)}
    del c["name"]
    return c


# ---- inputs, from the seed alone ------------------------------------------------

class _Rand:
    def __init__(self, seed):
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(int(seed) % (1 << 62))

    def normal(self, *shape, std=1.0, dtype=BF16, mean=0.0):
        out = torch.empty(shape, dtype=dtype, device=DEV)
        flat = out.view(-1)
        step = 1 << 28                      # drawn in fp32 pieces of 1 GB at most
        for s in range(0, flat.numel(), step):
            e = min(flat.numel(), s + step)
            flat[s:e].copy_(torch.empty(e - s, device=DEV).normal_(mean, std, generator=self.gen))
        return out

    def ints(self, hi, *shape):
        return torch.randint(0, hi, shape, generator=self.gen, device=DEV, dtype=torch.int32)

    def unit(self, n):
        return torch.rand(n, generator=self.gen, device=DEV).tolist()


def _tree(r, gamma):
    """Parents of a random draft tree: every node's parent is one of the ten
    or so nodes before it, so depths resemble a top-k expansion."""
    u = r.unit(gamma)
    return [-1] + [max(0, i - 1 - int(u[i] * min(i, 10))) for i in range(1, gamma)]


def _masks(parents):
    rows = []
    for i, p in enumerate(parents):
        rows.append((rows[p] if i else 0) | (1 << i))
    return rows


def _inputs(c, seed):
    """The case's tensors, weights row-major, as a dict."""
    r, k, t = _Rand(seed), c["kind"], {}
    if k == "attn":
        s = 0.02 * math.sqrt(4096)
        cap = c["ctx"] + c["gamma"] + 64
        t["q"] = r.normal(c["gamma"], c["hq"], c["dh"], std=s)
        t["k"] = r.normal(c["hkv"], cap, c["dh"], std=s)
        t["v"] = r.normal(c["hkv"], cap, c["dh"], std=s)
        t["masks"] = _masks(_tree(r, c["gamma"])) if c["tree"] else None
    elif k == "prefill":
        L, kd, cap = c["layers"], c["hkv"] * c["dh"], c["start"] + c["n"] + 16
        t["x"] = r.normal(L, c["n"], c["d"])
        t["wk"] = r.normal(L, kd, c["d"], std=0.02)
        t["wv"] = r.normal(L, kd, c["d"], std=0.02)
        t["kc"] = torch.zeros(L, c["hkv"], cap, c["dh"], dtype=BF16, device=DEV)
        t["vc"] = torch.zeros_like(t["kc"])
    elif k == "lmhead":
        g, v, m = c["gamma"], c["vocab"], c["d"] // 8
        if c["source"] == "logits":
            # half of the rows peaked, half of them flat
            t["logits"] = r.normal(g, v, dtype=F32)
            t["logits"] *= torch.where(torch.arange(g, device=DEV) % 2 == 0, 8.0, 0.5)[:, None]
            z = t["logits"]
        else:
            t["h"] = r.normal(g, c["d"])
            t["w"] = r.normal(v, c["d"], std=0.02)
            z = _logits(t["h"], t["w"], F32)
        am = z.argmax(1).to(torch.int32)
        # the drafter's tokens: right with probability 0.7
        u = torch.tensor(r.unit(g), device=DEV)
        guess = r.ints(v, g)
        if c["accept"] == "tree":
            par = _tree(r, g)
            t["parents"] = torch.tensor(par, dtype=torch.int32, device=DEV)
            t["tokens"] = torch.where(u < 0.7, am[t["parents"].long().clamp(min=0)], guess)
        else:
            t["draft"] = torch.where(u < 0.7, am, guess)[: g - 1].contiguous() if g > 1 else None
        if c["accept"] == "neural":
            t["w1"] = r.normal(m, c["d"], std=0.02)
            t["b1"], t["w2"] = r.normal(m, std=0.02), r.normal(m, std=0.05)
            t["b2"] = r.normal(1, std=0.05)
    elif k in ("forward", "catchup"):
        qd, kd, d, i = c["hq"] * c["dh"], c["hkv"] * c["dh"], c["d"], c["inter"]
        cap = c["pos"] + c["n"] + 16
        t["r"] = r.normal(c["n"], d)
        t["kc"] = r.normal(c["hkv"], cap, c["dh"], std=0.02 * math.sqrt(d))
        t["vc"] = r.normal(c["hkv"], cap, c["dh"], std=0.02 * math.sqrt(d))
        shapes = {"w_q": (qd, d), "w_k": (kd, d), "w_v": (kd, d), "w_o": (d, qd),
                  "w_gate": (i, d), "w_up": (i, d), "w_down": (d, i)}
        t["layer"] = {n: r.normal(*s, std=0.02) for n, s in shapes.items()}
        for n in ("attn_norm", "mlp_norm"):
            t["layer"][n] = r.normal(d, mean=1.0, std=0.1)
    else:
        kw = {"std": 0.02, "dtype": F32}
        d, hkv, dh, g, n = c["hidden"], c["hkv"], c["dh"], c["gamma"], c["n"]
        t["q"] = r.normal(g, c["hq"], dh, **kw)
        t["k"] = r.normal(hkv, c["ctx"] + g, dh, **kw)
        t["v"] = r.normal(hkv, c["ctx"] + g, dh, **kw)
        t["x"] = r.normal(n, d, **kw)
        t["wk"], t["wv"] = r.normal(hkv * dh, d, **kw), r.normal(hkv * dh, d, **kw)
        t["kc"] = torch.zeros(hkv, c["ctx"] + n, dh, device=DEV)
        t["vc"] = torch.zeros_like(t["kc"])
        t["h"], t["w"] = r.normal(g, d, **kw), r.normal(c["vocab"], d, **kw)
        am = _logits(t["h"], t["w"], F64).argmax(1).to(torch.int32)
        t["draft"] = am[: g - 1].contiguous() if g > 1 else None
    return t


def _logits(h, w, dtype):
    """h w^T, formed in pieces of the vocabulary."""
    hd = h.to(dtype)
    return torch.cat([hd @ w[s:s + 8192].to(dtype).t() for s in range(0, w.shape[0], 8192)], 1)


def _lm_out(s, g):
    s["argmax"] = torch.zeros(g, dtype=torch.int32, device=DEV)
    s["entropy"] = torch.zeros(g, dtype=F32, device=DEV)
    s["accept"] = torch.zeros(4, dtype=torch.int32, device=DEV)
    s["path"] = torch.zeros(g, dtype=torch.int32, device=DEV)
    s["delta"] = torch.zeros(g, dtype=F32, device=DEV)


def prepare(case, seed):
    c, s = case, _inputs(case, seed)
    s["case"] = c
    k = c["kind"]
    if k == "attn":
        s["out"] = torch.empty_like(s["q"])
        if s["masks"]:
            s["mask"] = torch.tensor([m - (1 << 64) if m >> 63 else m for m in s["masks"]],
                                     dtype=torch.int64, device=DEV)
        need = wf.wf_verify_attn_workspace_bytes(BF16, c["gamma"], c["ctx"], c["hq"], c["hkv"],
                                                 c["dh"])
    elif k == "prefill":
        if c["layers"] == 1:
            for n in ("x", "wk", "wv", "kc", "vc"):
                s[n] = s[n][0]
        if c["tiled"]:
            s["wk"], s["wv"] = wf.tile_weights(s["wk"]), wf.tile_weights(s["wv"])
        code = wf.WF_BF16_TILED if c["tiled"] else wf.WF_BF16
        need = wf.wf_kv_only_prefill_layers_workspace_bytes(code, c["n"], c["d"], c["hkv"],
                                                            c["dh"], c["layers"])
    elif k == "lmhead":
        _lm_out(s, c["gamma"])
        if c["tiled"]:
            s["w"] = wf.tile_weights(s["w"])
            if c["accept"] == "neural":
                s["w1"] = wf.tile_weights(s["w1"])
        if c["accept"] == "neural":
            code = wf.WF_BF16_TILED if c["tiled"] else wf.WF_BF16
            need = int(wf.lib.wf_lmhead_route_neural_workspace_bytes(
                code, c["gamma"], c["vocab"], c["d"], c["d"] // 8))
        else:
            need = wf.wf_lmhead_workspace_bytes(c["gamma"], c["vocab"])
    elif k in ("forward", "catchup"):
        w = s.pop("layer")
        if c["tiled"]:
            w = {n: m if n.endswith("norm") else wf.tile_weights(m) for n, m in w.items()}
        s["layer"] = wf.decoder_layer(w, c["hq"], c["hkv"], 1e-6, 1e6)
        query = (wf.wf_drafter_forward_workspace_bytes if k == "forward"
                 else wf.wf_drafter_catchup_workspace_bytes)
        need = query(s["layer"], c["n"], c["pos"])
        s["out"] = torch.empty(c["n"] if k == "forward" else 1, c["d"], dtype=BF16, device=DEV)
    else:
        _lm_out(s, c["gamma"])
        s["out"] = torch.empty_like(s["q"])
        need = max(wf.wf_verify_attn_workspace_bytes(F32, c["gamma"], c["ctx"], c["hq"],
                                                     c["hkv"], c["dh"]),
                   wf.wf_lmhead_workspace_bytes(c["gamma"], c["vocab"]))
    s["ws"] = wf.alloc_workspace(need, DEV)
    return s


# ---- one pass -----------------------------------------------------------------

def run(s):
    c = s["case"]
    k, ws = c["kind"], s["ws"]
    if k == "attn":
        if s["masks"]:
            return wf.wf_verify_attn_tree(s["q"], s["k"], s["v"], s["out"], c["ctx"], s["mask"],
                                          workspace=ws)
        return wf.wf_verify_attn(s["q"], s["k"], s["v"], s["out"], c["ctx"], workspace=ws)
    if k == "prefill":
        call = wf.wf_kv_only_prefill if c["layers"] == 1 else wf.wf_kv_only_prefill_layers
        call(s["x"], s["wk"], s["wv"], s["kc"], s["vc"], c["start"], 1e6, workspace=ws)
        return _rows(s, c["start"], c["n"])          # the cache rows the call writes
    if k == "lmhead":
        logits = s.get("logits")
        h, w = (None, None) if logits is not None else (s["h"], s["w"])
        if c["accept"] == "tree":
            wf.wf_lmhead_accept_tree(h, w, logits, s["tokens"], s["parents"], 1.0, s["argmax"],
                                     s["entropy"], s["accept"], s["path"], workspace=ws)
        elif c["accept"] == "neural":
            wf.wf_lmhead_accept_route_neural(h, w, s["draft"], s["w1"], s["b1"], s["w2"],
                                             s["b2"], 0.0, s["argmax"], s["entropy"],
                                             s["accept"], s["delta"], workspace=ws)
        else:
            wf.wf_lmhead_accept_entropy(h, w, logits, s["draft"], 1.0, s["argmax"], s["entropy"],
                                        s["accept"], workspace=ws)
        return [s["argmax"], s["entropy"], s["accept"], s["path"], s["delta"]]
    if k == "forward":
        wf.wf_drafter_forward(s["layer"], s["r"], c["pos"], s["kc"], s["vc"], s["out"],
                              workspace=ws)
        return [s["out"]] + _rows(s, c["pos"], c["n"])
    if k == "catchup":
        wf.wf_drafter_catchup(s["layer"], s["r"], c["pos"], s["kc"], s["vc"], s["out"],
                              workspace=ws)
        return [s["out"]] + _rows(s, c["pos"], c["n"])
    wf.wf_kv_only_prefill(s["x"], s["wk"], s["wv"], s["kc"], s["vc"], c["ctx"], 1e4)
    wf.wf_verify_attn(s["q"], s["k"], s["v"], s["out"], c["ctx"], workspace=ws)
    wf.wf_lmhead_accept_entropy(s["h"], s["w"], None, s["draft"], 8.0, s["argmax"], s["entropy"],
                                s["accept"], workspace=ws)
    return [s["out"], s["argmax"], s["entropy"], s["accept"]] + _rows(s, c["ctx"], c["n"])


def _rows(s, start, n):
    """The rows a call wrote in its caches, [...][Hkv][n][D] views."""
    return [s["kc"].narrow(-2, start, n), s["vc"].narrow(-2, start, n)]


# ---- what a pass cannot do without ---------------------------------------------

def _attn_work(c, b):
    g, n = c["gamma"], c["ctx"] + c["gamma"]
    keys = g * c["ctx"] + g * (g + 1) // 2
    return (2 * c["hkv"] * n * c["dh"] * b + 2 * g * c["hq"] * c["dh"] * b,
            4 * c["hq"] * c["dh"] * keys)


def _prefill_work(n, d, kd, b):
    return 2 * kd * d * b + n * d * b + 2 * n * kd * b, 4 * n * d * kd


def work(case):
    c, k = case, case["kind"]
    if k == "attn":
        by, fl = _attn_work(c, 2)
    elif k == "prefill":
        by, fl = _prefill_work(c["n"], c["d"], c["hkv"] * c["dh"], 2)
        by, fl = by * c["layers"], fl * c["layers"]
    elif k == "lmhead":
        g, v, d = c["gamma"], c["vocab"], c["d"]
        if c["source"] == "logits":
            by, fl = g * v * 4, 6 * g * v
        else:
            rows = v + (d // 8 if c["accept"] == "neural" else 0)
            by, fl = (rows + g) * d * 2, 2 * g * rows * d
    elif k in ("forward", "catchup"):
        qd, kd, d, i, n = c["hq"] * c["dh"], c["hkv"] * c["dh"], c["d"], c["inter"], c["n"]
        rows = n if k == "forward" else 1           # tokens that run the whole layer
        rest = 2 * qd * d + 3 * i * d               # weights besides W_k and W_v
        by = 2 * (rest + 2 * kd * d + 2 * d + n * d + rows * d
                  + 2 * kd * n + 2 * kd * c["pos"])
        fl = 4 * n * d * kd + 2 * rows * rest + 4 * c["hq"] * c["dh"] * rows * (c["pos"] + n)
    else:
        by, fl = _attn_work(c, 4)
        pb, pf = _prefill_work(c["n"], c["hidden"], c["hkv"] * c["dh"], 4)
        by += pb + (c["vocab"] + c["gamma"]) * c["hidden"] * 4
        fl += pf + 2 * c["gamma"] * c["vocab"] * c["hidden"]
    return {"bytes": by, "flops": fl}


def tolerance(case):
    """About four times the error measured against 64 bits: attention 2.6e-3
    to 2.9e-3, K/V rows 1.7e-3, a drafter layer's output 3.7e-3 to 5.7e-3 (all
    of it bf16 rounding); entropies 3e-8 to 4e-8 and the predicted gain 1e-7
    to 3e-7 (fp32 sums in another order), the fp32 step 1.6e-7."""
    return {"attn": {"rel": 1.2e-2}, "prefill": {"rel": 7e-3}, "forward": {"rel": 2e-2},
            "catchup": {"rel": 2e-2}, "lmhead": {"rel": 2e-6, "max": 1e-5},
            "step_f32": {"rel": 1e-6, "max": 1e-5}}[case["kind"]]


# ---- the same in 64 bits, plain torch --------------------------------------------

def _rope(x, start, base):
    """Rotate-half RoPE of x [..., n, D] at positions start .. start + n - 1."""
    half = x.shape[-1] // 2
    theta = base ** (-torch.arange(half, dtype=F64, device=DEV) / half)
    pos = torch.arange(start, start + x.shape[-2], dtype=F64, device=DEV)
    cos, sin = torch.cos(pos[:, None] * theta), torch.sin(pos[:, None] * theta)
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], -1)


def _attend(q, k, v, ctx, masks=None):
    """q [g][Hq][D] against k, v [Hkv][n][D]; row i sees the keys below ctx
    and block keys up to its own, or those its mask names."""
    g, hq, dh = q.shape
    per = hq // k.shape[0]
    n = ctx + g
    see = torch.ones(g, n, dtype=torch.bool, device=DEV)
    if masks:
        see[:, ctx:] = torch.tensor([[bool(m >> j & 1) for j in range(g)] for m in masks],
                                    device=DEV)
    else:
        see[:, ctx:] = torch.ones(g, g, dtype=torch.bool, device=DEV).tril()
    out = torch.empty(g, hq, dh, dtype=F64, device=DEV)
    for h in range(hq):
        kh, vh = k[h // per, :n].to(F64), v[h // per, :n].to(F64)
        z = (q[:, h].to(F64) @ kh.t()) / math.sqrt(dh)
        out[:, h] = torch.softmax(z.masked_fill(~see, -math.inf), -1) @ vh
    return out


def _kv(x, wk, wv, hkv, start, base):
    """K (rotated) and V rows [Hkv][n][D] of inputs x [n][d]."""
    def heads(w):
        return (x @ w.to(F64).t()).view(x.shape[0], hkv, -1).transpose(0, 1)
    return _rope(heads(wk), start, base), heads(wv).contiguous()


def _entropy(z):
    p = torch.log_softmax(z, -1)
    return -(p.exp() * p).nan_to_num(0.0).sum(-1)


def exact(case, seed):
    c, k = case, case["kind"]
    t = _inputs(c, seed)
    if k == "attn":
        return _attend(t["q"], t["k"], t["v"], c["ctx"], t["masks"])
    if k == "prefill":
        got = [_kv(t["x"][i].to(F64), t["wk"][i], t["wv"][i], c["hkv"], c["start"], 1e6)
               for i in range(c["layers"])]
        return list(got[0]) if c["layers"] == 1 else [torch.stack(x) for x in zip(*got)]
    if k == "lmhead":
        z = t["logits"].to(F64) if c["source"] == "logits" else _logits(t["h"], t["w"], F64)
        delta = None
        if c["accept"] == "neural":
            u = _logits(t["h"], t["w1"], F64) + t["b1"].to(F64)
            delta = torch.nn.functional.gelu(u) @ t["w2"].to(F64) + t["b2"].to(F64)
        return [z.argmax(1).to(torch.int32), _entropy(z), None, None, delta]
    if k in ("forward", "catchup"):
        w = {n: m.to(F64) for n, m in t["layer"].items()}

        def norm(x, gain):
            return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + 1e-6) * gain

        r, n, pos = t["r"].to(F64), c["n"], c["pos"]
        xn = norm(r, w["attn_norm"])
        kn, vn = _kv(xn, w["w_k"], w["w_v"], c["hkv"], pos, 1e6)
        kc = torch.cat([t["kc"][:, :pos].to(F64), kn], 1)
        vc = torch.cat([t["vc"][:, :pos].to(F64), vn], 1)
        if k == "catchup":                            # the whole layer for the last token
            r, xn, pos = r[-1:], xn[-1:], pos + n - 1
        q = _rope((xn @ w["w_q"].t()).view(-1, c["hq"], c["dh"]).transpose(0, 1), pos, 1e6)
        a = _attend(q.transpose(0, 1), kc, vc, pos).reshape(r.shape[0], -1)
        h1 = r + a @ w["w_o"].t()
        x2 = norm(h1, w["mlp_norm"])
        act = torch.nn.functional.silu(x2 @ w["w_gate"].t()) * (x2 @ w["w_up"].t())
        return [h1 + act @ w["w_down"].t(), kn, vn]
    z = _logits(t["h"], t["w"], F64)
    kn, vn = _kv(t["x"].to(F64), t["wk"], t["wv"], c["hkv"], c["ctx"], 1e4)
    return [_attend(t["q"], t["k"], t["v"], c["ctx"]), z.argmax(1).to(torch.int32),
            _entropy(z), None, kn, vn]
