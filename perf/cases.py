"""Performance cases of the framework: the work a program gives it, through its
public entry points (paper_2503_17707_amd.binding), from one projection of one
token to whole prefills, decodes, adapter switches and a cold start.

Sizes are those of the OPT shapes this repository serves (d_model 2048 ... 9216,
ReLU FFN of 4 d_model, vocab 50272, LoRA ranks 16 and 32), with prompt lengths
and batch sizes spread over what a server meets.  Inputs are drawn on the GPU
from the seed alone: N(0, 0.02) weights and biases, LayerNorm gains 1 + N(0,
0.02), LoRA A ~ N(0, 1/r) and B ~ N(0, 0.02), uniform prompt tokens.
"""
import ctypes
import math

import numpy as np
import torch

from paper_2503_17707_amd import binding as pb

DEV = "cuda:0"
DT = {"bf16": (torch.bfloat16, 0), "f16": (torch.float16, 1)}
VOCAB = 50272
MAX_POS = 2048
BITS = {"q": 1, "k": 2, "v": 4, "o": 8}


def listed():
    return [
        # the q, k, v projection of one decode token at the OPT-1.3B width, as a
        # serving loop that must not allocate calls it: the smallest call
        dict(name="token_qkv", kind="gemm", dtype="f16", epi=0, M=1, N=6144, K=2048, noalloc=True),
        # fc1 of a batched decode step at the OPT-6.7B width
        dict(name="batch_fc1", kind="gemm", dtype="bf16", epi=1, M=24, N=16384, K=4096, noalloc=False),
        # fc2 with the residual for one odd-sized prompt at the OPT-13B width
        dict(name="prompt_fc2", kind="gemm", dtype="f16", epi=2, M=333, N=5120, K=20480, noalloc=False),
        # fc1 of two full-length prompts at the OPT-66B width: the largest product
        dict(name="long_fc1", kind="gemm", dtype="f16", epi=1, M=4096, N=36864, K=9216, noalloc=False),
        # attention of a batch of short chat prompts, head_dim 64
        dict(name="attn_chats", kind="attention", dtype="bf16", B=48, T=77, H=32, hd=64),
        # attention of two full-length prompts at the OPT-66B shape
        dict(name="attn_long", kind="attention", dtype="f16", B=2, T=2048, H=72, hd=128),
        # a pipeline stage: two decoder layers of the OPT-13B shape over one long
        # prompt, rank-32 adapter on q, k, v, o, hidden state in and out
        dict(name="block_13b", kind="stage", dtype="f16", d=5120, H=40, layers=2, B=1, T=2000, rank=32,
             targets="qkvo", adapters=1),
        # time to first token of a short prompt on the resident OPT-1.3B, its adapter on q, v
        dict(name="prefill_short", kind="prefill", dtype="f16", d=2048, H=32, layers=24, B=1, T=61, rank=16,
             targets="qv", adapters=1),
        # one chat turn on the OPT-1.3B: a prompt of 1000 tokens, then 32 decode steps
        dict(name="chat_turn", kind="decode", dtype="f16", d=2048, H=32, layers=24, B=1, T=1000, steps=32, rank=16,
             targets="qv", adapters=1),
        # batched decode with mixed adapters: four layers of the OPT-6.7B shape (every
        # layer of the model does the same), 12 sequences, 24 steps
        dict(name="batch_turn", kind="decode", dtype="bf16", d=4096, H=32, layers=4, B=12, T=300, steps=24, rank=16,
             targets="qkvo", adapters=4),
        # two epochs of the merged OPT-1.3B: switch to one adapter, serve a batch of
        # short prompts, switch to the other, serve again
        dict(name="adapter_switch", kind="switch", dtype="f16", d=2048, H=32, layers=24, B=4, T=64, rank=16,
             targets="qv", adapters=2),
        # cold start of the OPT-1.3B: adapter and every layer from pinned host memory
        # to the first token of a 512-token prompt
        dict(name="cold_start", kind="cold", dtype="f16", d=2048, H=32, layers=24, B=1, T=512, rank=16, targets="qv",
             adapters=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gemm", "gemm", "gemm", "attention", "attention", "stage", "prefill", "decode", "decode",
                       "switch", "cold"])
    dtype = rng.choice(["f16", "bf16"])
    if kind == "gemm":
        d = rng.choice([2048, 4096, 5120, 9216])
        epi = rng.choice([0, 1, 2])
        N, K = {0: (3 * d, d), 1: (4 * d, d), 2: rng.choice([(d, d), (d, 4 * d)])}[epi]
        M = _log(rng, 1, 4096)
        noalloc = rng.random() < 0.3 and M * N * 4 <= 64 << 20
        return dict(kind=kind, dtype=dtype, epi=epi, M=M, N=N, K=K, noalloc=noalloc)
    if kind == "attention":
        H, hd = rng.choice([(32, 64), (32, 128), (40, 128), (72, 128)])
        T = _log(rng, 8, 2048)
        B = _log(rng, 1, max(1, min(64, 4096 // T)))
        return dict(kind=kind, dtype=dtype, B=B, T=T, H=H, hd=hd)
    if kind == "stage":
        d, H = rng.choice([(2048, 32), (4096, 32), (5120, 40)])
        T = _log(rng, 100, 2048)
        B = rng.randint(1, max(1, min(4, 4096 // T)))
        return dict(kind=kind, dtype=dtype, d=d, H=H, layers=2, B=B, T=T, rank=rng.choice([16, 32]),
                    targets=rng.choice(["qv", "qkvo"]), adapters=rng.randint(1, B))
    if kind == "prefill":
        d, H, layers = rng.choice([(2048, 32, 24), (4096, 32, 4)])
        T = _log(rng, 5, 700)
        B = rng.randint(1, max(1, min(4, 1024 // T)))
        return dict(kind=kind, dtype=dtype, d=d, H=H, layers=layers, B=B, T=T, rank=16,
                    targets=rng.choice(["qv", "qkvo"]), adapters=rng.randint(1, B))
    if kind == "decode":
        d, H, layers = rng.choice([(2048, 32, 24), (4096, 32, 4)])
        B = _log(rng, 1, 32)
        T = _log(rng, 16, min(1900, 6000 // B))
        return dict(kind=kind, dtype=dtype, d=d, H=H, layers=layers, B=B, T=T, steps=rng.randint(4, 24), rank=16,
                    targets=rng.choice(["qv", "qkvo"]), adapters=min(B, rng.randint(1, 4)))
    d, H, layers = 2048, 32, rng.choice([8, 12, 24])
    T = _log(rng, 20, 300)
    return dict(kind=kind, dtype=dtype, d=d, H=H, layers=layers, B=rng.randint(1, 4), T=T, rank=rng.choice([16, 32]),
                targets=rng.choice(["qv", "qkvo"]), adapters=2 if kind == "switch" else 1)


# ---- draws -------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, std, dt, mean=0.0):
    x = torch.empty(shape, dtype=torch.float32, device=DEV).normal_(mean, std, generator=g)
    return x if dt is torch.float32 else x.to(dt)


LAYER = ("wq", "wk", "wv", "wo", "w1", "w2", "bq", "bk", "bv", "bo", "b1", "b2", "ln1_g", "ln1_b", "ln2_g", "ln2_b")


def _shape(c, name):
    d, f = c["d"], 4 * c["d"]
    return {"w1": (f, d), "w2": (d, f), "b1": (f,)}.get(name, (d, d) if name in ("wq", "wk", "wv", "wo") else (d,))


def _layer(c, g):
    dt = DT[c["dtype"]][0]
    return {n: _normal(g, _shape(c, n), 0.02, dt, 1.0 if n.endswith("_g") else 0.0) for n in LAYER}


def _globals(c, g):
    dt = DT[c["dtype"]][0]
    return {"embed": _normal(g, (VOCAB, c["d"]), 0.02, dt), "pos": _normal(g, (MAX_POS, c["d"]), 0.02, dt),
            "lnf_g": _normal(g, (c["d"],), 0.02, dt, 1.0), "lnf_b": _normal(g, (c["d"],), 0.02, dt)}


def _adapter_layer(c, g):
    dt, r, d = DT[c["dtype"]][0], c["rank"], c["d"]
    return {t: (_normal(g, (r, d), 1.0 / r, dt), _normal(g, (d, r), 0.02, dt)) for t in c["targets"]}


def _model_draws(c, seed):
    """Globals, layers and adapters of a model, one generator each so that they can be drawn one at a time."""
    return (lambda: _globals(c, _gen(seed * 1000 + 1)), lambda l: _layer(c, _gen(seed * 1000 + 10 + l)),
            lambda a, l: _adapter_layer(c, _gen(seed * 1000 + 100 + 100 * a + l)))


def _tokens(c, seed, n):
    return np.random.default_rng(seed).integers(2, VOCAB, size=(c["B"], n), dtype=np.int32)


def _adapter_of_seq(c):
    """Sequences cycle through the adapters; in a batch of several the last one is served by the base model."""
    a = [b % c["adapters"] for b in range(c["B"])]
    if c["B"] > 2:
        a[-1] = -1
    return a


def _scale(c):
    return 2.0  # alpha = 2 r


# ---- the model a serving program keeps -----------------------------------------

class _Absent:
    """A layer that this GPU does not load."""

    ptr = None

    def free(self):
        pass


def _block(c):
    """Layers the GPU holds: a stage case is the middle stage of a model two layers longer."""
    return range(1, c["layers"] + 1) if c["kind"] == "stage" else range(c["layers"])


class _Blobs:
    """Host blobs of one model in pinned memory, as stream_layers takes them."""

    def __init__(self, c, cfg, seed):
        glob, layer, adapter = _model_draws(c, seed)
        L = pb.lib()
        block = _block(c)
        self.globals = self._blob(L.pb_globals_bytes(ctypes.byref(cfg)),
                                  {n: (pb.globals_tensor(cfg, n), t) for n, t in glob().items()})
        self.layers = [self._blob(L.pb_layer_bytes(ctypes.byref(cfg)),
                                  {n: (pb.layer_tensor(cfg, n), t) for n, t in layer(l).items()})
                       if l in block else _Absent() for l in range(cfg.n_layers)]
        self.mask = sum(BITS[t] for t in c["targets"])
        nb = L.pb_lora_layer_bytes(ctypes.byref(cfg), c["rank"], self.mask)
        self.loras = []
        for a in range(c["adapters"]):
            blobs = []
            for l in range(cfg.n_layers):
                parts = {}
                for t, (A, B) in adapter(a, l).items():
                    parts[t + "A"] = (pb.lora_tensor(cfg, c["rank"], self.mask, t, "A"), A)
                    parts[t + "B"] = (pb.lora_tensor(cfg, c["rank"], self.mask, t, "B"), B)
                blobs.append(self._blob(nb, parts))
            self.loras.append(blobs)

    @staticmethod
    def _blob(nbytes, parts):
        dev = torch.zeros(nbytes // 2, dtype=torch.int16, device=DEV)
        for (off, n), t in parts.values():
            dev[off:off + n] = t.reshape(-1).view(torch.int16)
        host = pb.Pinned(nbytes)
        torch.from_numpy(host.view(np.int16)).copy_(dev)
        return host

    def free(self):
        for b in [self.globals] + self.layers + [x for bl in self.loras for x in bl]:
            b.free()


def _make_model(c, seed, steps=0, shadow=False):
    n_layers = c["layers"] + (2 if c["kind"] == "stage" else 0)
    cfg = pb.Config(n_layers=n_layers, d_model=c["d"], n_heads=c["H"], d_ffn=4 * c["d"], vocab=VOCAB,
                    max_pos=MAX_POS, max_tokens=c["B"] * c["T"], max_batch=c["B"], max_adapters=c["adapters"],
                    max_rank=c["rank"], dtype=DT[c["dtype"]][1], ln_eps=1e-5, max_new_tokens=steps,
                    merge_shadow=1 if shadow else 0)
    blobs = _Blobs(c, cfg, seed)
    return pb.Model(cfg, DEV), blobs


def _load(c, m, blobs):
    for a, bl in enumerate(blobs.loras):
        m.attach_lora(a, bl, c["rank"], 2.0 * c["rank"], blobs.mask)
    m.stream_layers(blobs, _block(c))


def prepare(case, seed):
    c, seed = case, int(seed)
    if c["kind"] == "gemm":
        dt, code = DT[c["dtype"]]
        M, N, K, epi = c["M"], c["N"], c["K"], c["epi"]
        g = _gen(seed)
        X = _normal(g, (M, K), 1.0, dt)  # LayerNorm output; fc2 reads fc1's ReLU output
        if epi == 2 and K > N:
            X = X.relu_()
        s = {"case": c, "code": code, "X": X, "W": _normal(g, (N, K), 0.02, dt), "b": _normal(g, (N,), 0.02, dt)}
        if epi == 2:
            s["R0"] = _normal(g, (M, N), 1.0, torch.float32)
            s["out"] = torch.empty((M, N), dtype=torch.float32, device=DEV)
        else:
            s["out"] = torch.empty((M, N), dtype=dt, device=DEV)
        s["ws"] = None if c["noalloc"] else torch.empty(
            min(1 << 30, max(64 << 20, 16 * M * N)), dtype=torch.uint8, device=DEV)
        return s
    if c["kind"] == "attention":
        dt, code = DT[c["dtype"]]
        g = _gen(seed)
        B, T, H, hd = c["B"], c["T"], c["H"], c["hd"]
        qkv = torch.empty((B * T, 3 * H * hd), dtype=torch.float32, device=DEV).normal_(0.0, 1.3, generator=g)
        qkv[:, :H * hd] /= math.sqrt(hd)
        return {"case": c, "code": code, "qkv": qkv.to(dt), "out": torch.empty((B * T, H * hd), dtype=dt, device=DEV)}
    steps = c.get("steps", 0)
    m, blobs = _make_model(c, seed, steps=steps, shadow=c["kind"] == "switch")
    s = {"case": c, "m": m, "adapters": _adapter_of_seq(c), "tokens": _tokens(c, seed, c["T"] + steps)}
    if c["kind"] == "cold":
        s["blobs"] = blobs
        return s
    _load(c, m, blobs)
    m.load_stats()
    torch.cuda.synchronize()
    blobs.free()
    if c["kind"] == "stage":
        s["x"] = _normal(_gen(seed * 1000 + 7), (c["B"] * c["T"], c["d"]), 0.5, torch.float32)
        s["y"] = torch.empty_like(s["x"])
        torch.cuda.synchronize()
    return s


def run(state):
    s = state
    c = s["case"]
    if c["kind"] == "gemm":
        kw = dict(qscale=0.125, qcols=c["K"]) if c["epi"] == 0 else {}
        if c["epi"] == 2:
            s["out"].copy_(s["R0"])  # the residual stream the product is added to
            kw["R"] = s["out"]
        else:
            kw["C"] = s["out"]
        if c["noalloc"]:
            pb.op_gemm_noalloc(s["code"], c["epi"], s["X"], s["W"], s["b"], **kw)
        else:
            pb.op_gemm(s["code"], c["epi"], s["X"], s["W"], s["b"], workspace=s["ws"], **kw)
        return s["out"]
    if c["kind"] == "attention":
        pb.op_attention(s["code"], s["qkv"], s["out"], c["B"], c["T"], c["H"], c["hd"])
        return s["out"]
    m, toks, ad = s["m"], s["tokens"], s["adapters"]
    if c["kind"] == "stage":
        m.prefill_stage(toks, ad, 1, c["layers"] + 1, hidden_in=s["x"], hidden_out=s["y"])
        return s["y"]
    if c["kind"] == "decode":
        # the prompt, then known continuation tokens one by one; the last step's logits
        T, n = c["T"], c["steps"]
        out = [m.prefill(toks[:, :T], ad, want_logits=False)[0]]
        for i in range(n):
            tok, logits = m.decode(toks[:, T + i], ad, want_logits=i == n - 1)
            out.append(tok)
        return {"tokens": np.stack(out), "logits": logits}
    if c["kind"] == "switch":
        out = {}
        for a in range(2):
            m.merge_lora(a)
            out["logits%d" % a] = m.prefill(toks, None)[1]
        return out
    if c["kind"] == "cold":
        _load(c, m, s["blobs"])
    tok, logits = m.prefill(toks, ad)
    return {"tokens": tok, "logits": logits}


# ---- what a pass cannot do without ----------------------------------------------

def _layer_work(c, rows, ctx, lora_rows):
    """Bytes of weights and flops of one layer over `rows` tokens; ctx: keys seen, summed over the rows."""
    d = c["d"]
    params = 12 * d * d
    flops = 2.0 * rows * params + 4.0 * d * ctx + 4.0 * lora_rows * c["rank"] * d * len(c["targets"])
    return 2.0 * params + 4.0 * c["adapters"] * c["rank"] * d * len(c["targets"]), flops


def work(case):
    c = case
    if c["kind"] == "gemm":
        M, N, K = c["M"], c["N"], c["K"]
        out = M * N * (8 if c["epi"] == 2 else 2)
        return {"bytes": 2.0 * (M * K + N * K + N) + out, "flops": 2.0 * M * N * K}
    if c["kind"] == "attention":
        B, T, H, hd = c["B"], c["T"], c["H"], c["hd"]
        return {"bytes": 8.0 * B * T * H * hd, "flops": 2.0 * B * H * hd * T * (T + 1)}
    B, T, d, L = c["B"], c["T"], c["d"], c["layers"]
    n = B * T
    served = sum(1 for a in _adapter_of_seq(c) if a >= 0) if c["kind"] != "switch" else 0
    wb, fl = _layer_work(c, n, B * T * (T + 1) / 2.0, served * T)
    head_b, head_f = 2.0 * VOCAB * d + 4.0 * B * VOCAB, 2.0 * B * VOCAB * d
    if c["kind"] == "stage":
        return {"bytes": L * wb + 8.0 * n * d, "flops": L * fl}
    one = {"bytes": L * wb + 2.0 * n * d + head_b, "flops": L * fl + head_f}
    if c["kind"] == "decode":
        for i in range(c["steps"]):
            sb, sf = _layer_work(c, B, B * (T + i + 1.0), served)
            one["bytes"] += L * (sb + 4.0 * d * B * (T + i + 1)) + 2.0 * VOCAB * d
            one["flops"] += L * sf + head_f
        one["bytes"] += L * 4.0 * d * n  # the prompt's keys and values
    if c["kind"] == "switch":
        # per switch: the unmerged targets read, the merged ones written
        one = {"bytes": 2 * (one["bytes"] + L * len(c["targets"]) * 4.0 * d * d),
               "flops": 2 * (one["flops"] + L * len(c["targets"]) * 2.0 * d * d * c["rank"])}
    return one


def tolerance(case):
    """Relative errors measured against `exact` over cases and seeds of each kind, times about four."""
    c = case
    if c["kind"] == "gemm":
        # the fp32 residual output shows the accumulation alone, the others one rounding to dt
        return {"rel": 2e-6 if c["epi"] == 2 else {"f16": 9e-4, "bf16": 7e-3}[c["dtype"]]}
    if c["kind"] == "attention":  # probabilities and outputs rounded to dt
        return {"rel": {"f16": 1.2e-3, "bf16": 8e-3}[c["dtype"]]}
    # activations rounded to dt between the kernels, layer after layer
    rel = {"f16": 3e-3, "bf16": 2.4e-2}[c["dtype"]]
    if c["kind"] in ("stage", "switch"):
        return {"rel": rel}
    return {"rel": rel, "differ": 0.1}  # a token of two nearly equal logits may differ


# ---- the same in 64 bits -----------------------------------------------------------

def _ln64(x, g, b):
    mu = x.mean(-1, keepdim=True)
    var = ((x - mu) ** 2).mean(-1, keepdim=True)
    return (x - mu) / torch.sqrt(var + 1e-5) * g.double() + b.double()


def _attention64(q, k, v, B, T, H):
    """q already divided by sqrt(head_dim); [B*T, d] each."""
    hd = q.shape[1] // H
    out = torch.empty_like(q)
    mask = torch.ones((T, T), dtype=torch.bool, device=q.device).triu(1)
    per = max(1, (1 << 28) // (T * T))  # heads at a time
    for b in range(B):
        rows = slice(b * T, (b + 1) * T)
        qh, kh, vh = (x[rows].reshape(T, H, hd).transpose(0, 1).contiguous() for x in (q, k, v))
        for h in range(0, H, per):
            s = torch.matmul(qh[h:h + per], kh[h:h + per].transpose(1, 2).contiguous())
            p = torch.softmax(s.masked_fill_(mask, -math.inf), -1)
            out[rows, h * hd:(h + per) * hd] = torch.matmul(p, vh[h:h + per]).transpose(0, 1).reshape(T, -1)
    return out


def _layer64(c, x, w, lora, ad, B, T):
    d, H = c["d"], c["H"]

    def proj(u, t, wn, bn):
        y = u @ w[wn].double().t() + w[bn].double()
        for b, a in enumerate(ad):
            if a >= 0 and t in lora[a]:
                A, Bm = lora[a][t]
                rows = slice(b * T, (b + 1) * T)
                y[rows] += _scale(c) * ((u[rows] @ A.double().t()) @ Bm.double().t())
        return y

    u = _ln64(x, w["ln1_g"], w["ln1_b"])
    q, k, v = proj(u, "q", "wq", "bq") / math.sqrt(d // H), proj(u, "k", "wk", "bk"), proj(u, "v", "wv", "bv")
    x = x + proj(_attention64(q, k, v, B, T, H), "o", "wo", "bo")
    u = _ln64(x, w["ln2_g"], w["ln2_b"])
    h = (u @ w["w1"].double().t() + w["b1"].double()).relu_()
    return x + h @ w["w2"].double().t() + w["b2"].double()


def _model64(c, seed, toks, ad, head_pos):
    """Logits at the positions head_pos of every sequence, [len(head_pos), B, VOCAB]."""
    glob, layer, adapter = _model_draws(c, seed)
    B, T = toks.shape
    gl = glob()
    t = torch.from_numpy(np.ascontiguousarray(toks)).to(DEV).long()
    x = (gl["embed"][t].double() + gl["pos"][:T].double()[None]).reshape(B * T, -1)
    for l in range(c["layers"]):
        x = _layer64(c, x, layer(l), [adapter(a, l) for a in range(c["adapters"])], ad, B, T)
    E = gl["embed"].double()
    z = _ln64(x.reshape(B, T, -1), gl["lnf_g"], gl["lnf_b"])
    return torch.stack([z[:, p].contiguous() @ E.t() for p in head_pos])


def exact(case, seed):
    c, seed = case, int(seed)
    if c["kind"] == "gemm":
        s = prepare(c, seed)
        y = s["X"].double() @ s["W"].double().t() + s["b"].double()
        if c["epi"] == 0:
            y[:, :c["K"]] *= 0.125
            return y
        return y.relu_() if c["epi"] == 1 else y + s["R0"].double()
    if c["kind"] == "attention":
        s = prepare(c, seed)
        d = c["H"] * c["hd"]
        q, k, v = (s["qkv"][:, i * d:(i + 1) * d].double() for i in range(3))
        return _attention64(q, k, v, c["B"], c["T"], c["H"])
    toks, ad = _tokens(c, seed, c["T"] + c.get("steps", 0)), _adapter_of_seq(c)
    if c["kind"] == "stage":
        _, layer, adapter = _model_draws(c, seed)
        x = _normal(_gen(seed * 1000 + 7), (c["B"] * c["T"], c["d"]), 0.5, torch.float32).double()
        for l in _block(c):
            x = _layer64(c, x, layer(l), [adapter(a, l) for a in range(c["adapters"])], ad, c["B"], c["T"])
        return x
    if c["kind"] == "switch":
        return {"logits%d" % a: _model64(c, seed, toks, [a] * c["B"], [c["T"] - 1])[0] for a in range(2)}
    n = c.get("steps", 0)
    lg = _model64(c, seed, toks, ad, range(c["T"] - 1, c["T"] + n))
    tok = lg.argmax(-1).to(torch.int32)
    return {"tokens": tok if c["kind"] == "decode" else tok[0], "logits": lg[-1]}
