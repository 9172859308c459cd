"""Performance cases of the decode layer: one token-phase step through the public binding.

Every case is what a serving loop does once per layer and token: the packed
weights, the layer handle, the static KV caches and the new token's
activations are in hand, and one call of ``Layer.step`` (or ``step_kv8`` over
an 8-bit cache) produces the layer's output and appends the new K and V. The
shapes are the ones this repository's workloads, sweeps and tests name: the
tiny layer, Phi-3-mini, and the Llama3.2-1B-, Llama2-7B- and Llama3-8B-like
layers, and for the drawn cases also generic layers of the same kind.

A case is a dict of plain values:
  hidden, heads, kv_heads, head_dim, inter, rope_base   the layer's shape
  batch, max_batch   sequences of the step, and those the handle is made for
  lo, hi             the sequences' cached entries, spread over [lo, hi]
  kv                 "bf16", "fp8_e4m3" or "int8": what the caches hold
  layers             layers of the call (more than one: each reads the output
                     of the one before, with weights and caches of its own)
"""
from __future__ import annotations

import math

import torch

from paper_2607_11211_amd import layer as L
from paper_2607_11211_amd.configs import LayerConfig

EPS = 1e-5

# hidden, query heads, KV heads, head dim, MLP width, RoPE base
TINY = (256, 4, 4, 64, 688, 1e4)
LLAMA32_1B = (2048, 32, 32, 64, 8192, 1e4)
PHI3 = (3072, 32, 32, 96, 8192, 1e4)
LLAMA2_7B = (4096, 32, 32, 128, 11008, 1e4)
LLAMA3_8B = (4096, 32, 8, 128, 14336, 5e5)


def _case(name, shape, batch, lo, hi=None, kv="bf16", layers=1, max_batch=None):
    d = dict(hidden=shape[0], heads=shape[1], kv_heads=shape[2], head_dim=shape[3], inter=shape[4],
             rope_base=shape[5], batch=batch, max_batch=max_batch or batch, lo=lo, hi=lo if hi is None else hi,
             kv=kv, layers=layers)
    return dict(d, name=name) if name else d


def listed():
    return [
        # the smallest call: a layer of 1.7 MB of weights, where launches and latency are all there is
        _case("tiny_b1_kv128", TINY, 1, 128),
        # one user of a small model
        _case("llama32_1b_b1_kv2048", LLAMA32_1B, 1, 2048),
        # one user of a Phi-3-mini layer with a short history
        _case("phi3_b1_kv1024", PHI3, 1, 1024),
        # a whole call: consecutive layers of a Phi-3-mini stack, 4096 cached tokens each
        _case("phi3_stack8_b1_kv4096", PHI3, 1, 4096, layers=8),
        # one user with a long document: the attention outweighs the weights
        _case("phi3_b1_kv32768", PHI3, 1, 32768),
        # one user of an 8B model with grouped queries, an odd number of cached tokens
        _case("llama3_8b_b1_kv8191", LLAMA3_8B, 1, 8191),
        # three users of a 7B model on a handle made for four, with short and long histories
        _case("llama2_7b_b3_ragged", LLAMA2_7B, 3, 65, 2500, max_batch=4),
        # long-context serving with grouped queries
        _case("llama3_8b_b4_kv32768", LLAMA3_8B, 4, 32768),
        # the ragged serving batch
        _case("phi3_b16_ragged", PHI3, 16, 512, 4096),
        # the same batch with an FP8 cache
        _case("phi3_b16_ragged_fp8", PHI3, 16, 512, 4096, kv="fp8_e4m3"),
        # a larger batch of an 8B model with an INT8 cache
        _case("llama3_8b_b32_ragged_int8", LLAMA3_8B, 32, 256, 8192, kv="int8"),
        # the largest batch a handle takes
        _case("phi3_b64_ragged", PHI3, 64, 512, 4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _generic(rng):
    """A layer of the usual proportions and of no model in particular."""
    d = rng.choice((64, 96, 128))
    group = rng.choice((1, 2, 4))
    kv_heads = rng.randint(1, 8192 // d // group // 2)
    heads = group * kv_heads
    hidden = 8 * max(8, int(heads * d * rng.uniform(0.6, 1.25)) // 8)
    inter = 8 * int(hidden * rng.uniform(2.0, 4.0) / 8)
    return (min(hidden, 8192), heads, kv_heads, d, min(inter, 32768), rng.choice((1e4, 5e5)))


def draw(rng):
    shape = rng.choice((TINY, LLAMA32_1B, PHI3, LLAMA2_7B, LLAMA3_8B, None, None)) or _generic(rng)
    kv = rng.choice(("bf16", "bf16", "fp8_e4m3", "int8"))
    batch = _log_int(rng, 1, 64)
    max_batch = next(m for m in (1, 4, 16, 64) if m >= batch)
    lo = hi = _log_int(rng, 16, 32768)
    if batch > 1 and rng.random() < 0.7:
        lo = max(1, int(hi * rng.uniform(0.05, 1.0)))
    # no more cached bytes than the largest listed case reads
    limit = work(listed()[-1])["bytes"] - _weight_elems(*shape[:5]) * 2
    per = 2 * shape[2] * shape[3] * (2 if kv == "bf16" else 1)
    room = int(limit / (per * batch))
    hi = max(1, min(hi, room))
    return _case("", shape, batch, min(lo, hi), hi, kv=kv, max_batch=max_batch)


def _positions(case):
    """Cached entries of each sequence: spread over [lo, hi] in no particular order."""
    n, lo, hi = case["batch"], case["lo"], case["hi"]
    return [lo + int((hi - lo + 1) * (((i + 1) * 0.6180339887498949) % 1.0)) if hi > lo else lo for i in range(n)]


def _weight_elems(hidden, heads, kv_heads, d, inter):
    return hidden * (heads + 2 * kv_heads) * d + hidden * heads * d + 3 * hidden * inter + 2 * hidden


def work(case):
    D, H, G, d, K = (case[k] for k in ("hidden", "heads", "kv_heads", "head_dim", "inter"))
    B, n, w = case["batch"], sum(_positions(case)), _weight_elems(D, H, G, d, K)
    cell = 2 if case["kv"] == "bf16" else 1
    # weights and cached entries once, the new entries, x and y
    nbytes = 2 * w + 2 * G * d * cell * (n + B) + 4 * B * D
    flops = 2 * B * w + 4 * H * d * (n + B)
    return {"bytes": case["layers"] * nbytes, "flops": case["layers"] * flops}


def tolerance(case):
    # y, K and V are rounded once to bf16 from 32-bit sums: a sum that lands on the other side of a
    # rounding boundary moves by one step, at most 2^-7 of its value. 8-bit entries may fall on the
    # neighbouring code. Two orders of the sums (the vector and the matrix-core projections) differ by
    # up to 1.6e-4 in the norm of y, more in narrow layers, and by one step at most; in the stack of 8
    # a moved rounding travels through the layers that follow: 5.4e-3 and 2.4e-2 after the last.
    if case["layers"] > 1:
        return {"rel": 2e-2, "max": 1e-1}
    return {"rel": 2e-3, "max": 3e-2, "differ": 2e-6}


# ---- inputs ---------------------------------------------------------------------------------------

def _generator(seed, salt=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + salt)
    return g


def _normal(gen, shape, scale=1.0, mean=0.0):
    return torch.randn(shape, generator=gen, device="cuda").mul_(scale).add_(mean).to(torch.bfloat16)


def _weights(case, seed, i):
    D, H, G, d, K = (case[k] for k in ("hidden", "heads", "kv_heads", "head_dim", "inter"))
    g = _generator(seed, 10 + i)
    return {
        "attn_norm": _normal(g, (D,), 0.1, 1.0),
        "w_q": _normal(g, (H * d, D), 0.02), "w_k": _normal(g, (G * d, D), 0.02), "w_v": _normal(g, (G * d, D), 0.02),
        "w_o": _normal(g, (D, H * d), 0.02),
        "mlp_norm": _normal(g, (D,), 0.1, 1.0),
        "w_gate": _normal(g, (K, D), 0.02), "w_up": _normal(g, (K, D), 0.02), "w_down": _normal(g, (D, K), 0.02),
    }


def _max_seq(case):
    return case["hi"] + 128


def _caches(case, seed, i):
    """K and V of one layer: random entries up to each sequence's length, zeros beyond."""
    B, G, d, N = case["batch"], case["kv_heads"], case["head_dim"], _max_seq(case)
    g = _generator(seed, 5000 + i)
    out = []
    for _ in range(2):
        if case["kv"] == "bf16":
            c = torch.zeros((B, G, N, d), dtype=torch.bfloat16, device="cuda")
        else:
            c = torch.zeros((B, G, N, d), dtype=torch.uint8, device="cuda")
        for b, n in enumerate(_positions(case)):
            if case["kv"] == "bf16":
                c[b, :, :n] = torch.randn((G, n, d), generator=g, device="cuda").to(torch.bfloat16)
            elif case["kv"] == "int8":
                # values of about one unit in the last 7 bits: a scale of 1/32 spans +-4
                v = torch.randn((G, n, d), generator=g, device="cuda").mul_(32.0).round_().clamp_(-127, 127)
                c[b, :, :n] = v.to(torch.int8).view(torch.uint8)
            else:
                v = torch.randn((G, n, d), generator=g, device="cuda").mul_(64.0).clamp_(-448, 448)
                c[b, :, :n] = v.to(torch.float8_e4m3fn).view(torch.uint8)
        out.append(c)
    return out


def _scales(case, seed):
    """Per-KV-head scales of an 8-bit cache (host), about what its codes above stand for."""
    g = torch.Generator()
    g.manual_seed(int(seed) * 1000003 + 7)
    unit = 1 / 32 if case["kv"] == "int8" else 1 / 64
    return [((0.75 + 0.5 * torch.rand(case["kv_heads"], generator=g)) * unit).tolist() for _ in range(2)]


def prepare(case, seed):
    cfg = LayerConfig(name="perf", index=0, batch=case["batch"], hidden=case["hidden"], n_heads=case["heads"],
                      n_kv_heads=case["kv_heads"], head_dim=case["head_dim"], intermediate=case["inter"],
                      rope_base=case["rope_base"], max_seq=_max_seq(case), pos=tuple(_positions(case)), rms_eps=EPS)
    lay = L.Layer(cfg, max_batch=case["max_batch"])
    stack = []
    for i in range(case["layers"]):
        kc, vc = _caches(case, seed, i)
        x = torch.empty((case["batch"], case["hidden"]), dtype=torch.bfloat16, device="cuda")
        stack.append((lay.pack(_weights(case, seed, i)), kc, vc, x))
    state = {"layer": lay, "stack": stack, "x": _normal(_generator(seed, 1), (case["batch"], case["hidden"])),
             "pos": list(cfg.pos), "kv": case["kv"]}
    if case["kv"] != "bf16":
        state["k_scale"], state["v_scale"] = _scales(case, seed)
    return state


def run(state):
    """One step: the layers' outputs and the caches with their new entries."""
    lay, pos, x = state["layer"], state["pos"], state["x"]
    for w, kc, vc, y in state["stack"]:
        if state["kv"] == "bf16":
            lay.step(w, x, pos, kc, vc, y)
        else:
            lay.step_kv8(w, state["kv"], x, pos, kc, vc, state["k_scale"], state["v_scale"], y)
        x = y
    return [{"y": y, "k_cache": kc, "v_cache": vc} for _, kc, vc, y in state["stack"]]


# ---- the same step in 64 bits ------------------------------------------------------------------------

def _rms(x, gain):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * gain


def _project(x, w):
    return (w.double() @ x.T).T


def _to_code(v, kv):
    """v rounded once to the 8-bit format's values (nearest, ties to even, saturating)."""
    if kv == "int8":
        return v.round().clamp(-127, 127)
    a = v.abs().clamp(max=448.0)
    quantum = torch.exp2(torch.floor(torch.log2(a.clamp(min=2.0 ** -6))) - 3)
    return torch.sign(v) * ((a / quantum).round() * quantum).clamp(max=448.0)


def exact(case, seed):
    H, G, d, B, kv = (case[k] for k in ("heads", "kv_heads", "head_dim", "batch", "kv"))
    pos = _positions(case)
    x = _normal(_generator(seed, 1), (B, case["hidden"])).double()
    ks, vs = ([1.0] * G,) * 2 if kv == "bf16" else _scales(case, seed)
    ks, vs = (torch.tensor(s, dtype=torch.float32, device="cuda").double().view(G, 1) for s in (ks, vs))
    j = torch.arange(d // 2, dtype=torch.float64, device="cuda")
    angle = torch.tensor(pos, dtype=torch.float64, device="cuda")[:, None] * float(case["rope_base"]) ** (-2.0 * j / d)
    cos, sin = torch.cos(angle)[:, None, :], torch.sin(angle)[:, None, :]

    def rope(t):
        a, b = t[..., : d // 2], t[..., d // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    def stored(t, s):
        return t.to(torch.float32).to(torch.bfloat16).double() if kv == "bf16" else _to_code(t / s, kv) * s

    def values(c):
        if kv == "bf16":
            return c.double()
        return c.view(torch.int8).double() if kv == "int8" else c.view(torch.float8_e4m3fn).double()

    out = []
    for i in range(case["layers"]):
        w = _weights(case, seed, i)
        kc, vc = _caches(case, seed, i)
        h = _rms(x, w["attn_norm"].double())
        q = rope(_project(h, w["w_q"]).view(B, H, d))
        k = rope(_project(h, w["w_k"]).view(B, G, d))
        v = _project(h, w["w_v"]).view(B, G, d)
        o = torch.empty((B, H * d), dtype=torch.float64, device="cuda")
        for b, n in enumerate(pos):
            for g in range(G):
                K = torch.cat([values(kc[b, g, :n]) * ks[g], stored(k[b, g], ks[g])[None]])
                V = torch.cat([values(vc[b, g, :n]) * vs[g], stored(v[b, g], vs[g])[None]])
                qg = q[b].view(G, H // G, d)[g]
                p = torch.softmax(qg @ K.T.contiguous() / math.sqrt(d), -1)
                o[b].view(G, H // G, d)[g] = p @ V
        h1 = x + _project(o, w["w_o"])
        h2 = _rms(h1, w["mlp_norm"].double())
        gate, up = _project(h2, w["w_gate"]), _project(h2, w["w_up"])
        y = h1 + _project(gate * torch.sigmoid(gate) * up, w["w_down"])
        if kv == "bf16":
            kc, vc = kc.double(), vc.double()
            for b, n in enumerate(pos):
                kc[b, :, n], vc[b, :, n] = k[b], v[b]
            out.append({"y": y, "k_cache": kc, "v_cache": vc})
        else:
            out.append({"y": y, "k_cache": None, "v_cache": None})
        x = y.to(torch.float32).to(torch.bfloat16).double()  # the next layer reads the rounded output
    return out
