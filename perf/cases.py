"""Performance cases of the decode library: what a program that uses it has it do.

Three kinds, each through an entry point a program calls:
  generate   Decoder.generate: prefill of the prompts, then dex_step rounds
             until every sequence holds its tokens (lattice decoding, or plain
             autoregressive decoding with the explored set {L});
  prompt     Decoder.prefill alone: the time to the first token;
  attention  dex_debug_attention_noalloc: one layer's decode attention with its
             split combine, for programs that bring their own layers.

Model shapes, explored sets, width caps, batches and prompt lengths are those
of synth/configs.py and of the GPU tests (the 32-layer model also cut to fewer
layers, as the tests do).  Weights are random with the variances of synth/gen.py,
except the LM head: every token has a few successors with well separated
logits (about 40, 30, 20 ...), as a trained model has, so that a change of
rounding does not decide which token comes next.
"""

from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

from paper_2606_29223_amd import dexlib
from synth import configs

MODELS = {"tiny": "tiny-4L-d128-fp32", "small": "small-12L-d768-bf16", "llama": "llama-32L-d4096-x8-w4"}


# ------------------------------------------------------------------ the cases

def listed():
    def gen(name, model, layers, step, width, batch, prompt, tokens, temperature=0.0):
        return {"name": name, "kind": "generate", "model": model, "layers": layers, "step": step, "width": width,
                "batch": batch, "prompt": prompt, "tokens": tokens, "decs": 1, "temperature": temperature,
                "adapters": False}

    def pre(name, model, layers, batch, prompt):
        return {"name": name, "kind": "prompt", "model": model, "layers": layers, "batch": batch, "prompt": prompt}

    def att(name, batch, keys, rows):
        return {"name": name, "kind": "attention", "dtype": "bf16", "head_dim": 128, "kv_heads": 8, "group": 4,
                "batch": batch, "keys": keys, "rows": rows}

    return [
        # the smallest decode: fp32, uncapped lattice, one short request; launches and latency
        gen("tiny_generate", "tiny", 4, 1, 0, 1, 16, 64),
        # a small model's request: 12 layers, four explored depths, width 4
        gen("small_generate", "small", 12, 3, 4, 1, 128, 64),
        # the headline workload: one request on the 32-layer model, lattice decoding
        gen("llama_generate", "llama", 32, 8, 4, 1, 512, 128),
        # the same model decoding plainly (explored set {L}) after a short ragged prompt
        gen("llama_plain", "llama", 32, 32, 1, 1, 45, 64),
        # a batch of lattices, eight explored depths, width 8: up to 64 rows a stage
        gen("llama_batch_lattice", "llama", 8, 1, 8, 8, 1024, 32),
        # time to first token: a chat turn, a full prompt, a batch of long documents (fewer layers)
        pre("llama_prompt_97", "llama", 4, 1, 97),
        pre("llama_prompt_512", "llama", 4, 1, 512),
        pre("llama_prompt_8x8192", "llama", 2, 8, 8192),
        # prompts of the 12-layer model (head_dim 64), ragged against every tile
        pre("small_prompt_2x1100", "small", 12, 2, 1100),
        # fp32 prompts
        pre("tiny_prompt_4x256", "tiny", 4, 4, 256),
        # one layer's decode attention: a lattice's four rows at short context, and
        # eight sequences at long context with two rows each
        att("attention_1x700", 1, 700, 4),
        att("attention_8x8300", 8, 8300, 2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("generate", "prompt", "prompt", "attention"))
    if kind == "attention":
        dtype = rng.choice(("bf16", "bf16", "bf16", "bf16", "f32"))
        hd = rng.choice((64, 128, 128)) if dtype == "bf16" else rng.choice((32, 64))
        group = rng.choice((1, 2, 4, 4, 8))
        c = {"kind": kind, "dtype": dtype, "head_dim": hd, "kv_heads": rng.choice((4, 8, 12)), "group": group,
             "batch": rng.randint(1, 8), "keys": _log_int(rng, 48, 16000), "rows": rng.randint(1, 8)}
        # the call's fixed scratch holds 63.75 MiB of split partials
        while c["batch"] * c["rows"] * c["kv_heads"] * group * (c["keys"] // 64 + 2) * (hd + 2) * 4 > 63 << 20:
            if c["rows"] > 1:
                c["rows"] -= 1
            elif c["batch"] > 1:
                c["batch"] -= 1
            else:
                c["keys"] = c["keys"] * 3 // 4
        return c
    model = rng.choice(("tiny", "small", "llama", "llama"))
    batch = rng.choice((1, 1, 2, 4, 8))
    if kind == "prompt":
        total = _log_int(rng, 1, {"tiny": 2048, "small": 16384, "llama": 32768}[model])
        return {"kind": kind, "model": model, "layers": {"tiny": 4, "small": 12, "llama": rng.choice((2, 4))}[model],
                "batch": batch, "prompt": max(1, min(8192, total // batch))}
    layers, steps, widths = {"tiny": (4, (1, 2, 4), (0, 4)), "small": (12, (3, 4, 12), (4, 8)),
                             "llama": (rng.choice((4, 8)), (1, 2), (4, 8))}[model]
    step = rng.choice(steps)
    temperature = 1.0 if layers // step <= 4 and rng.random() < 0.25 else 0.0
    return {"kind": kind, "model": model, "layers": layers, "step": step,
            "width": 1 if step == layers else rng.choice(widths), "batch": batch,
            "prompt": _log_int(rng, 1, 1024), "tokens": rng.randint(8, 48), "decs": rng.choice((1, 1, 1, 0)),
            "temperature": temperature, "adapters": step < layers and rng.random() < 0.25}


# ------------------------------------------------------------- inputs on the GPU

def _config(case):
    cfg = configs.get(MODELS[case["model"]], n_layers=case["layers"], batch=case["batch"], prompt_len=case["prompt"])
    step = case.get("step", case["layers"])
    cfg["explored"] = list(range(step, case["layers"] + 1, step))
    cfg["width_cap"] = case.get("width", 1)
    cfg["decs"] = case.get("decs", 1)
    cfg["gen_len"] = case.get("tokens", 1)
    return cfg


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _uniform(g, shape, var, dtype):
    a = math.sqrt(3.0 * var)
    return torch.rand(shape, generator=g, device="cuda").mul_(2 * a).sub_(a).to(dtype)


def _gain(g, n):
    return torch.rand(n, generator=g, device="cuda").mul_(0.1).add_(0.95)


def _weights(cfg, seed):
    """Tensors by the names of dexlib.Decoder."""
    g = _generator(seed)
    dt = torch.bfloat16 if cfg["dtype"] == "bf16" else torch.float32
    d, F, V, hd = cfg["d_model"], cfg["d_ffn"], cfg["vocab"], cfg["head_dim"]
    H, Hkv = cfg["n_heads"], cfg["n_kv_heads"]
    w = {"embed": _uniform(g, (V, d), 9.0, dt), "final_norm": _gain(g, d)}
    # successors: token v follows x with logit about 40 (1 - j / N) if x is v's j-th predecessor
    n = max(len(cfg["explored"]), 2)
    head = torch.zeros((V, d), device="cuda")
    for j in range(n - 1):
        perm = torch.randperm(V, generator=g, device="cuda")
        head += (40.0 / (3.0 * d) * (1.0 - j / n)) * w["embed"][perm].float()
    w["lm_head"] = head.to(dt)
    for l in range(cfg["n_layers"]):
        p = f"layers.{l}."
        w[p + "attn_norm"] = _gain(g, d)
        w[p + "wq"] = _uniform(g, (H * hd, d), 4.0 / d, dt)
        w[p + "wk"] = _uniform(g, (Hkv * hd, d), 4.0 / d, dt)
        w[p + "wv"] = _uniform(g, (Hkv * hd, d), 1.0 / d, dt)
        w[p + "wo"] = _uniform(g, (d, H * hd), 1.0 / (H * hd), dt)
        w[p + "ffn_norm"] = _gain(g, d)
        w[p + "w_gate"] = _uniform(g, (F, d), 1.0 / d, dt)
        w[p + "w_up"] = _uniform(g, (F, d), 1.0 / d, dt)
        w[p + "w_down"] = _uniform(g, (d, F), 1.0 / F, dt)
    return w


def _adapters(cfg, seed):
    g = _generator(seed + 1)
    dt = torch.bfloat16 if cfg["dtype"] == "bf16" else torch.float32
    d = cfg["d_model"]
    m = 2 * d
    out = {}
    for k in range(len(cfg["explored"]) - 1):
        p = f"adapters.{k}."
        out[p + "norm"] = _gain(g, d)
        out[p + "w1"], out[p + "b1"] = _uniform(g, (m, d), 1.0 / d, dt), _uniform(g, (m,), 0.0033, torch.float32)
        out[p + "w2"], out[p + "b2"] = _uniform(g, (d, m), 1.0 / m, dt), _uniform(g, (d,), 0.0033, torch.float32)
        out[p + "alpha"] = torch.full((1,), 0.5, device="cuda")
    return out


def _prompts(cfg, seed):
    return np.random.default_rng(seed).integers(0, cfg["vocab"], (cfg["batch"], cfg["prompt_len"])).astype(np.int32)


class _CacheView:
    """One of a decoder's caches as an array of its GPU; keeps the decoder alive."""

    def __init__(self, dec, ptr, shape, bf16):
        self.dec = dec
        self.__cuda_array_interface__ = {"shape": shape, "typestr": "<i2" if bf16 else "<f4", "data": (ptr, False),
                                         "strides": None, "version": 3}


def _attention_inputs(case, seed):
    g = _generator(seed)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    B, Hkv, hd, H = case["batch"], case["kv_heads"], case["head_dim"], case["kv_heads"] * case["group"]
    rng = np.random.default_rng(seed)
    # committed lengths differ a little between sequences; a row's chain is its
    # ancestor slots and its own, in the cache entries after the committed ones
    nc = [case["keys"] - int(rng.integers(0, min(32, case["keys"] // 2))) for _ in range(B)]
    E = case["keys"] + 32
    seqs, pos, ncs, off, chain = [], [], [], [], []
    for s in range(B):
        slots = case["keys"] + rng.permutation(32)
        for r in range(case["rows"]):
            n = 1 + r % 4
            seqs.append(s), ncs.append(nc[s]), pos.append(nc[s] + n - 1), off.append(len(chain))
            chain += [int(x) for x in slots[: n - 1]] + [int(slots[8 + r])]
    R = len(seqs)
    i32 = lambda v: np.asarray(v, dtype=np.int32)  # noqa: E731
    return {
        "k": torch.randn((B, Hkv, E, hd), generator=g, device="cuda").mul_(2.0).to(dt),
        "v": torch.randn((B, Hkv, E, hd), generator=g, device="cuda").to(dt),
        "q": torch.randn((R, H * hd), generator=g, device="cuda").mul_(2.0),
        "out": torch.zeros((R, H * hd), device="cuda", dtype=dt),
        "seq": i32(seqs), "pos": i32(pos), "nc": i32(ncs), "off": i32(off), "chain": i32(chain), "entries": E,
    }


def prepare(case, seed):
    if case["kind"] == "attention":
        return dict(_attention_inputs(case, seed), case=case)
    cfg = _config(case)
    ad = _adapters(cfg, seed) if case.get("adapters") else None
    dec = dexlib.Decoder(cfg, _weights(cfg, seed), temperature=case.get("temperature", 0.0), seed=seed, adapters=ad)
    N = len(cfg["explored"])
    rows = case["batch"] * (cfg["width_cap"] or 2 ** (N - 1))
    tap = torch.zeros((rows, cfg["vocab"]), device="cuda")
    torch.cuda.synchronize()
    dec.set_logits_tap(tap)
    kp, vp, E = dec.kv_layout()
    bf16 = cfg["dtype"] == "bf16"
    shape = (cfg["n_layers"], cfg["batch"], cfg["n_kv_heads"], E, cfg["head_dim"])
    k, v = (torch.as_tensor(_CacheView(dec, p, shape, bf16), device="cuda") for p in (kp, vp))
    n = cfg["prompt_len"] + cfg["gen_len"] - 1         # committed cache entries after the call
    k, v = ((t.view(torch.bfloat16) if bf16 else t)[:, :, :, :n] for t in (k, v))
    return {"case": case, "dec": dec, "prompts": _prompts(cfg, seed), "tap": tap, "k": k, "v": v}


def run(state):
    case = state["case"]
    if case["kind"] == "attention":
        s = state
        p32 = lambda a: a.ctypes.data_as(ctypes.POINTER(ctypes.c_int32))  # noqa: E731
        st = dexlib.load().dex_debug_attention_noalloc(
            dexlib.DEX_BF16 if case["dtype"] == "bf16" else dexlib.DEX_F32, case["head_dim"],
            case["kv_heads"] * case["group"], case["kv_heads"], case["batch"], s["entries"], s["k"].data_ptr(),
            s["v"].data_ptr(), s["q"].data_ptr(), len(s["seq"]), p32(s["seq"]), p32(s["pos"]), p32(s["nc"]),
            p32(s["off"]), p32(s["chain"]), len(s["chain"]), s["out"].data_ptr(),
            torch.cuda.current_stream().cuda_stream)
        if st != dexlib.DEX_OK:
            raise RuntimeError("dex_debug_attention_noalloc: status %d" % st)
        return s["out"]
    dec = state["dec"]
    if case["kind"] == "prompt":
        dec.prefill(state["prompts"])
        return {"logits": state["tap"], "k": state["k"], "v": state["v"]}
    toks, _ = dec.generate(state["prompts"], case["tokens"])
    return {"tokens": np.asarray(toks, dtype=np.int64), "logits": state["tap"], "k": state["k"], "v": state["v"]}


# ------------------------------------------------------------------ what it takes

def work(case):
    if case["kind"] == "attention":
        es = 2 if case["dtype"] == "bf16" else 4
        R, H = case["batch"] * case["rows"], case["kv_heads"] * case["group"]
        keys, hd = case["keys"], case["head_dim"]
        return {"bytes": 2.0 * case["batch"] * keys * case["kv_heads"] * hd * es + R * H * hd * (4 + es),
                "flops": 4.0 * R * H * keys * hd}
    cfg = _config(case)
    es = 2 if cfg["dtype"] == "bf16" else 4
    L, d, F, V, B, P = cfg["n_layers"], cfg["d_model"], cfg["d_ffn"], cfg["vocab"], cfg["batch"], cfg["prompt_len"]
    hhd, kvd = cfg["n_heads"] * cfg["head_dim"], cfg["n_kv_heads"] * cfg["head_dim"]
    layer = d * (2 * hhd + 2 * kvd + 3 * F)             # weights of one layer
    kv = 2.0 * L * B * kvd * es                         # keys and values of one position
    # the prompt: every layer but the last on every position; the last layer's
    # keys and values everywhere, the rest of it and the head where a token follows
    flops = 2.0 * B * P * ((L - 1) * layer + 2 * d * kvd) + (L - 1) * 2.0 * B * P * P * hhd
    flops += 2.0 * B * (layer - 2 * d * kvd + V * d) + 4.0 * B * P * hhd
    nbytes = es * (L * layer + V * d + B * P * d) + kv * P + 4.0 * B * V
    if case["kind"] == "generate":
        # a round for each further token, and the lattice's fill of N - 1 partial
        # rounds (one full stream of the weights between them, half of it spare)
        rounds = case["tokens"] - 1 + (len(cfg["explored"]) - 1) / 2.0
        nbytes += rounds * (es * (L * layer + V * d) + kv * (P + case["tokens"] / 2.0))
        flops += rounds * B * (2.0 * (L * layer + V * d) + 4.0 * L * hhd * (P + case["tokens"] / 2.0))
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the distance from the 64-bit results (measured: 2.4e-3 for the bf16
    models' caches, which is their own rounding, 1.7e-3 for their logits, 4.6e-3 for the bf16
    attention, whose split records are rounded too; 1.3e-7 in fp32).  max: a few bf16 steps
    of the largest values, or a value whose error sits at the tail."""
    if case["kind"] == "attention":
        return {"rel": 1.5e-2, "max": 0.15} if case["dtype"] == "bf16" else {"rel": 2e-6, "max": 5e-5}
    if case["model"] == "tiny":
        return {"rel": 1e-6, "max": 5e-5, "differ": 0.0}
    return {"rel": 1e-2, "max": 0.15, "differ": 0.0}


# --------------------------------------------------- the same in 64 bits, plain torch

def _rms64(h, gain, eps):
    return h * torch.rsqrt(h.pow(2).mean(-1, keepdim=True) + eps) * gain.double()


def _rope64(x, pos, hd, theta):
    """x [rows, heads * hd]: rotate the pairs (i, i + hd/2) of every head."""
    i = torch.arange(hd // 2, device="cuda", dtype=torch.float64)
    ang = pos.double()[:, None] * theta ** (-2.0 * i / hd)
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    y = x.view(x.shape[0], -1, hd)
    a, b = y[..., : hd // 2], y[..., hd // 2:]
    return torch.cat((a * c - b * s, b * c + a * s), -1).reshape(x.shape)


def _attend64(q, k, v, first):
    """One head: query row i sees keys 0 .. first + i."""
    out = torch.empty((q.shape[0], v.shape[1]), dtype=torch.float64, device="cuda")
    col = torch.arange(k.shape[0], device="cuda")
    for i0 in range(0, q.shape[0], 2048):
        s = (q[i0:i0 + 2048] @ k.T) / math.sqrt(q.shape[1])
        row = torch.arange(i0, i0 + s.shape[0], device="cuda") + first
        s.masked_fill_(col[None] > row[:, None], -math.inf)
        out[i0:i0 + 2048] = torch.softmax(s, -1) @ v
    return out


def _forward64(cfg, w, toks, first, kc, vc):
    """Tokens at positions first .. of one sequence; fills kc, vc [L][Hkv][n][hd] and
    returns the last position's final state."""
    hd, H, Hkv, L, eps = cfg["head_dim"], cfg["n_heads"], cfg["n_kv_heads"], cfg["n_layers"], cfg["rms_eps"]
    n = len(toks)
    pos = torch.arange(first, first + n, device="cuda")
    h = w["embed"][torch.as_tensor(toks, device="cuda", dtype=torch.long)].double()
    for l in range(L):
        g = lambda p: w[f"layers.{l}.{p}"].double()  # noqa: E731, B023
        alpha = cfg["residual_scale"] * (l + 1) / L
        x = _rms64(h, g("attn_norm"), eps)
        q = _rope64(x @ g("wq").T, pos, hd, cfg["rope_theta"])
        k = _rope64(x @ g("wk").T, pos, hd, cfg["rope_theta"])
        v = x @ g("wv").T
        att = torch.empty_like(q)
        for u in range(Hkv):
            kc[l, u, first:first + n] = k[:, u * hd:(u + 1) * hd]
            vc[l, u, first:first + n] = v[:, u * hd:(u + 1) * hd]
        if l == L - 1:                                  # only the last position's state is read on
            h, q, att = h[-1:], q[-1:].contiguous(), att[-1:].contiguous()
        G = H // Hkv
        for u in range(Hkv):
            kk, vv = kc[l, u, :first + n], vc[l, u, :first + n]
            if q.shape[0] == 1:                         # the group's heads as rows, every key seen
                qg = q.view(H, hd)[u * G:(u + 1) * G]
                att.view(H, hd)[u * G:(u + 1) * G] = torch.softmax(qg @ kk.T / math.sqrt(hd), -1) @ vv
                continue
            for c0 in range(u * G * hd, (u + 1) * G * hd, hd):
                att[:, c0:c0 + hd] = _attend64(q[:, c0:c0 + hd], kk, vv, first)
        h = h + alpha * (att @ g("wo").T)
        x = _rms64(h, g("ffn_norm"), eps)
        for i0 in range(0, h.shape[0], 8192):
            gate, up = x[i0:i0 + 8192] @ g("w_gate").T, x[i0:i0 + 8192] @ g("w_up").T
            h[i0:i0 + 8192] += alpha * ((torch.nn.functional.silu(gate) * up) @ g("w_down").T)
    return h[-1:]


_M64 = (1 << 64) - 1


def _mix64(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _gumbel64(seed, seq, pos, V):
    """The Gumbel row of (seed, sequence, position), as include/dex.h defines it."""
    with np.errstate(over="ignore"):
        inner = _mix64(np.array([((seq << 32) + pos) & _M64], dtype=np.uint64))
        key = _mix64(np.array([seed & _M64], dtype=np.uint64) ^ inner)
        z = _mix64(key + np.arange(1, V + 1, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15))
    u = ((z >> np.uint64(41)).astype(np.float64) + 0.5) / 2.0 ** 23
    return torch.from_numpy(-np.log(-np.log(u))).cuda()


def exact(case, seed):
    if case["kind"] == "attention":
        s = _attention_inputs(case, seed)
        hd, G = case["head_dim"], case["group"]
        out = torch.empty(s["q"].shape, dtype=torch.float64, device="cuda")
        for r in range(len(s["seq"])):
            nc, n = int(s["nc"][r]), int(s["pos"][r]) - int(s["nc"][r]) + 1
            ents = list(range(nc)) + [int(x) for x in s["chain"][s["off"][r]:s["off"][r] + n]]
            ents = torch.as_tensor(ents, device="cuda")
            for u in range(case["kv_heads"]):
                k, v = (s[t][int(s["seq"][r]), u][ents].double() for t in ("k", "v"))
                q = s["q"][r].view(-1, hd)[u * G:(u + 1) * G].double()
                p = torch.softmax(q @ k.T / math.sqrt(hd), -1)
                out[r].view(-1, hd)[u * G:(u + 1) * G] = p @ v
        return out
    cfg = _config(case)
    w = _weights(cfg, seed)
    T, B, V, P = cfg["gen_len"], cfg["batch"], cfg["vocab"], cfg["prompt_len"]
    prompts = _prompts(cfg, seed)
    shape = (cfg["n_layers"], B, cfg["n_kv_heads"], P + T - 1, cfg["head_dim"])
    k, v = (torch.zeros(shape, dtype=torch.float64, device="cuda") for _ in range(2))
    logits = torch.zeros((B, V), dtype=torch.float64, device="cuda")
    if T > 1:                                           # every weight is read for every token
        w = {name: t.double() for name, t in w.items()}
    head = w["lm_head"].double()
    tokens = np.zeros((B, T), dtype=np.int64)
    for b in range(B):
        toks, first = prompts[b], 0
        for t in range(T):
            h = _forward64(cfg, w, toks, first, k[:, b], v[:, b])
            logits[b] = (_rms64(h, w["final_norm"], cfg["rms_eps"]) @ head.T)[0]
            first += len(toks)
            z = logits[b]
            if case.get("temperature", 0.0) > 0:
                z = z / case["temperature"] + _gumbel64(seed, b, first - 1, V)
            tokens[b, t] = int(z.argmax())
            toks = tokens[b, t:t + 1]
    if case["kind"] == "prompt":
        return {"logits": logits, "k": k, "v": v}
    # a lattice's last round taps speculative rows too: no plain counterpart
    return {"tokens": tokens, "logits": logits if len(cfg["explored"]) == 1 else None, "k": k, "v": v}
