"""The work that programs have this library do, as cases that can be timed and compared.

Five kinds, each through the public entry points of ``paper_2311_08263_amd``:

  attn      window-causal attention of one layer on a bf16 cache (``attn_window``)
  lmhead    LM head fused with the per-row argmax (``lmhead_argmax``)
  step      one Jacobi step of a running batch (``Context.step``), returning the step's logits
  prompt    a new batch of prompts up to the logits of its first step (``Context.prefill`` + ``Context.step``)
  generate  a whole call on the small fp32 model (``Context.prefill`` + ``Context.generate``)

Shapes are the Llama-2 7B / 13B / 70B dimensions of the benchmark, some with fewer layers (every layer is alike, so
a few stand for all), and the small fp32 configuration.  Weights are random with the usual scaled initialisation
(residual projections divided by sqrt(2 * layers)) and a head that points along the embeddings, so that a row has a
clear winner, as a trained model's rows have: the next window never hangs on a rounding error.

A step moves its state on by one token, as a decoding loop does, until the room of the case (``room`` tokens) is used
up; from then on the finished sequences repeat the same step.
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

import paper_2311_08263_amd as fc

# layers are the case's own; d_model, heads, K/V heads, head dim, FFN, vocabulary
SHAPES = {
    "tiny": (256, 4, 4, 64, 688, 1024),
    "small": (2048, 16, 4, 128, 5632, 32000),
    "7b": (4096, 32, 32, 128, 11008, 32000),
    "13b": (5120, 40, 40, 128, 13824, 32000),
    "70b": (8192, 64, 8, 128, 28672, 32000),
}
EPS, ROPE_BASE, STD = 1e-5, 1e4, 0.02


def listed():
    return [
        # a decode step's attention of one 7B layer at a 2k context: the window of the benchmark
        {"name": "attn_7b_n2048_w16", "kind": "attn", "n": 2048, "W": 16, "H": 32, "Hkv": 32},
        # grouped K/V heads (70B layer), a ragged length, a narrow window: the smallest attention call
        {"name": "attn_70b_n777_w5", "kind": "attn", "n": 777, "W": 5, "H": 64, "Hkv": 8},
        # a wide window (the window sweep goes up to 128 rows) over the 13B heads
        {"name": "attn_13b_n1024_w64", "kind": "attn", "n": 1024, "W": 64, "H": 40, "Hkv": 40},
        # next-token choice of one 7B window
        {"name": "lmhead_7b_m16", "kind": "lmhead", "M": 16, "d": 4096, "V": 32000, "logits": False},
        # next-token choice of a 13B batch: 8 sequences x 32 rows
        {"name": "lmhead_13b_m256", "kind": "lmhead", "M": 256, "d": 5120, "V": 32000, "logits": False},
        # the benchmark's decoding step: the whole 7B-shaped model, batch 1, prompt 256, window 16
        {"name": "step_7b_full_w16", "kind": "step", "shape": "7b", "layers": 32, "B": 1, "P": 256, "W": 16, "room": 256, "windows": "", "planes": 2},
        # greedy decoding (window 1) over a longer context
        {"name": "step_7b_l4_w1", "kind": "step", "shape": "7b", "layers": 4, "B": 1, "P": 1500, "W": 1, "room": 256, "windows": "", "planes": 2},
        # the benchmark's batched step: 13B layers, 8 sequences of about 1024 tokens, window 32 (256 rows)
        {"name": "step_13b_l4_b8_w32", "kind": "step", "shape": "13b", "layers": 4, "B": 8, "P": 1024, "W": 32, "room": 160, "windows": "", "planes": 2},
        # the benchmark's 70B layers (grouped K/V heads), prompt 512, window 16
        {"name": "step_70b_l2_w16", "kind": "step", "shape": "70b", "layers": 2, "B": 1, "P": 512, "W": 16, "room": 160, "windows": "", "planes": 2},
        # four sequences with windows of their own in one batch: packed rows (16 + 23 + 7 + 31 of them)
        {"name": "step_7b_l4_ragged", "kind": "step", "shape": "7b", "layers": 4, "B": 4, "P": 700, "W": 31, "room": 160, "windows": "16,23,7,31", "planes": 2},
        # time to the first window of a long prompt
        {"name": "prompt_7b_l4_p2048", "kind": "prompt", "shape": "7b", "layers": 4, "B": 1, "P": 2048, "W": 16, "planes": 2},
        # the small fp32 configuration end to end: prompt 32, window 8, 32 new tokens
        {"name": "generate_tiny_f32", "kind": "generate", "shape": "tiny", "layers": 2, "B": 1, "P": 32, "W": 8, "N": 32},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw(rng):
    kind = rng.choice(("attn", "lmhead", "step", "step", "prompt", "generate"))
    if kind == "attn":
        H, Hkv = rng.choice(((32, 32), (40, 40), (64, 8), (16, 4)))
        return {"kind": "attn", "n": _log_int(rng, 64, 4096), "W": _log_int(rng, 1, 96), "H": H, "Hkv": Hkv}
    if kind == "lmhead":
        return {"kind": "lmhead", "M": _log_int(rng, 1, 256), "d": rng.choice((2048, 4096, 5120, 8192)),
                "V": 16 * rng.randint(500, 3200), "logits": rng.random() < 0.3}
    if kind == "generate":
        return {"kind": "generate", "shape": "tiny", "layers": 2, "B": rng.randint(1, 3), "P": _log_int(rng, 4, 64),
                "W": rng.randint(2, 16), "N": _log_int(rng, 8, 48)}
    shape = rng.choice(("small", "7b", "13b", "70b"))
    layers = rng.randint(1, 2 if shape == "70b" else 4)
    if kind == "prompt":
        return {"kind": "prompt", "shape": shape, "layers": layers, "B": rng.choice((1, 1, 2, 4)), "P": _log_int(rng, 33, 2048),
                "W": rng.randint(1, 32), "planes": rng.choice((2, 2, 2, 1))}
    B = rng.choice((1, 1, 2, 3, 4, 8))
    W = _log_int(rng, 1, 64 if B <= 4 else 32)
    windows = ",".join(str(rng.randint(1, W)) for _ in range(B)) if B > 1 and W > 1 and rng.random() < 0.35 else ""
    return {"kind": "step", "shape": shape, "layers": layers, "B": B, "P": _log_int(rng, 32, 2048), "W": W, "room": 128,
            "windows": windows, "planes": rng.choice((2, 2, 2, 2, 1, 3))}


def _cost(case):
    w = work(case)
    return w["bytes"] / 4e12 + w["flops"] / (2e13 if case["kind"] == "lmhead" and case["M"] > 32 else 4e14)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        case = _draw(rng)
        if _cost(case) <= most:
            return case


# ---------------------------------------------------------------------------- inputs
def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + stream * 7919 + 17) % (1 << 62))
    return g


def _normal(shape, seed, stream, std, dtype):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=_gen(seed, stream))


def _weights(case, seed, dtype):
    """(name, layer, tensor) of every tensor of the model in the library's canonical layout, one at a time."""
    d, H, Hkv, Dh, F, V = SHAPES[case["shape"]]
    L, qd, kvd = case["layers"], H * Dh, Hkv * Dh
    res = STD / math.sqrt(2.0 * L)
    emb = _normal((V, d), seed, 1, 1.0, dtype)
    yield "emb", -1, emb
    yield "wlm", -1, (emb.t().float() * STD).to(dtype).contiguous()
    yield "gf", -1, 1.0 + _normal((d,), seed, 2, 0.1, torch.float32)
    for l in range(L):
        dims = {"wq": (d, qd, STD), "wk": (d, kvd, STD), "wv": (d, kvd, STD), "wo": (qd, d, res),
                "wg": (d, F, STD), "wu": (d, F, STD), "wd": (F, d, res)}
        for i, (name, (r, c, std)) in enumerate(dims.items()):
            yield name, l, _normal((r, c), seed, 100 + 16 * l + i, std, dtype)
        yield "g1", l, 1.0 + _normal((d,), seed, 100 + 16 * l + 8, 0.1, torch.float32)
        yield "g2", l, 1.0 + _normal((d,), seed, 100 + 16 * l + 9, 0.1, torch.float32)


def _room(case):
    if case["kind"] == "step":
        return case["room"]
    return case["N"] if case["kind"] == "generate" else case["W"]


def _tokens(case, seed):
    """Prompts [B][P], their lengths (ragged in a batch) and the draft buffer: uniform token ids; one buffer entry in
    eight repeats the prompt's last token, which is what the copying head predicts, so that some drafts verify."""
    B, P, V = case["B"], case["P"], SHAPES[case["shape"]][5]
    r = np.random.RandomState((int(seed) * 31 + 5) % (1 << 32))
    lens = np.array([max(1, P - (37 * b) % (P // 4 + 1)) for b in range(B)], dtype=np.int32)
    prompts = r.randint(0, V, (B, P)).astype(np.int32)
    buf = r.randint(0, V, (B, _room(case) + 2 * case["W"])).astype(np.int32)
    last = prompts[np.arange(B), lens - 1]
    buf = np.where(r.rand(*buf.shape) < 0.125, last[:, None], buf).astype(np.int32)
    return prompts, lens, buf


def _config(case):
    d, H, Hkv, Dh, F, V = SHAPES[case["shape"]]
    S = case["P"] + _room(case) + 2 * case["W"]
    return fc.Config(case["layers"], d, H, Hkv, Dh, F, V, EPS, ROPE_BASE, 0 if case["shape"] == "tiny" else 1, case["B"], S, case["W"])


def _prepare_model(case, seed):
    cfg = _config(case)
    dtype = torch.float32 if case["shape"] == "tiny" else torch.bfloat16
    lib, st = fc.lib(), torch.cuda.current_stream().cuda_stream
    packed = torch.zeros(lib.fastcot_weight_bytes(ctypes.byref(cfg)), dtype=torch.uint8, device="cuda")
    for name, layer, t in _weights(case, seed, dtype):
        rc = lib.fastcot_pack_tensor(ctypes.byref(cfg), fc.binding.T[name], max(layer, 0), t.data_ptr(), packed.data_ptr(), st)
        if rc:
            raise RuntimeError("fastcot_pack_tensor: %d" % rc)
    ctx = fc.Context(cfg, packed)
    if case.get("planes", 2) != 2:
        ctx.set_option(fc.binding.OPT_KV_PLANES, case["planes"])
    logits = ctx.debug_logits(True)
    prompts, lens, buf = _tokens(case, seed)
    s = {"kind": case["kind"], "ctx": ctx, "prompts": prompts, "lens": lens, "buf": buf, "logits": logits[:case["B"] * case["W"]], "N": case.get("N", 0)}
    if case["kind"] == "step":
        ctx.prefill(prompts, lens, buf)
        if case["windows"]:
            ctx.set_windows([int(w) for w in case["windows"].split(",")])
            s["logits"] = logits[:int(ctx.step_rows()[-1])]
    torch.cuda.synchronize()
    return s


def _attn_inputs(case, seed):
    n, W, H, Hkv = case["n"], case["W"], case["H"], case["Hkv"]
    q = _normal((W, H, 128), seed, 1, 1.0, torch.float32)
    k = _normal((n + W, Hkv, 128), seed, 2, 1.0, torch.bfloat16)
    v = _normal((n + W, Hkv, 128), seed, 3, 1.0, torch.bfloat16)
    return q, k, v


def _lmhead_inputs(case, seed):
    M, d, V = case["M"], case["d"], case["V"]
    w = _normal((d, V), seed, 1, STD, torch.bfloat16)
    # rows as the final norm leaves them: unit scale, leaning towards one token's column
    want = torch.randint(0, V, (M,), generator=_gen(seed, 3), device="cuda")
    act = _normal((M, d), seed, 2, 1.0, torch.float32) + 0.4 * w.t()[want].float() / STD
    return act.contiguous(), w


def prepare(case, seed):
    if case["kind"] == "attn":
        q, k, v = _attn_inputs(case, seed)
        S = (case["n"] + case["W"] + 31) // 32 * 32
        kc, vc = fc.kv_scatter(k, v, S)
        nbytes = fc.lib().fastcot_attn_scratch_bytes(case["W"], case["H"], 128)
        return {"kind": "attn", "q": q, "kc": kc, "vc": vc, "n": case["n"], "scratch": torch.zeros(nbytes, dtype=torch.uint8, device="cuda")}
    if case["kind"] == "lmhead":
        act, w = _lmhead_inputs(case, seed)
        packed = fc.lmhead_pack(w)
        nbytes = fc.lib().fastcot_lmhead_scratch_bytes(case["M"], case["d"], case["V"])
        return {"kind": "lmhead", "act": act, "packed": packed, "V": case["V"], "logits": case["logits"],
                "scratch": torch.zeros(nbytes, dtype=torch.uint8, device="cuda")}
    return _prepare_model(case, seed)


def _step(ctx, logits):
    """One step whose logits are used on the caller's stream: the step waits for what that stream still does with the
    logits of the step before, and the stream waits for the step."""
    here = torch.cuda.current_stream()
    ctx.stream.wait_stream(here)
    ctx.step(sync=False)
    here.wait_stream(ctx.stream)
    return logits


def run(state):
    if state["kind"] == "attn":
        return fc.attn_window(state["q"], state["kc"], state["vc"], state["n"], state["scratch"])
    if state["kind"] == "lmhead":
        ids, top, logits = fc.lmhead_argmax(state["act"], state["packed"], state["V"], state["logits"], state["scratch"])
        return {"ids": ids, "top": top, "logits": logits}
    ctx = state["ctx"]
    if state["kind"] == "step":
        return {"logits": _step(ctx, state["logits"])}
    ctx.prefill(state["prompts"], state["lens"], state["buf"])
    if state["kind"] == "prompt":
        return {"logits": _step(ctx, state["logits"])}
    out = ctx.generate(state["N"])
    return {"ids": out["ids"], "len": out["len"], "steps": out["steps"], "logits": state["logits"]}


# ---------------------------------------------------------------------------- what a pass cannot do without
def work(case):
    if case["kind"] == "attn":
        n, W, H, Hkv = case["n"], case["W"], case["H"], case["Hkv"]
        keys = W * n + W * (W + 1) // 2
        return {"bytes": 2 * (n + W) * Hkv * 128 * 2 + 2 * W * H * 128 * 4, "flops": 4 * keys * H * 128}
    if case["kind"] == "lmhead":
        M, d, V = case["M"], case["d"], case["V"]
        return {"bytes": d * V * 2 + M * d * 4 + M * 8 + (M * V * 4 if case["logits"] else 0), "flops": 2 * M * d * V}
    d, H, Hkv, Dh, F, V = SHAPES[case["shape"]]
    L, W, esz = case["layers"], case["W"], 4 if case["shape"] == "tiny" else 2
    layer = d * (H + 2 * Hkv) * Dh + H * Dh * d + 3 * d * F
    kv = 2 * Hkv * Dh * (4 if case["shape"] == "tiny" else {1: 2, 2: 4, 3: 3}[case.get("planes", 2)])     # bytes of one cached position
    _, lens, _ = _tokens(case, 0)
    if case["kind"] == "generate":
        # one exact token per step: what a random draft gives
        steps, M, n = case["N"], case["B"] * W, sum(int(p) for p in lens)
        pf = n - case["B"]
        nbytes = steps * ((L * layer + d * V) * esz + L * kv * (n + M)) + L * layer * esz + case["B"] * case["N"] * 4
        return {"bytes": nbytes, "flops": 2 * (steps * M * (L * layer + d * V) + pf * L * layer) + 4 * steps * L * M * H * Dh * n // case["B"]}
    rows = [int(w) for w in case["windows"].split(",")] if case.get("windows") else [W] * case["B"]
    M, ctx = sum(rows), [int(p) - 1 for p in lens]
    nbytes = (L * layer + d * V) * esz + L * kv * (sum(ctx) + M) + M * d * esz + M * V * 4
    flops = 2 * M * (L * layer + d * V) + 4 * L * H * Dh * sum(r * (c + (r + 1) / 2) for r, c in zip(rows, ctx))
    if case["kind"] == "prompt":
        nbytes += L * layer * esz + L * kv * sum(ctx)
        flops += 2 * sum(ctx) * L * layer + 4 * L * H * Dh * sum(c * (c + 1) / 2 for c in ctx)
    return {"bytes": nbytes, "flops": flops}


# About four times what the path shows against 64 bits: activations, queries and probabilities travel as bf16 hi + lo
# pairs (17 bits), sums in 32 bits: 3e-6 for one attention, up to 1.6e-5 for the logits of one to 32 layers; with one
# plane (planes = 1) the cached K and V are plain bf16: 1.3e-3.
def tolerance(case):
    if case["kind"] == "attn":
        return {"rel": 1.5e-5, "max": 5e-4}
    if case["kind"] == "lmhead":
        return {"rel": 1e-5, "max": 5e-4, "differ": 0.01}
    if case["kind"] == "generate":
        return {"rel": 2e-6, "max": 1e-4}
    return {"rel": 6e-3, "max": 0.2} if case["planes"] == 1 else {"rel": 8e-5, "max": 3e-3}


# ---------------------------------------------------------------------------- the same in 64 bits
def _rope(x, pos):
    """x [rows][heads][Dh] at positions pos: pairs (i, i + Dh/2)."""
    half = x.shape[-1] // 2
    freq = ROPE_BASE ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / x.shape[-1])
    ang = pos.double()[:, None] * freq[None, :]
    c, s = ang.cos()[:, None, :], ang.sin()[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat((a * c - b * s, b * c + a * s), dim=-1)


def _attend(q, k, v, n):
    """q [W][H][Dh] over k, v [n + W][Hkv][Dh]: row j sees positions 0 .. n + j."""
    W, H, Dh = q.shape
    T, Hkv = k.shape[0], k.shape[1]
    seen = torch.arange(T, device="cuda")[None, :] <= n + torch.arange(W, device="cuda")[:, None]
    out = torch.empty(W, H, Dh, dtype=torch.float64, device="cuda")
    for h in range(H):
        kh = h // (H // Hkv)
        s = (q[:, h] @ k[:, kh].t().contiguous()) / math.sqrt(Dh)
        out[:, h] = torch.softmax(s.masked_fill(~seen, -math.inf), dim=-1) @ v[:, kh].contiguous()
    return out.reshape(W, H * Dh)


def _norm(x, g):
    return x / torch.sqrt((x * x).mean(dim=-1, keepdim=True) + EPS) * g.double()


def _forward(case, seed, rows_of):
    """Logits in 64 bits of the last rows_of[b][1] rows of the token rows rows_of[b][0], every sequence from position 0."""
    d, H, Hkv, Dh, F, V = SHAPES[case["shape"]]
    dtype = torch.float32 if case["shape"] == "tiny" else torch.bfloat16
    xs, layer, head = None, {}, {}
    for name, l, t in _weights(case, seed, dtype):
        if l < 0:
            head[name] = t
            continue
        if xs is None:
            xs = [head["emb"][torch.as_tensor(np.asarray(r), device="cuda").long()].double() for r, _ in rows_of]
        layer[name] = t
        if name != "g2":
            continue
        w = {k: (v.double() if v.dim() == 2 else v) for k, v in layer.items()}
        for b, x in enumerate(xs):
            T = x.shape[0]
            pos = torch.arange(T, device="cuda")
            nx = _norm(x, w["g1"])
            q = _rope((nx @ w["wq"]).view(T, H, Dh), pos)
            k = _rope((nx @ w["wk"]).view(T, Hkv, Dh), pos)
            v = (nx @ w["wv"]).view(T, Hkv, Dh)
            x = x + _attend(q, k, v, 0) @ w["wo"]
            nx = _norm(x, w["g2"])
            g = nx @ w["wg"]
            xs[b] = x + (g * torch.sigmoid(g) * (nx @ w["wu"])) @ w["wd"]
        layer = {}
    wlm = head["wlm"].double()
    return [_norm(x[-r:], head["gf"]) @ wlm for x, (_, r) in zip(xs, rows_of)]


def exact(case, seed):
    if case["kind"] == "attn":
        q, k, v = _attn_inputs(case, seed)
        return _attend(q.double(), k.double(), v.double(), case["n"])
    if case["kind"] == "lmhead":
        act, w = _lmhead_inputs(case, seed)
        logits = act.double() @ w.double()
        top, ids = logits.max(dim=1)
        return {"ids": ids.int(), "top": top, "logits": logits if case["logits"] else None}
    prompts, lens, buf = _tokens(case, seed)
    B, W = case["B"], case["W"]
    if case["kind"] != "generate":
        rows = [int(w) for w in case["windows"].split(",")] if case.get("windows") else [W] * B
        # the first step's window: the prompt's last token, then the head of the draft buffer
        seqs = [np.concatenate((prompts[b, :lens[b]], buf[b, :rows[b] - 1])) for b in range(B)]
        return {"logits": torch.cat(_forward(case, seed, [(s, r) for s, r in zip(seqs, rows)]))}
    # the whole trajectory: accept the matching prefix of the draft plus one, write all outputs back, slide the window
    N = case["N"]
    done = [list(map(int, prompts[b, :lens[b]])) for b in range(B)]
    new, steps, draft, logits = [[] for _ in range(B)], [0] * B, buf.copy(), [None] * B
    while any(len(t) < N for t in new):
        live = [b for b in range(B) if len(new[b]) < N]
        out = _forward(case, seed, [(np.array(done[b] + [int(t) for t in draft[b, len(new[b]):len(new[b]) + W - 1]]), W) for b in live])
        for b, lg in zip(live, out):
            o, g = lg.argmax(dim=1).tolist(), len(new[b])
            K = 0
            while K < W - 1 and o[K] == draft[b, g + K]:
                K += 1
            draft[b, g:g + W] = o
            new[b] += o[:K + 1]
            done[b] += o[:K + 1]
            steps[b] += 1
            logits[b] = lg
    # sequences that end early keep stepping with their rows as they are, or leave the batch: their last logits have no value here
    one = B == 1
    return {"ids": torch.tensor([t[:N] for t in new], dtype=torch.int32), "len": torch.tensor([N] * B, dtype=torch.int32),
            "steps": torch.tensor(steps, dtype=torch.int32), "logits": logits[0] if one else None}
