"""What a program built on libyoco has it do, as cases that can be timed and whose outputs can be compared.

A case is a dict of plain values. `listed()` gives the fixed ones, `draw(rng)` one more of the same ranges, `prepare`
makes what a program has in hand before the call, `run` is one pass through the public entry points, `work` says what
that pass cannot do without, and `tolerance` how far a correct implementation's outputs may lie apart.

Shapes are the paper's profiling setup as this repository configures it (24 query and 8 KV heads of 128, windows of
1024, 13 + 13 layers, prompts of 32K and caches up to 512K rows, the 1.4B row of the scaling table for whole stacks),
and the smaller, odd and ragged ones that a server meets around it.
"""
import math

import torch

import paper_2405_05254_amd as yoco
from paper_2405_05254_amd.stack import YocoStack

DEV = "cuda"
BF16_BYTES, F32_BYTES = 2, 4
EPS = 1e-6


def listed():
    return [
        # Self-decoder prefill of one long prompt: the call that the headline metric counts.
        dict(name="swa_prefill_32k", op="swa_prefill", dtype="bf16", B=1, T=32768, Hq=24, Hkv=24, d=128, window=1024),
        # A batch of ordinary prompts with grouped KV heads; the length is no multiple of any tile.
        dict(name="swa_prefill_batch", op="swa_prefill", dtype="bf16", B=4, T=1500, Hq=24, Hkv=8, d=128, window=1024),
        # The fp32 configuration that checks run in: one short prompt, 4 heads of 64, window 128.
        dict(name="swa_prefill_f32", op="swa_prefill", dtype="f32", B=1, T=512, Hq=4, Hkv=4, d=64, window=128),
        # A chunk of rows that goes through the cross-decoder as well (a full forward, chunked): dense causal attention.
        dict(name="cross_prefill_chunk", op="cross_prefill", cache="bf16", pos0=14000, Tq=2000, Hq=24, Hkv=8),
        # End of an early-exit prefill: the prompt's rows are coded into the 8-bit cache, its last row alone goes on.
        dict(name="early_exit_int8", op="early_exit", cache="int8", T=32768, Hq=24, Hkv=8, layers=13),
        # One generation step's cross-decoder attention over 16 caches of 32K rows: append, then 13 layers.
        dict(name="decode_b16_32k", op="decode", cache="bf16", B=16, N=32768, Hq=24, Hkv=8, layers=13, ragged=False),
        # The same over one cache of 512K rows held in 8 bits.
        dict(name="decode_b1_512k_int8", op="decode", cache="int8", B=1, N=524288, Hq=24, Hkv=8, layers=13, ragged=False),
        # Short conversations of different lengths: small caches, where latency and launches count.
        dict(name="decode_short_ragged", op="decode", cache="bf16", B=8, N=3000, Hq=24, Hkv=8, layers=13, ragged=True),
        # One generation step's self-decoder attention: 13 rolling window caches of 1024 rows, 16 sequences.
        dict(name="swa_decode_b16", op="swa_decode", B=16, window=1024, Hq=24, Hkv=24, layers=13, ragged=False),
        # Gated-retention self-decoder: prefill of one long prompt with GroupNorm, gate and final state.
        dict(name="gret_prefill_32k", op="gret_prefill", B=1, T=32768, H=24),
        # Its generation step, 13 layers of 16 sequences.
        dict(name="gret_decode_b16", op="gret_decode", B=16, H=24, layers=13),
        # A whole request on a stack of the 1.4B shape's layers (4 + 4 of its 12 + 12, so that the bf16 roundings of one
        # layer after another stay small next to the logits): prompt with early exit, then token by token.
        dict(name="stack_generate", op="stack", self_kind="swa", cache="bf16", Hq=16, layers=4, ffn=5632, T=2000, new=16),
    ]


def _log(rng, lo, hi):
    """A whole number in [lo, hi], even over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _heads(rng):
    """(query heads, KV heads) of the cross-decoder."""
    return rng.choice([(24, 8), (24, 8), (16, 16), (16, 4), (32, 8), (64, 8)])


def draw(rng):
    op = rng.choice(["swa_prefill", "swa_prefill", "cross_prefill", "early_exit", "decode", "decode", "swa_decode",
                     "gret_prefill", "gret_decode", "stack"])
    if op == "swa_prefill":
        if rng.random() < 0.25:
            Hq = rng.choice([4, 8])
            return dict(op=op, dtype="f32", B=rng.choice([1, 1, 2]), T=_log(rng, 100, 2048), Hq=Hq, Hkv=rng.choice([Hq, Hq // 4]), d=rng.choice([64, 128]),
                        window=rng.choice([128, 256, 1024]))
        Hq, Hkv = rng.choice([(24, 24), (24, 8), (16, 16)])
        B = rng.choice([1, 1, 2, 4, 8])
        return dict(op=op, dtype="bf16", B=B, T=_log(rng, 200, 32768 // B), Hq=Hq, Hkv=Hkv, d=128, window=rng.choice([512, 1024, 1024, 2048]))
    if op == "cross_prefill":
        Hq, Hkv = _heads(rng)
        return dict(op=op, cache="bf16", pos0=rng.choice([0, _log(rng, 100, 24000)]), Tq=_log(rng, 16, 4096 * 24 // max(Hq, 24)), Hq=Hq, Hkv=Hkv)
    if op == "early_exit":
        Hq, Hkv = _heads(rng)
        return dict(op=op, cache=rng.choice(["bf16", "int8"]), T=_log(rng, 500, 131072 * 8 // max(Hkv, 8)), Hq=Hq, Hkv=Hkv, layers=rng.choice([12, 13, 16]))
    if op == "decode":
        Hq, Hkv = _heads(rng)
        B = _log(rng, 1, 64)
        return dict(op=op, cache=rng.choice(["bf16", "bf16", "int8"]), B=B, N=_log(rng, 300, 524288 * 8 // max(Hkv, 8) // B), Hq=Hq, Hkv=Hkv,
                    layers=rng.choice([12, 13]), ragged=rng.random() < 0.5)
    if op == "swa_decode":
        Hq, Hkv = rng.choice([(24, 24), (24, 24), (16, 16), (24, 8)])
        return dict(op=op, B=_log(rng, 1, 32), window=rng.choice([512, 1024, 1024, 2048]), Hq=Hq, Hkv=Hkv, layers=rng.choice([12, 13]), ragged=rng.random() < 0.5)
    if op == "gret_prefill":
        B = rng.choice([1, 1, 2, 4])
        return dict(op=op, B=B, T=_log(rng, 200, 32768 // B), H=rng.choice([16, 24]))
    if op == "gret_decode":
        return dict(op=op, B=_log(rng, 1, 32), H=rng.choice([16, 24]), layers=rng.choice([12, 13]))
    Hq, kind = rng.choice([8, 16, 16]), rng.choice(["swa", "swa", "gret"])
    return dict(op="stack", self_kind=kind, cache=rng.choice(["bf16", "bf16", "int8"]), Hq=Hq, layers=2 if kind == "gret" else rng.choice([2, 3, 4]),
                ffn=352 * Hq, T=_log(rng, 50, 2000), new=rng.randint(4, 16))


# ---------------------------------------------------------------- inputs
class _Draws:
    """Normal and exponential tensors on the GPU from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def normal(self, shape, std=1.0, dtype=torch.bfloat16):
        return torch.empty(shape, dtype=torch.float32, device=DEV).normal_(0.0, std, generator=self.g).to(dtype)

    def log_decay(self, shape):
        """ln(gamma), gamma mostly in 0.9 .. 1: what a sigmoid raised to 1/16 gives."""
        return torch.empty(shape, dtype=torch.float32, device=DEV).exponential_(25.0, generator=self.g).neg_()

    def lens(self, B, N, ragged):
        if not ragged:
            return torch.full((B,), N, dtype=torch.int64, device=DEV)
        return torch.randint(max(1, N // 8), N + 1, (B,), dtype=torch.int64, device=DEV, generator=self.g)


def _cache_dtype(case):
    return torch.int8 if case["cache"] == "int8" else torch.bfloat16


def _filled_cache(r, case, B, N):
    """A cache of B sequences whose N rows have been written, and the tensor that holds all of it."""
    cache = yoco.KVCache(B, case["Hkv"], 128, N, _cache_dtype(case))
    if case["cache"] == "int8":
        cache.mem.zero_()
        for b in range(B):
            yoco.global_kv_write(cache, r.normal((N, case["Hkv"], 128)), r.normal((N, case["Hkv"], 128)), b, 0)
    else:
        for plane in cache.planes():
            plane.copy_(r.normal(plane.shape))
    return cache


def _whole(cache):
    return cache.mem if cache.dtype == torch.int8 else cache.mem.view(cache.dtype)


def _decode_workspace(cache, Hq):
    return torch.empty(yoco.cross_attn_decode_workspace(cache, Hq)[0], dtype=torch.uint8, device=DEV)


def _stack_weights(r, case):
    Hq, ffn, vocab, dm = case["Hq"], case["ffn"], 32000, case["Hq"] * 128

    def mat(*shape):
        return r.normal(shape, 0.02)

    def gain():
        return 1.0 + r.normal((dm,), 0.1, torch.float32)

    def rest():
        return dict(ln1=gain(), ln2=gain(), W_G=mat(dm, ffn), W_1=mat(dm, ffn), W_2=mat(ffn, dm))

    w = dict(Hq=Hq, Hkv_self=Hq, Hkv=Hq, d=128, window=1024, eps=EPS, embed=mat(vocab, dm), final_ln=gain(), W_out=mat(dm, vocab))
    w["self"] = [dict(W_Q=mat(dm, dm), W_K=mat(dm, dm), W_V=mat(dm, dm), W_O=mat(dm, dm), **rest()) for _ in range(case["layers"])]
    w["kv"] = dict(ln=gain(), W_K=mat(dm, dm), W_V=mat(dm, dm))
    w["cross"] = [dict(W_Q=mat(dm, dm), W_O=mat(dm, dm), **rest()) for _ in range(case["layers"])]
    if case["self_kind"] == "gret":
        w["self_kind"], w["tau"] = "gret", 16.0
        for L in w["self"]:
            L["W_gamma"], L["W_gate"] = mat(dm, Hq), mat(dm, dm)
    return w


def prepare(case, seed):
    r, op, s = _Draws(seed), case["op"], dict(case)
    s["scale"] = 1.0 / math.sqrt(case.get("d", 128))
    if op == "swa_prefill":
        dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        B, T, d = case["B"], case["T"], case["d"]
        s["q"] = r.normal((B, T, case["Hq"], d), 0.5, dt)
        s["k"], s["v"] = (r.normal((B, T, case["Hkv"], d), 0.5, dt) for _ in range(2))
    elif op == "cross_prefill":
        s["kv"] = _filled_cache(r, case, 1, case["pos0"] + case["Tq"])
        s["q"] = r.normal((case["Tq"], case["Hq"], 128))
    elif op == "early_exit":
        T = case["T"]
        s["kv"] = yoco.KVCache(1, case["Hkv"], 128, T, _cache_dtype(case))
        s["kv"].mem.zero_()
        # Eq. 2 with the norm behind the projections: raw products and one factor per row
        s["k"], s["v"] = (r.normal((T, case["Hkv"], 128), 2.0) for _ in range(2))
        s["row_scale"] = r.normal((T,), 0.05, torch.float32) + 0.5
        s["qs"] = [r.normal((1, case["Hq"], 128)) for _ in range(case["layers"])]
        s["os"] = [torch.empty_like(q) for q in s["qs"]]
        s["ws"] = _decode_workspace(s["kv"], case["Hq"])
    elif op == "decode":
        B = case["B"]
        s["kv"] = _filled_cache(r, case, B, case["N"])
        s["lens"] = r.lens(B, case["N"], case["ragged"])
        s["pos"] = s["lens"] - 1
        s["k"], s["v"] = (r.normal((B, case["Hkv"], 128)) for _ in range(2))
        s["qs"] = [r.normal((B, case["Hq"], 128)) for _ in range(case["layers"])]
        s["os"] = [torch.empty_like(q) for q in s["qs"]]
        s["ws"] = _decode_workspace(s["kv"], case["Hq"])
    elif op == "swa_decode":
        B, L = case["B"], range(case["layers"])
        s["rings"] = [_filled_cache(r, dict(case, cache="bf16"), B, case["window"]) for _ in L]
        s["lens"] = r.lens(B, 4 * case["window"], True) if case["ragged"] else torch.full((B,), 32768, dtype=torch.int64, device=DEV)
        s["qs"] = [r.normal((B, case["Hq"], 128)) for _ in L]
        s["ks"], s["vs"] = ([r.normal((B, case["Hkv"], 128)) for _ in L] for _ in range(2))
        s["os"] = [torch.empty_like(q) for q in s["qs"]]
        s["ws"] = _decode_workspace(s["rings"][0], case["Hq"])
    elif op == "gret_prefill":
        B, T, H = case["B"], case["T"], case["H"]
        s["q"], s["k"], s["v"], s["gate"] = (r.normal((B, T, H, 128)) for _ in range(4))
        s["lg"] = r.log_decay((B, T, H))
        s["state"] = torch.empty((B, H, 128, 128), dtype=torch.float32, device=DEV)
        s["o"] = torch.empty_like(s["v"])
        s["ws"] = torch.empty(yoco.gret_prefill_workspace(B, T, H, 128, 128, 256, yoco.BF16), dtype=torch.uint8, device=DEV)
    elif op == "gret_decode":
        B, H, L = case["B"], case["H"], range(case["layers"])
        s["states"] = [r.normal((B, H, 128, 128), 2.0, torch.float32) for _ in L]
        s["qs"], s["ks"], s["vs"], s["gates"] = ([r.normal((B, H, 128)) for _ in L] for _ in range(4))
        s["lgs"] = [r.log_decay((B, H)) for _ in L]
        s["os"] = [torch.empty_like(v) for v in s["vs"]]
    else:
        s["stack"] = YocoStack(_stack_weights(r, case), torch.bfloat16, glue_dtype=torch.bfloat16, cache_dtype=_cache_dtype(case))
        s["tokens"] = torch.randint(0, 32000, (case["T"] + case["new"],), device=DEV, generator=r.g)
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    op, scale = s["op"], s["scale"]
    if op == "swa_prefill":
        return yoco.swa_prefill(s["q"], s["k"], s["v"], s["window"], scale)
    if op == "cross_prefill":
        return yoco.cross_attn_prefill(s["kv"], s["q"], 0, s["pos0"], scale)
    if op == "early_exit":
        yoco.global_kv_write_scaled(s["kv"], s["k"], s["v"], s["row_scale"], 0, 0)
        for q, o in zip(s["qs"], s["os"]):
            yoco.cross_attn_prefill(s["kv"], q, 0, s["T"] - 1, scale, out=o, workspace=s["ws"])
        return {"o": s["os"], "cache": _whole(s["kv"])}
    if op == "decode":
        yoco.kv_cache_append(s["kv"], s["k"], s["v"], s["pos"], False)
        for q, o in zip(s["qs"], s["os"]):
            yoco.cross_attn_decode(s["kv"], q, s["lens"], scale, s["ws"], out=o)
        return {"o": s["os"], "cache": _whole(s["kv"])}
    if op == "swa_decode":
        for ring, q, k, v, o in zip(s["rings"], s["qs"], s["ks"], s["vs"], s["os"]):
            yoco.swa_decode(ring, q, s["lens"], scale, s["ws"], out=o, k_new=k, v_new=v)
        return {"o": s["os"], "rings": [_whole(ring) for ring in s["rings"]]}
    if op == "gret_prefill":
        o = yoco.gret_prefill(s["q"], s["k"], s["v"], s["lg"], scale, chunk=256, group_norm=True, eps=EPS, state_out=s["state"],
                              workspace=s["ws"], out=s["o"], gate=s["gate"])
        return {"o": o, "state": s["state"]}
    if op == "gret_decode":
        for q, k, v, g, lg, state, o in zip(s["qs"], s["ks"], s["vs"], s["gates"], s["lgs"], s["states"], s["os"]):
            yoco.gret_decode(q, k, v, lg, state, scale, group_norm=True, eps=EPS, out=o, gate=g)
        return {"o": s["os"], "states": s["states"]}
    stack, tokens, T, new = s["stack"], s["tokens"], s["T"], s["new"]
    with torch.no_grad():
        state = stack.new_generation_state(T + new)
        logits = [stack.prefill(tokens[:T], state)]
        for i in range(T, T + new):
            logits.append(stack.decode_step(tokens[i], state))
    out = {"logits": torch.cat(logits)}
    if s["cache"] == "bf16":           # 8-bit codes are whole numbers, and those of two correct stacks need not agree
        out["cache"] = _whole(state["cache"])
    out["rings"] = list(state["rings"]) if s["self_kind"] == "gret" else [p[:, :, :T + new] for ring in state["rings"] for p in ring.planes()]
    return out


# ---------------------------------------------------------------- what a pass cannot do without
def _row_bytes(case, heads):
    """Bytes of one cached row over its KV heads, K and V."""
    return 2 * heads * (132 if case.get("cache") == "int8" else 128 * BF16_BYTES)


def _window_pairs(T, C):
    """(query, key) pairs of causal attention over T rows with a window of C."""
    return T * (T + 1) // 2 if T <= C else C * (C + 1) // 2 + (T - C) * C


def _mean_len(case, N):
    return N * 9 // 16 if case["ragged"] else N


def work(case):
    op = case["op"]
    if op == "swa_prefill":
        B, T, Hq, Hkv, d = (case[x] for x in ("B", "T", "Hq", "Hkv", "d"))
        size = F32_BYTES if case["dtype"] == "f32" else BF16_BYTES
        return {"bytes": B * T * 2 * (Hq + Hkv) * d * size, "flops": 4 * d * B * Hq * _window_pairs(T, case["window"])}
    if op == "cross_prefill":
        Tq, p, Hq = case["Tq"], case["pos0"], case["Hq"]
        return {"bytes": (p + Tq) * _row_bytes(case, case["Hkv"]) + 2 * Tq * Hq * 128 * BF16_BYTES,
                "flops": 4 * 128 * Hq * (Tq * p + Tq * (Tq + 1) // 2)}
    if op == "early_exit":
        T, L, cached = case["T"], case["layers"], case["T"] * _row_bytes(case, case["Hkv"])
        return {"bytes": T * (2 * case["Hkv"] * 128 * BF16_BYTES + F32_BYTES) + cached + L * (cached + 2 * case["Hq"] * 128 * BF16_BYTES),
                "flops": 4 * 128 * L * case["Hq"] * T}
    if op == "decode":
        B, L, n = case["B"], case["layers"], _mean_len(case, case["N"])
        new = B * (2 * case["Hkv"] * 128 * BF16_BYTES + _row_bytes(case, case["Hkv"]))
        return {"bytes": L * B * (n * _row_bytes(case, case["Hkv"]) + 2 * case["Hq"] * 128 * BF16_BYTES) + new,
                "flops": 4 * 128 * L * B * case["Hq"] * n}
    if op == "swa_decode":
        # drawn lengths lie evenly in window/2 .. 4 windows: the mean number of rows in a ring is 27/28 of it
        B, L, n = case["B"], case["layers"], case["window"] * 27 // 28 if case["ragged"] else case["window"]
        return {"bytes": L * B * ((n + 1) * _row_bytes(case, case["Hkv"]) + 2 * case["Hq"] * 128 * BF16_BYTES), "flops": 4 * 128 * L * B * case["Hq"] * n}
    if op == "gret_prefill":
        rows = case["B"] * case["T"] * case["H"]
        return {"bytes": rows * (5 * 128 * BF16_BYTES + F32_BYTES) + case["B"] * case["H"] * 128 * 128 * F32_BYTES, "flops": rows * 4 * 128 * 128}
    if op == "gret_decode":
        units = case["layers"] * case["B"] * case["H"]
        return {"bytes": units * (2 * 128 * 128 * F32_BYTES + 5 * 128 * BF16_BYTES + F32_BYTES), "flops": units * 6 * 128 * 128}
    L, T, new, Hq, dm = case["layers"], case["T"], case["new"], case["Hq"], case["Hq"] * 128
    ffn, gret = 3 * dm * case["ffn"], case["self_kind"] == "gret"
    own = L * ((5 if gret else 4) * dm * dm + ffn) + 2 * dm * dm        # weights that every row of the prompt meets
    rest = L * (2 * dm * dm + ffn) + dm * 32000                         # weights that only the last row meets
    row = _row_bytes(case, Hq)
    kept = L * Hq * 128 * 128 * F32_BYTES * 2 if gret else L * min(T, 1024) * 2 * Hq * 128 * BF16_BYTES
    attn = L * T * 4 * dm * 128 if gret else L * 4 * 128 * Hq * _window_pairs(T, 1024)
    return {"bytes": (1 + new) * (own + rest) * BF16_BYTES + new * (kept + L * T * row) + T * row,
            "flops": 2 * own * (T + new) + 2 * rest * (1 + new) + attn + new * L * 4 * 128 * Hq * T}


def tolerance(case):
    if case["op"] == "swa_prefill" and case["dtype"] == "f32":
        return {"rel": 2e-5}
    if case["op"] == "stack":          # every layer rounds its activations to bf16, some thirty roundings one after another
        return {"rel": 2e-2}
    return {"rel": 5e-3, "max": 5e-2, "differ": 0.0}
