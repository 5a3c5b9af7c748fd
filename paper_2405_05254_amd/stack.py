"""YOCO decoder-decoder stack for the end-to-end early-exit and generation
checks (section 2, Eq. 1-3, Fig. 2 and 3). Attention runs in libyoco; RMSNorm, the projections,
SwiGLU and the classifier are plain torch ops on the GPU for fp32 glue and for head dims other than 128.

A bf16 stack (kernel dtype and glue bf16, head_dim 128) runs its token steps wholly in libyoco (yoco_stack_step: one
call enqueues every launch of the token; as torch ops a step was bound by the host, 2.3 ms for 4 + 4 layers whose
weights stream in 0.13 ms) and its prompts with torch GEMMs and libyoco's row-wise passes between them. Its weights
are laid out once, a row per output, which is the order a matrix-vector product reads them in; the tensors in the
layer dicts are views of that, and what a program puts in their place is laid out when it is next used. So a stack made
from bf16 tensors that are on the GPU already holds copies of them, where other stacks hold the tensors themselves
(4 + 4 layers: 2.5 ms and 0.9 GB; asking at each call whether they are still the same: 9 us).

Precision: the attention operands (Q, K, V, the global cache, O) have the
kernel dtype; the residual stream and the glue GEMMs run in `glue_dtype`
(fp32 by default, with the weights' stored values), so the only bf16 roundings
on the path are the ones at the attention boundary.
"""
import ctypes
import math
import threading

import torch

from . import binding as yb


def _rmsnorm(x, gain, eps):
    xf = x.float()
    y = xf * torch.rsqrt(xf.pow(2).mean(-1, keepdim=True) + eps) * gain.float()
    return y.to(x.dtype)


def _rows(x, fn, chunk=16384):
    """Apply a row-wise function in row chunks (bounds the FFN intermediates at long T)."""
    if x.shape[0] <= chunk:
        return fn(x)
    return torch.cat([fn(x[i:i + chunk]) for i in range(0, x.shape[0], chunk)])


def _swiglu(x, L):
    return (torch.nn.functional.silu(x @ L["W_G"]) * (x @ L["W_1"])) @ L["W_2"]


def _plain(X):
    """A tensor as libyoco reads it: contiguous and 16-byte aligned (a copy where it is not)."""
    X = X.contiguous()
    return X if X.data_ptr() % 16 == 0 else X.clone()


class YocoStack:
    """weights: the dict produced by the synthetic generator (numpy arrays);
    dtype: torch.float32 or torch.bfloat16."""

    def __init__(self, weights, dtype, device="cuda", glue_dtype=torch.float32, cache_dtype=None, fused_kv_norm=False):
        self.dtype, self.device, self.glue = dtype, device, glue_dtype
        self.cache_dtype = dtype if cache_dtype is None else cache_dtype   # torch.int8: the global cache holds 8-bit codes
        self.fused_kv_norm = fused_kv_norm   # Eq. 2 with the norm's 1/rms folded into the cache write (yoco_global_kv_write_scaled)
        self.capture = None          # dict layer-name -> (q, k, v, o) (gated retention: + log-decays, gate) when set by a test

        def dev(a):
            return torch.as_tensor(a).to(device=device, dtype=glue_dtype)

        def layer(L):
            return {k: dev(v) for k, v in L.items()}

        w = weights
        self.Hq, self.Hkv_self, self.Hkv, self.d = w["Hq"], w["Hkv_self"], w["Hkv"], w["d"]
        self.window, self.eps = w["window"], w["eps"]
        self.self_kind, self.tau = w.get("self_kind", "swa"), w.get("tau", 16.0)   # "swa" (Eq. 8) or "gret" (Eq. 7)
        self.scale = 1.0 / math.sqrt(self.d)
        self.embed = dev(w["embed"])
        self.self_layers = [layer(L) for L in w["self"]]
        self.kv = layer(w["kv"])
        if fused_kv_norm:             # gain-scaled weights diag(g) W_K, diag(g) W_V, formed once
            self.kv["gW_K"] = (self.kv["ln"].float()[:, None] * self.kv["W_K"].float()).to(glue_dtype)
            self.kv["gW_V"] = (self.kv["ln"].float()[:, None] * self.kv["W_V"].float()).to(glue_dtype)
        self.cross_layers = [layer(L) for L in w["cross"]]
        self.final_ln, self.W_out = dev(w["final_ln"]), dev(w["W_out"])
        self._lock = threading.Lock()
        self._native = self._lay_out() if dtype == glue_dtype == torch.bfloat16 and self.d == 128 else None

    def __getstate__(self):          # addresses are this process's and this object's own
        return dict(self.__dict__, _lock=None, _native=self._native is not None)

    def __setstate__(self, state):
        self.__dict__.update(state, _lock=threading.Lock(), _native=None)
        self._native = self._lay_out() if state["_native"] else None

    def _settings(self):
        return (self.Hq, self.Hkv_self, self.Hkv, self.d, self.self_kind, self.scale, self.eps, self.tau, len(self.self_layers), len(self.cross_layers))

    def _is_laid(self, native):
        """Whether the weights and settings are those that were laid out: the same tensors at the same addresses."""
        return self._settings() == native.settings and all(a is b for a, b in zip(self.self_layers + self.cross_layers, native.layers)) and \
            self.kv is native.kv and all(holder.get(name) is t and t.data_ptr() == at for holder, name, t, at in native.weights)

    def _current(self):
        """The layout for the native calls, None where torch ops serve. What a program has replaced since is laid out anew;
        the wait is for callers on other streams. (A capture would record the layout and not do it: torch ops.)"""
        native = self._native
        if native is None or self._is_laid(native):
            return native
        if torch.cuda.is_current_stream_capturing():
            return None
        with self._lock:
            if self._native is not None and not self._is_laid(self._native):
                native = self._lay_out()
                torch.cuda.current_stream(self.embed.device).synchronize()
                self._native = native
            return self._native

    def _lay_out(self):
        """The stack as libyoco sees it: every weight with a row per output, matrices that read the same input joined.
        None when a shape has no kernel or a weight is not the plain matrix or row that the kernels read (torch ops serve such a
        stack, and say what they miss)."""
        layers = self.self_layers + self.cross_layers
        if not self.cross_layers or self.embed.device.type != "cuda":
            return None
        gret = self.self_kind == "gret"
        into = ("W_Q", "W_K", "W_V") + (("W_gate", "W_gamma") if gret else ())
        dm, ffn, vocab = self.embed.shape[1], layers[0]["W_2"].shape[0], self.W_out.shape[-1]
        qd, kd, ckd = (h * self.d for h in (self.Hq, self.Hkv_self, self.Hkv))
        if dm % 8 or ffn % 8 or max(dm, ffn, qd) > 16384 or min(dm, ffn, vocab, qd, kd, ckd) < 1 or not self.tau > 0:
            return None
        if self.Hq % self.Hkv or (self.self_layers and (self.Hq != self.Hkv_self if gret else self.Hq % self.Hkv_self)):
            return None
        shapes = dict(ln=(dm,), ln1=(dm,), ln2=(dm,), W_Q=(dm, qd), W_K=(dm, kd), W_V=(dm, kd), W_gate=(dm, qd), W_gamma=(dm, self.Hq), W_O=(qd, dm),
                      W_G=(dm, ffn), W_1=(dm, ffn), W_2=(ffn, dm))
        rest = ("ln1", "ln2", "W_O", "W_G", "W_1", "W_2")
        wanted = [(L.get(n), shapes[n]) for L in self.self_layers for n in into + rest]
        wanted += [(L.get(n), shapes[n]) for L in self.cross_layers for n in ("W_Q",) + rest]
        wanted += [(self.kv.get("ln"), (dm,)), (self.kv.get("W_K"), (dm, ckd)), (self.kv.get("W_V"), (dm, ckd)), (self.final_ln, (dm,)), (self.W_out, (dm, vocab))]
        if any(t is None or t.shape != shape or t.dtype != torch.bfloat16 or t.device != self.embed.device for t, shape in wanted):
            return None
        st = yb._Stack()
        st.n_self, st.n_cross, st.d_model, st.ffn, st.vocab = len(self.self_layers), len(self.cross_layers), dm, ffn, vocab
        st.Hq, st.Hkv_self, st.Hkv, st.d, st.gret = self.Hq, self.Hkv_self, self.Hkv, self.d, int(gret)
        st.scale, st.eps, st.tau = self.scale, self.eps, self.tau

        weights = []                 # what was laid out: holder, name, tensor, its address

        def place(L, n, t):
            L[n] = t
            weights.append((L, n, t, t.data_ptr()))
            return t.data_ptr()

        def join(L, rows_name, *names):
            """L[rows_name]: the named matrices, a row per output; they become views of it (and stay, where they are)."""
            rows, width, at, views = L.get(rows_name), L[names[0]].shape[0], 0, []
            total = sum(L[n].shape[1] for n in names)
            kept = torch.is_tensor(rows) and rows.shape == (total, width) and rows.dtype == torch.bfloat16 and rows.is_contiguous() and rows.data_ptr() % 16 == 0
            for n in names:
                end = at + L[n].shape[1]
                kept = kept and L[n].data_ptr() == rows[at:end].data_ptr() and L[n].stride() == rows[at:end].t().stride()
                views.append((n, at, end))
                at = end
            if not kept:
                rows = torch.cat([L[n].t() for n in names])
            for n, at, end in views:
                place(L, n, L[n] if kept else rows[at:end].t())
            return place(L, rows_name, rows)

        def describe(layers, names):
            out = (yb._Layer * len(layers))()
            for s, L in zip(out, layers):
                s.ln1, s.ln2 = place(L, "ln1", _plain(L["ln1"])), place(L, "ln2", _plain(L["ln2"]))
                s.w_in, s.w_o = join(L, "w_in", *names), join(L, "w_o", "W_O")
                s.w_gu, s.w_2 = join(L, "w_gu", "W_G", "W_1"), join(L, "w_2", "W_2")
            return out

        own = self.__dict__
        st.self, st.cross = describe(self.self_layers, into), describe(self.cross_layers, ("W_Q",))
        st.kv_ln, st.w_kv = place(self.kv, "ln", _plain(self.kv["ln"])), join(self.kv, "w_kv", "W_K", "W_V")
        st.final_ln, st.w_out = place(own, "final_ln", _plain(self.final_ln)), join(own, "w_out", "W_out")
        st.scratch_bytes = yb.stack_step_scratch(st)
        st.weights, st.layers, st.kv, st.settings = weights, layers, self.kv, self._settings()
        return st

    def _scratch(self, native):
        return torch.empty(native.scratch_bytes, dtype=torch.uint8, device=self.device)

    def _norm(self, X, gain, native):
        if native is None or X.dtype != torch.bfloat16 or X.dim() != 2 or X.shape[1] != gain.shape[0]:
            return _rmsnorm(X, gain, self.eps)
        return yb.norm_rows(_plain(X), gain, self.eps)

    def _after_attention(self, a, X, L, native):
        """W_O, the residual and the SwiGLU half of Eq. 1 for the rows of a prompt."""
        if native is None:
            Y = a @ L["W_O"] + X
            return _rows(Y, lambda y: _swiglu(_rmsnorm(y, L["ln2"], self.eps), L) + y)
        Y, xn = yb.norm_rows(a @ L["W_O"], L["ln2"], self.eps, add=_plain(X))
        return Y.add_(_rows(xn, lambda x: yb.glu_rows(x @ L["w_gu"].t()) @ L["W_2"]))

    # -- self-decoder: Eq. 1 with sliding-window attention (Eq. 8)
    def _log_decay(self, xn, L):
        """ln(gamma) of Eq. 4: logsigmoid(x W_gamma) / tau, float32 [rows, H]."""
        return (torch.nn.functional.logsigmoid(xn.float() @ L["W_gamma"].float()) / self.tau).contiguous()

    def self_decoder(self, tokens, rings=None):
        """rings: optional per-layer generation caches that receive what a later decode step needs: rolling
        caches (the last `window` K/V rows) for sliding-window attention, fp32 states for gated retention."""
        X, native = self.embed[tokens], self._current()
        T = X.shape[0]
        for n, L in enumerate(self.self_layers):
            xn = self._norm(X, L["ln1"], native)
            q = (xn @ L["W_Q"]).to(self.dtype).view(1, T, self.Hq, self.d)
            k = (xn @ L["W_K"]).to(self.dtype).view(1, T, self.Hkv_self, self.d)
            v = (xn @ L["W_V"]).to(self.dtype).view(1, T, self.Hkv_self, self.d)
            if self.self_kind == "gret":
                lg = self._log_decay(xn, L).view(1, T, self.Hq)
                code = yb.F32 if self.dtype == torch.float32 else yb.BF16
                nbytes = yb.gret_prefill_workspace(1, T, self.Hq, self.d, self.d, 256, code)
                ws = torch.empty(nbytes, dtype=torch.uint8, device=self.device) if nbytes else None
                gate = (xn @ L["W_gate"]).to(self.dtype).view(1, T, self.Hq, self.d)
                o = yb.gret_prefill(q, k, v, lg, self.scale, chunk=256, group_norm=True, eps=self.eps,
                                    state_out=None if rings is None else rings[n], workspace=ws, gate=gate)
                a = o.view(T, self.Hq * self.d).to(self.glue)
                if self.capture is not None and ("self%d" % n) in self.capture:
                    self.capture["self%d" % n] = (q[0], k[0], v[0], o[0], lg[0], gate[0])
                del ws, lg, gate
            else:
                o = yb.swa_prefill(q, k, v, self.window, self.scale)
                if rings is not None:
                    yb.swa_cache_write(rings[n], k[0], v[0], 0, 0)
                a = o.view(T, self.Hq * self.d).to(self.glue)
            if self.capture is not None and self.self_kind != "gret" and ("self%d" % n) in self.capture:
                self.capture["self%d" % n] = (q[0], k[0], v[0], o[0])
            del q, k, v, o, xn
            X = self._after_attention(a, X, L, native)
            del a
        return X

    # -- Eq. 2: the global cache, written once
    def write_cache(self, X, cache=None, pos0=0):
        T = X.shape[0]
        if cache is None:
            cache = yb.KVCache(1, self.Hkv, self.d, T, self.cache_dtype, self.device)
        if self.fused_kv_norm:
            # RMSNorm(x) W = (1 / rms(x)) (x (diag(g) W)): no normalised copy of X, the factor rides on the write
            rs = torch.rsqrt(torch.linalg.vector_norm(X, dim=-1, dtype=torch.float32).pow(2) / X.shape[-1] + self.eps).contiguous()
            k = (X @ self.kv["gW_K"]).view(T, self.Hkv, self.d)
            v = (X @ self.kv["gW_V"]).view(T, self.Hkv, self.d)
            yb.global_kv_write_scaled(cache, k, v, rs, 0, pos0)
            return cache
        xn = self._norm(X, self.kv["ln"], self._current())
        k = (xn @ self.kv["W_K"]).to(self.dtype).view(T, self.Hkv, self.d)
        v = (xn @ self.kv["W_V"]).to(self.dtype).view(T, self.Hkv, self.d)
        yb.global_kv_write(cache, k, v, 0, pos0)
        return cache

    # -- cross-decoder: Eq. 3
    def _cross_layer(self, X, L, attn, native=None):
        Tq = X.shape[0]
        q = (self._norm(X, L["ln1"], native) @ L["W_Q"]).to(self.dtype).view(Tq, self.Hq, self.d)
        a = attn(q).view(Tq, self.Hq * self.d).to(self.glue)
        del q
        return self._after_attention(a, X, L, native)

    def cross_decoder_rows(self, X, cache, q_pos0):
        ws, native = None, self._current()
        if X.shape[0] <= 8:          # few rows: let the call split over the cache
            nbytes, _ = yb.cross_attn_decode_workspace(cache, self.Hq)
            ws = torch.empty(nbytes, dtype=torch.uint8, device=self.device)
        for n, L in enumerate(self.cross_layers):
            def attn(q, n=n):
                o = yb.cross_attn_prefill(cache, q, 0, q_pos0, self.scale, workspace=ws)
                if self.capture is not None and ("cross%d" % n) in self.capture:
                    self.capture["cross%d" % n] = (q, o)
                return o
            X = self._cross_layer(X, L, attn, native)
        return X

    def cross_decoder_decode(self, x_last, cache, length):
        """One token through the cross-decoder with the split-KV decode kernel."""
        nbytes, _ = yb.cross_attn_decode_workspace(cache, self.Hq)
        ws = torch.empty(nbytes, dtype=torch.uint8, device=self.device)
        native = self._current()
        if native is not None and length > 0:                # nothing cached: the torch ops, on zeros from the attention
            X = torch.empty_like(x_last, memory_format=torch.contiguous_format)
            yb.stack_step(native, _plain(x_last), None, None, cache, length - 1, self._scratch(native), ws, x_out=X)
            return X
        lens = torch.tensor([length], dtype=torch.int64, device=self.device)
        X = x_last
        for L in self.cross_layers:
            X = self._cross_layer(X, L, lambda q: yb.cross_attn_decode(cache, q, lens, self.scale, ws))
        return X

    def logits(self, X):
        return _rmsnorm(X, self.final_ln, self.eps) @ self.W_out

    def forward_full(self, tokens, rows=None):
        """Every row through both decoders; logits of `rows` (default: all)."""
        X = self.self_decoder(tokens)
        cache = self.write_cache(X)
        X = self.cross_decoder_rows(X, cache, 0)
        return self.logits(X if rows is None else X[rows])

    def forward_early_exit(self, tokens, decode_kernel=True):
        """Prefill that leaves after the self-decoder and the cache write; only
        the last position enters the cross-decoder (Fig. 3)."""
        X = self.self_decoder(tokens)
        T = X.shape[0]
        cache = self.write_cache(X)
        x_last = X[T - 1:T].contiguous()
        if decode_kernel:
            x_last = self.cross_decoder_decode(x_last, cache, T)
        else:
            x_last = self.cross_decoder_rows(x_last, cache, T - 1)
        return self.logits(x_last), cache

    # -- token-by-token generation (Fig. 3 "Generation"): rolling caches in the self-decoder
    def new_generation_state(self, max_len):
        """Caches of one sequence: per self-decoder layer a ring of `window` rows (sliding-window attention) or an
        fp32 state (gated retention), and the global cache."""
        if self.self_kind == "gret":
            rings = [torch.zeros(1, self.Hq, self.d, self.d, dtype=torch.float32, device=self.device) for _ in self.self_layers]
        else:
            rings = [yb.KVCache(1, self.Hkv_self, self.d, self.window, self.dtype, self.device) for _ in self.self_layers]
        cache = yb.KVCache(1, self.Hkv, self.d, max_len, self.cache_dtype, self.device)
        ws = []
        for c in ((cache, cache) if self.self_kind == "gret" else (rings[0], cache)):
            nbytes, _ = yb.cross_attn_decode_workspace(c, self.Hq)
            ws.append(torch.empty(nbytes, dtype=torch.uint8, device=self.device))
        state = dict(rings=rings, cache=cache, ws_ring=ws[0], ws_cache=ws[1], length=0)
        native = self._current()
        if native is not None:
            state["scratch"] = self._scratch(native)
        return state

    def _native_logits(self, native, x, state, pos, whole):
        """Logits [1,vocab] of one token at position pos; whole: through both decoders, else through the cross-decoder alone."""
        logits = torch.empty((1, native.vocab), dtype=self.glue, device=self.device)
        if "scratch" not in state or state["scratch"].numel() < native.scratch_bytes:      # made for other layers, or for torch ops
            state["scratch"] = self._scratch(native)
        ws = max(state["ws_ring"], state["ws_cache"], key=torch.numel)
        rings, descs, states = state["rings"], None, None       # described anew: a caller may have put copies in their place
        if whole and self.self_kind == "gret":
            states = (ctypes.c_void_p * len(rings))(*(yb._state(r, "state", 1, self.Hq, self.d, self.d) for r in rings))
        elif whole:
            descs = (yb._Cache * len(rings))(*(r.desc for r in rings))
        yb.stack_step(native, _plain(x), descs, states, state["cache"], pos, state["scratch"], ws, logits=logits)
        return logits

    def prefill(self, tokens, state):
        """Early-exit prefill of a prompt (state must be fresh); returns the logits of its last position."""
        assert state["length"] == 0
        X = self.self_decoder(tokens, rings=state["rings"])
        T = X.shape[0]
        self.write_cache(X, state["cache"], 0)
        state["length"] = T
        native = self._current()
        if native is not None:
            return self._native_logits(native, X[T - 1:T], state, T - 1, False)
        lens = torch.tensor([T], dtype=torch.int64, device=self.device)
        x = X[T - 1:T].contiguous()
        for L in self.cross_layers:
            x = self._cross_layer(x, L, lambda q: yb.cross_attn_decode(state["cache"], q, lens, self.scale, state["ws_cache"]))
        return self.logits(x)

    def decode_step(self, token, state):
        """One new token through both decoders; returns its logits [1,vocab]."""
        p = state["length"]
        native = self._current()
        if native is not None:
            logits = self._native_logits(native, self.embed[torch.as_tensor(token, device=self.device).view(1)], state, p, True)
            state["length"] = p + 1
            return logits
        pos = torch.tensor([p], dtype=torch.int64, device=self.device)
        lens = pos + 1
        x = self.embed[torch.as_tensor(token, device=self.device).view(1)]
        for L, ring in zip(self.self_layers, state["rings"]):
            xn = _rmsnorm(x, L["ln1"], self.eps)
            q = (xn @ L["W_Q"]).to(self.dtype).view(1, self.Hq, self.d)
            k = (xn @ L["W_K"]).to(self.dtype).view(1, self.Hkv_self, self.d)
            v = (xn @ L["W_V"]).to(self.dtype).view(1, self.Hkv_self, self.d)
            if self.self_kind == "gret":
                gate = (xn @ L["W_gate"]).to(self.dtype).view(1, self.Hq, self.d)
                o = yb.gret_decode(q, k, v, self._log_decay(xn, L).view(1, self.Hq), ring, self.scale, group_norm=True,
                                   eps=self.eps, gate=gate)
                a = o.view(1, self.Hq * self.d).to(self.glue)
            else:
                o = yb.swa_decode(ring, q, lens, self.scale, state["ws_ring"], k_new=k, v_new=v)   # appends the row itself
                a = o.view(1, self.Hq * self.d).to(self.glue)
            y = a @ L["W_O"] + x
            x = _swiglu(_rmsnorm(y, L["ln2"], self.eps), L) + y
        xn = _rmsnorm(x, self.kv["ln"], self.eps)
        k = (xn @ self.kv["W_K"]).to(self.dtype).view(1, self.Hkv, self.d)
        v = (xn @ self.kv["W_V"]).to(self.dtype).view(1, self.Hkv, self.d)
        yb.kv_cache_append(state["cache"], k, v, pos, False)
        for L in self.cross_layers:
            x = self._cross_layer(x, L, lambda q: yb.cross_attn_decode(state["cache"], q, lens, self.scale, state["ws_cache"]))
        state["length"] = p + 1
        return self.logits(x)
