"""Binding of include/yoco.h: same names, argument marshalling only. Sizing, description and measurement calls go through
ctypes; the calls of a running model are checked and marshalled in native code (csrc/py_calls.cpp), because a step over a
small cache or state takes no longer than Python took to check its arguments."""
import ctypes as C
import os

import torch

F32, BF16, INT8 = 0, 1, 2
_PKG = os.path.dirname(os.path.abspath(__file__))
_LIB = None
_CALLS = None


class YocoError(RuntimeError):
    pass


class _Layer(C.Structure):
    _fields_ = [(n, C.c_void_p) for n in ("ln1", "w_in", "w_o", "ln2", "w_gu", "w_2")]


class _Stack(C.Structure):
    _fields_ = [("self", C.POINTER(_Layer)), ("cross", C.POINTER(_Layer))] + \
               [(n, C.c_void_p) for n in ("kv_ln", "w_kv", "final_ln", "w_out")] + \
               [(n, C.c_int32) for n in ("n_self", "n_cross", "d_model", "Hq", "Hkv_self", "Hkv", "d", "ffn", "vocab", "gret")] + \
               [(n, C.c_float) for n in ("scale", "eps", "tau")]


class _Cache(C.Structure):
    _fields_ = [("k", C.c_void_p), ("v", C.c_void_p), ("B", C.c_int32), ("Hkv", C.c_int32),
                ("d", C.c_int32), ("dtype", C.c_int32), ("N_cap", C.c_int64)]


def lib_path():
    """The in-tree libyoco.so (the only build this binding loads)."""
    return os.path.join(_PKG, "libyoco.so")


def lib():
    """Load libyoco.so (built by paper_2405_05254_amd/build.py); fail loudly if absent."""
    global _LIB
    if _LIB is not None:
        return _LIB
    path = lib_path()
    if not os.path.exists(path):
        raise YocoError("libyoco.so is not built: run `python -m paper_2405_05254_amd.build` "
                        "(or __graft_entry__.build()); there is no fallback path")
    L = C.CDLL(path)
    vp, i32, i64, f32, sz = C.c_void_p, C.c_int, C.c_int64, C.c_float, C.c_size_t
    L.yoco_version.restype = i32
    L.yoco_last_error_string.restype = C.c_char_p
    L.yoco_kv_cache_bytes.argtypes = [i32, i32, i32, i64, i32, C.POINTER(sz)]
    L.yoco_kv_cache_init.argtypes = [vp, sz, i32, i32, i32, i64, i32, C.POINTER(_Cache)]
    L.yoco_swa_prefill.argtypes = [vp, vp, vp, vp, i32, i64, i32, i32, i32, i64, f32, i32, vp]
    L.yoco_global_kv_write.argtypes = [C.POINTER(_Cache), vp, vp, i32, i64, i64, i32, vp]
    L.yoco_global_kv_write_scaled.argtypes = [C.POINTER(_Cache), vp, vp, vp, i32, i64, i64, i32, vp]
    L.yoco_cross_attn_prefill.argtypes = [C.POINTER(_Cache), vp, vp, i32, i64, i64, i32, f32, vp, sz, vp]
    L.yoco_cross_attn_prefill_workspace.argtypes = [C.POINTER(_Cache), i64, i64, i32, f32, C.POINTER(sz)]
    L.yoco_cross_attn_decode_workspace.argtypes = [C.POINTER(_Cache), i32, C.POINTER(sz), C.POINTER(i32)]
    L.yoco_cross_attn_decode.argtypes = [C.POINTER(_Cache), vp, vp, vp, i32, f32, vp, sz, vp]
    L.yoco_cross_attn_decode_noalloc.argtypes = [C.POINTER(_Cache), vp, vp, vp, i32, f32, vp]
    L.yoco_swa_cache_write.argtypes = [C.POINTER(_Cache), vp, vp, i32, i64, i64, i32, vp]
    L.yoco_kv_cache_append.argtypes = [C.POINTER(_Cache), vp, vp, vp, i32, i32, vp]
    L.yoco_swa_decode.argtypes = [C.POINTER(_Cache), vp, vp, vp, vp, vp, i32, f32, vp, sz, vp]
    L.yoco_gret_prefill_workspace.argtypes = [i32, i64, i32, i32, i32, i32, i32, C.POINTER(sz)]
    L.yoco_gret_prefill.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, i32, i64, i32, i32, i32, i32, f32, i32, f32, i32, vp, sz, vp]
    L.yoco_gret_decode.argtypes = [vp, vp, vp, vp, vp, vp, vp, i32, i32, i32, i32, f32, i32, f32, i32, vp]
    L.yoco_stack_step_scratch.argtypes = [C.POINTER(_Stack), C.POINTER(sz)]
    L.yoco_stack_step.argtypes = [C.POINTER(_Stack), vp, C.POINTER(_Cache), C.POINTER(vp), C.POINTER(_Cache), i64, vp, vp, vp, sz, vp, sz, vp]
    L.yoco_norm_rows.argtypes = [vp, vp, vp, vp, vp, i64, i32, f32, vp]
    L.yoco_glu_rows.argtypes = [vp, vp, i64, i32, vp]
    L.yoco_ceiling_mfma.argtypes = [vp, vp, i32, i32, vp]
    L.yoco_ceiling_attn_loop.argtypes = [vp, vp, i32, i32, i32, vp]
    L.yoco_ceiling_stream_read.argtypes = [vp, sz, vp, i32, vp]
    for name in ("yoco_ceiling_mfma", "yoco_ceiling_attn_loop", "yoco_ceiling_stream_read", "yoco_kv_cache_bytes", "yoco_kv_cache_init", "yoco_swa_prefill", "yoco_global_kv_write", "yoco_global_kv_write_scaled",
                 "yoco_cross_attn_prefill", "yoco_cross_attn_prefill_workspace", "yoco_cross_attn_decode_workspace", "yoco_cross_attn_decode", "yoco_cross_attn_decode_noalloc",
                 "yoco_swa_cache_write", "yoco_kv_cache_append", "yoco_swa_decode",
                 "yoco_gret_prefill_workspace", "yoco_gret_prefill", "yoco_gret_decode",
                 "yoco_stack_step_scratch", "yoco_stack_step", "yoco_norm_rows", "yoco_glu_rows"):
        getattr(L, name).restype = i32
    _LIB = L
    return L


def _calls():
    """The native calls, bound to the loaded library; fail loudly if they are not built."""
    global _CALLS
    if _CALLS is None:
        lib()
        try:
            from . import _calls as calls
        except ImportError as e:
            raise YocoError("the native calls are not built: run `python -m paper_2405_05254_amd.build` (%s)" % e)
        calls.init(lib_path(), YocoError)
        _CALLS = calls
    return _CALLS


def _check(rc):
    if rc != 0:
        raise YocoError("libyoco error %d: %s" % (rc, lib().yoco_last_error_string().decode()))


def _dev(t, name):
    if not t.is_cuda:
        raise YocoError("%s must be a device tensor" % name)
    if not t.is_contiguous():
        raise YocoError("%s must be contiguous" % name)
    return t.data_ptr()


def _ws(workspace):
    """(pointer, bytes) of an optional workspace tensor on the current device."""
    if workspace is None:
        return None, 0
    ptr = _dev(workspace, "workspace")
    if workspace.device.index != torch.cuda.current_device():
        raise YocoError("workspace must live on the current device")
    return ptr, workspace.numel() * workspace.element_size()


def _stream():
    return torch.cuda.current_stream().cuda_stream


def version():
    return lib().yoco_version()


def kv_cache_bytes(B, Hkv, d, N_cap, dtype):
    n = C.c_size_t()
    _check(lib().yoco_kv_cache_bytes(B, Hkv, d, N_cap, dtype, C.byref(n)))
    return n.value


class KVCache:
    """The once-only global K^/V^ cache, or (N_cap = window) the rolling cache of one self-decoder layer:
    torch owns the memory, the descriptor is yoco_kv_cache."""

    def __init__(self, B, Hkv, d, N_cap, dtype=torch.bfloat16, device="cuda"):
        if dtype not in (torch.float32, torch.bfloat16, torch.int8):
            raise YocoError("unsupported cache dtype %s" % dtype)
        code = {torch.float32: F32, torch.bfloat16: BF16, torch.int8: INT8}[dtype]
        self.bytes = kv_cache_bytes(B, Hkv, d, N_cap, code)
        self.mem = torch.empty(self.bytes, dtype=torch.uint8, device=device)
        self.desc = _Cache()
        _check(lib().yoco_kv_cache_init(self.mem.data_ptr(), self.bytes, B, Hkv, d, N_cap, code, C.byref(self.desc)))
        self.B, self.Hkv, self.d, self.N_cap, self.dtype = B, Hkv, d, N_cap, dtype
        self.io_dtype = torch.bfloat16 if dtype == torch.int8 else dtype     # of the queries and outputs on this cache

    @property
    def address(self):
        """Where the descriptor is, for the native calls (asked each time: a program may put another in its place)."""
        return C.addressof(self.desc)

    def planes(self):
        """Views [B,Hkv,N_cap,d] of the K and V planes (for tests and for filling synthetic caches)."""
        if self.dtype == torch.int8:
            raise YocoError("an 8-bit cache is a run of blocks, not a [B,Hkv,N_cap,d] array: use blocks()")
        half = self.bytes // 2
        shape = (self.B, self.Hkv, self.N_cap, self.d)
        return (self.mem[:half].view(self.dtype).view(shape), self.mem[half:].view(self.dtype).view(shape))

    def blocks(self):
        """Byte views [B,Hkv,ceil(N_cap/64),8448] of the K and V planes of an 8-bit cache: per block 8192 code bytes
        in the order yoco.h documents, then the 64 float32 scales of the block's rows."""
        if self.dtype != torch.int8:
            raise YocoError("blocks() is the layout of an 8-bit cache")
        half = self.bytes // 2
        shape = (self.B, self.Hkv, (self.N_cap + 63) // 64, 8448)
        return self.mem[:half].view(shape), self.mem[half:].view(shape)


def swa_prefill(q, k, v, window, scale, out=None):
    """q [B,T,Hq,d]; k, v [B,T,Hkv,d] -> o [B,T,Hq,d] (yoco_swa_prefill)."""
    return (_CALLS or _calls()).swa_prefill(q, k, v, window, scale, out)


def global_kv_write(cache, k, v, b, pos0):
    """k, v [n,Hkv,d] rows -> cache rows [pos0, pos0+n) of sequence b (yoco_global_kv_write)."""
    (_CALLS or _calls()).global_kv_write(cache.address, k, v, None, b, pos0)


def global_kv_write_scaled(cache, k, v, row_scale, b, pos0):
    """k, v [n,Hkv,d] un-normalised projections x (diag(g) W), row_scale float32 [n] = 1/rms(x): rows are scaled in
    float32 and stored like global_kv_write (yoco_global_kv_write_scaled)."""
    if row_scale is None:
        raise YocoError("row_scale must be float32 [n]")
    (_CALLS or _calls()).global_kv_write(cache.address, k, v, row_scale, b, pos0)


def cross_attn_prefill(cache, q, b, q_pos0, scale, out=None, workspace=None):
    """q [Tq,Hq,d] -> o [Tq,Hq,d], causal over the cache of sequence b (yoco_cross_attn_prefill).
    workspace: optional device scratch tensor (cross_attn_decode_workspace for up to 8 rows, cross_attn_prefill_workspace
    for more). Without one, a call of more rows that is not given its output either takes both from torch's allocator.
    It does without scratch under stream capture and where memory is short, and so does every call that is given its
    output: slower where query tiles are few, and with other low-order bits (yoco_cross_attn_prefill)."""
    return (_CALLS or _calls()).cross_attn_prefill(cache.address, q, b, q_pos0, scale, out, workspace)


def cross_attn_prefill_workspace(cache, q_pos0, Tq, Hq, scale):
    """Bytes of scratch that cross_attn_prefill can make use of for more than 8 rows; 0: none."""
    n = C.c_size_t()
    _check(lib().yoco_cross_attn_prefill_workspace(C.byref(cache.desc), q_pos0, Tq, Hq, scale, C.byref(n)))
    return n.value


def cross_attn_decode_workspace(cache, Hq):
    n, s = C.c_size_t(), C.c_int()
    _check(lib().yoco_cross_attn_decode_workspace(C.byref(cache.desc), Hq, C.byref(n), C.byref(s)))
    return n.value, s.value


def cross_attn_decode(cache, q, lens, scale, workspace, out=None):
    """q [B,Hq,d], lens int64 [B] (device) -> o [B,Hq,d] (yoco_cross_attn_decode)."""
    return (_CALLS or _calls()).cross_attn_decode(cache.address, q, lens, scale, workspace, out)


NOALLOC_SCRATCH_BYTES = 4 << 20


def cross_attn_decode_noalloc(cache, q, lens, scale, out):
    """yoco_cross_attn_decode_noalloc: the decode step with the library's static scratch instead of a workspace.
    `out` is required (this wrapper allocates nothing either)."""
    return (_CALLS or _calls()).cross_attn_decode_noalloc(cache.address, q, lens, scale, out)


def swa_cache_write(ring, k, v, b, pos0):
    """k, v [n,Hkv,d] rows of positions pos0.. -> ring slots (pos0 + r) mod N_cap of sequence b (yoco_swa_cache_write)."""
    (_CALLS or _calls()).swa_cache_write(ring.address, k, v, b, pos0)


def kv_cache_append(cache, k, v, pos, ring):
    """k, v [B,Hkv,d], pos int64 [B] (device): one row per sequence at slot pos[b] (mod N_cap if ring)
    (yoco_kv_cache_append)."""
    (_CALLS or _calls()).kv_cache_append(cache.address, k, v, pos, ring)


def swa_decode(ring, q, lens, scale, workspace, out=None, k_new=None, v_new=None):
    """q [B,Hq,d], lens int64 [B] (device, tokens so far including the new one) -> o [B,Hq,d] (yoco_swa_decode).
    k_new, v_new [B,Hkv,d]: the new token's rows, stored by the same call; None when they were appended before."""
    return (_CALLS or _calls()).swa_decode(ring.address, q, lens, scale, workspace, out, k_new, v_new)


def gret_prefill_workspace(B, T, H, dk, dv, chunk, dtype):
    n = C.c_size_t()
    _check(lib().yoco_gret_prefill_workspace(B, T, H, dk, dv, chunk, dtype, C.byref(n)))
    return n.value


def gret_prefill(q, k, v, log_gamma, scale, chunk=256, group_norm=True, eps=1e-6, state_in=None, state_out=None,
                 workspace=None, out=None, gate=None):
    """q, k [B,T,H,dk]; v [B,T,H,dv]; log_gamma float32 [B,T,H] -> o [B,T,H,dv] (yoco_gret_prefill).
    States are float32 [B,H,dv,dk]; workspace: device tensor from gret_prefill_workspace bytes (None: recurrent path);
    gate: optional tensor like v, the output is multiplied by swish(gate)."""
    return (_CALLS or _calls()).gret_prefill(q, k, v, log_gamma, scale, chunk, group_norm, eps, state_in, state_out, workspace, out, gate)


def gret_decode(q, k, v, log_gamma, state, scale, group_norm=True, eps=1e-6, out=None, gate=None):
    """q, k [B,H,dk]; v [B,H,dv]; log_gamma float32 [B,H]; state float32 [B,H,dv,dk], updated in place
    -> o [B,H,dv] (yoco_gret_decode)."""
    return (_CALLS or _calls()).gret_decode(q, k, v, log_gamma, state, scale, group_norm, eps, out, gate)


def _state(t, name, B, H, dk, dv):
    if t.dtype != torch.float32 or t.shape != (B, H, dv, dk):
        raise YocoError("%s must be float32 [B,H,dv,dk]" % name)
    return _dev(t, name)


def _bf16(t, name, shape):
    if t.dtype != torch.bfloat16 or t.shape != shape:
        raise YocoError("%s must be bfloat16 %s, not %s %s" % (name, list(shape), t.dtype, list(t.shape)))


def stack_step_scratch(stack):
    n = C.c_size_t()
    _check(lib().yoco_stack_step_scratch(C.byref(stack), C.byref(n)))
    return n.value


def stack_step(stack, x, rings, states, cache, pos, scratch, workspace, x_out=None, logits=None):
    """One token through a bf16 stack (yoco_stack_step). x, x_out [1,d_model], logits [1,vocab]; rings: ctypes array of
    cache descriptors or None; states: ctypes array of state pointers or None; both None: the cross-decoder alone."""
    for t, name, width in ((x, "x", stack.d_model), (x_out, "x_out", stack.d_model), (logits, "logits", stack.vocab)):
        if t is not None:
            _bf16(t, name, (1, width))
    for per_layer, name in ((rings, "rings"), (states, "states")):
        if per_layer is not None and len(per_layer) != stack.n_self:
            raise YocoError("%s must hold one entry per self-decoder layer" % name)
    _check(lib().yoco_stack_step(C.byref(stack), _dev(x, "x"), rings, states, C.byref(cache.desc), pos,
                                 None if x_out is None else _dev(x_out, "x_out"), None if logits is None else _dev(logits, "logits"),
                                 *_ws(scratch), *_ws(workspace), _stream()))


def norm_rows(x, gain, eps, add=None):
    """RMSNorm(x) * gain over the rows of a bf16 [rows,dim] tensor; with `add`: (x + add, RMSNorm(x + add) * gain) (yoco_norm_rows)."""
    if x.dim() != 2:
        raise YocoError("x must be [rows,dim]")
    _bf16(x, "x", x.shape)
    _bf16(gain, "gain", x.shape[1:])
    if add is not None:
        _bf16(add, "add", x.shape)
    xn = torch.empty_like(x)
    y = None if add is None else torch.empty_like(x)
    if not x.shape[0]:
        return xn if add is None else (y, xn)
    _check(lib().yoco_norm_rows(_dev(x, "x"), None if add is None else _dev(add, "add"), None if y is None else _dev(y, "y"),
                                _dev(gain, "gain"), _dev(xn, "xn"), x.shape[0], x.shape[1], eps, _stream()))
    return xn if add is None else (y, xn)


def glu_rows(gu):
    """bf16 [rows, 2 ffn] -> swish(first half) * second half (yoco_glu_rows)."""
    if gu.dim() != 2 or gu.shape[1] % 2:
        raise YocoError("gu must be [rows, 2 ffn]")
    _bf16(gu, "gu", gu.shape)
    h = torch.empty((gu.shape[0], gu.shape[1] // 2), dtype=gu.dtype, device=gu.device)
    if not h.shape[0]:
        return h
    _check(lib().yoco_glu_rows(_dev(gu, "gu"), _dev(h, "h"), h.shape[0], h.shape[1], _stream()))
    return h


def ceiling_mfma(seed, sink, iters, workgroups):
    """Launch the MFMA-only loop (yoco_ceiling_mfma); returns the flops of the launch."""
    _check(lib().yoco_ceiling_mfma(_dev(seed, "seed"), _dev(sink, "sink"), iters, workgroups, _stream()))
    return workgroups * 8 * 8 * iters * 32768.0


def ceiling_attn_loop(seed, sink, iters, workgroups, mode):
    """Launch the attention inner loop on its own (yoco_ceiling_attn_loop; mode 1: LDS-fed products, 2: with the
    softmax work); returns the flops of the launch."""
    _check(lib().yoco_ceiling_attn_loop(_dev(seed, "seed"), _dev(sink, "sink"), iters, workgroups, mode, _stream()))
    return workgroups * 8 * 32 * iters * 32768.0


def ceiling_stream_read(buf, sink, workgroups):
    """Launch the streaming read of `buf` (yoco_ceiling_stream_read); returns the bytes read."""
    nbytes = buf.numel() * buf.element_size()
    _check(lib().yoco_ceiling_stream_read(_dev(buf, "buf"), nbytes, _dev(sink, "sink"), workgroups, _stream()))
    return float(nbytes)
