"""One token through a bf16 stack in one call (yoco_stack_step) and the row-wise passes of its prompts, against the same
stack as torch ops: the same roundings in the same places, so the two differ by the order of fp32 sums alone."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2405_05254_amd as yoco  # noqa: E402
import yoco_synth as ys  # noqa: E402

pytestmark = pytest.mark.gpu


def stack_config(Hq, Hkv_self, Hkv, dm, ffn, vocab, kind):
    return dict(d_model=dm, Hq=Hq, Hkv_self=Hkv_self, Hkv=Hkv, d=128, n_self=2, n_cross=2, window=64, ffn=ffn, vocab=vocab, eps=1e-6, self_kind=kind)


@pytest.mark.parametrize("Hq,Hkv_self,Hkv,dm,ffn,vocab,kind,cache", [
    (2, 2, 1, 256, 704, 1001, "swa", "bf16"),        # odd vocabulary: surplus rows of the last workgroup
    (4, 2, 4, 520, 1032, 300, "swa", "int8"),        # widths that are no multiple of a wavefront's 512 elements
    (17, 17, 17, 2184, 4104, 16390, "swa", "bf16"),  # more than one trip over K (2048), the wide classifier's variant
    (17, 1, 1, 128, 256, 99, "swa", "bf16"),         # more heads per KV head than the fused decode serves: the row is appended by itself
    (34, 2, 17, 256, 256, 50, "swa", "bf16"),
    (3, 3, 3, 384, 1056, 97, "gret", "bf16"),        # gated retention: log-decay rows behind the projections, odd head count
])
def test_bf16_stack_matches_the_torch_ops(Hq, Hkv_self, Hkv, dm, ffn, vocab, kind, cache):
    from paper_2405_05254_amd.stack import YocoStack
    w = ys.stack_weights(3, stack_config(Hq, Hkv_self, Hkv, dm, ffn, vocab, kind), "bf16")
    if kind == "gret":
        for L in w["self"]:
            L["W_gamma"] = (L["W_gamma"] * 0.05).astype(np.float32)
    for L in w["self"] + w["cross"] + [w["kv"]]:                     # gains that matter
        for n in ("ln1", "ln2", "ln"):
            if n in L:
                L[n] = (1.0 + 0.2 * np.random.default_rng(7).standard_normal(L[n].shape)).astype(np.float32)
    cdt = torch.int8 if cache == "int8" else torch.bfloat16
    new, old = (YocoStack(w, torch.bfloat16, glue_dtype=torch.bfloat16, cache_dtype=cdt) for _ in range(2))
    assert new._native is not None
    old._native = None
    toks = torch.from_numpy(ys.tokens(1, 75, vocab)).cuda()
    got, ref = [], []
    for st, out in ((new, got), (old, ref)):
        state = st.new_generation_state(75)
        out.append(st.prefill(toks[:70], state))
        for t in toks[70:]:
            out.append(st.decode_step(t, state))
        assert state["length"] == 75
        out.append(st.forward_early_exit(toks)[0])
    got, ref = torch.cat(got).double(), torch.cat(ref).double()
    assert got.shape == ref.shape == (7, vocab)
    assert ((got - ref).norm() / ref.norm()).item() < 1.5e-2         # bf16 roundings that fall the other way, over eight layer halves
    assert (got[5] - got[6]).norm() < 3e-2 * got[6].norm()           # token by token against the early-exit prefill


@pytest.mark.parametrize("rows,dim", [(1, 8), (3, 2048), (5, 4104), (2, 16384)])
def test_row_passes(rows, dim):
    g = torch.Generator(device="cuda")
    g.manual_seed(dim)
    x, add = (torch.randn(rows, dim, device="cuda", generator=g).bfloat16() for _ in range(2))
    gain = (1 + 0.1 * torch.randn(dim, device="cuda", generator=g)).bfloat16()
    from paper_2405_05254_amd import binding as yb

    def norm(t):
        f = t.float()
        return (f * torch.rsqrt(f.pow(2).mean(-1, keepdim=True) + 1e-6) * gain.float()).bfloat16().float()
    y, xn = yb.norm_rows(x, gain, 1e-6, add=add)
    assert torch.equal(y, x + add)
    for got, ref in ((xn, norm(x + add)), (yb.norm_rows(x, gain, 1e-6), norm(x))):
        assert ((got.float() - ref).abs() <= 2 ** -7 * ref.abs()).all()       # one bf16 step at most
    gu = torch.randn(rows, 2 * dim, device="cuda", generator=g).bfloat16()
    ref = (torch.nn.functional.silu(gu[:, :dim]) * gu[:, dim:]).float()
    assert ((yb.glu_rows(gu).float() - ref).abs() <= 2 ** -6 * ref.abs() + 1e-30).all()
    with pytest.raises(yoco.YocoError):
        yb.norm_rows(x[:, ::2], gain, 1e-6)


def small_stack(kind):
    from paper_2405_05254_amd.stack import YocoStack
    w = ys.stack_weights(3, stack_config(2, 2, 2, 256, 704, 200, kind), "bf16")
    return YocoStack(w, torch.bfloat16, glue_dtype=torch.bfloat16)


def test_rows_of_any_stride_and_alignment_are_accepted():
    st = small_stack("swa")
    X = st.self_decoder(torch.from_numpy(ys.tokens(1, 40, 200)).cuda())
    cache = st.write_cache(X)
    wide = torch.zeros(40, 260, dtype=X.dtype, device="cuda")
    wide[:, 3:259] = X
    shifted = torch.zeros(40 * 256 + 1, dtype=X.dtype, device="cuda")[1:].view(40, 256)
    shifted.copy_(X)
    ref, last = st.cross_decoder_rows(X, cache, 0), st.cross_decoder_decode(X[39:], cache, 40)
    for view in (wide[:, 3:259], shifted):
        assert torch.equal(st.cross_decoder_rows(view, cache, 0), ref)
        assert torch.equal(st.cross_decoder_decode(view[39:], cache, 40), last)


@pytest.mark.parametrize("kind", ["swa", "gret"])
def test_a_state_whose_caches_were_replaced_by_copies(kind):
    st = small_stack(kind)
    toks = torch.from_numpy(ys.tokens(1, 40, 200)).cuda()
    state = st.new_generation_state(48)
    st.prefill(toks[:30], state)
    fork = st.new_generation_state(48)
    held = dict(fork, rings=[r for r in fork["rings"]], length=30)
    for n, r in enumerate(state["rings"]):
        if kind == "gret":
            held["rings"][n] = r.clone()
        else:
            held["rings"][n] = yoco.KVCache(1, 2, 128, st.window, torch.bfloat16)
            held["rings"][n].mem.copy_(r.mem)
    held["cache"].mem.copy_(state["cache"].mem)
    for t in toks[30:34]:
        a, b = st.decode_step(t, state), st.decode_step(t, held)
        assert torch.equal(a, b)


def test_rows_that_do_not_fit_the_stack_are_refused():
    st = small_stack("swa")
    X = st.self_decoder(torch.from_numpy(ys.tokens(1, 40, 200)).cuda())
    cache = st.write_cache(X)
    for bad in (X[38:], X[39:].float(), X[39:, :128]):
        with pytest.raises(RuntimeError):
            st.cross_decoder_decode(bad, cache, 40)
    for bad in (X.float(), X[:, :128].contiguous()):
        with pytest.raises(RuntimeError):
            st.cross_decoder_rows(bad, cache, 0)
        with pytest.raises(RuntimeError):
            st.write_cache(bad)
    again = st.write_cache(X[:, None])                               # rows with a dim of 1 between: as torch ops take them
    assert torch.allclose(again.planes()[0].float(), cache.planes()[0].float(), rtol=2 ** -6, atol=1e-3)


def weights_on_device(kind="swa"):
    """The small stack's weights as bf16 GPU tensors, which a stack takes as they are."""
    w = ys.stack_weights(3, stack_config(2, 2, 2, 256, 704, 200, kind), "bf16")

    def dev(x):
        return torch.as_tensor(x).to("cuda", torch.bfloat16)
    for holder in w["self"] + w["cross"] + [w["kv"], w]:
        for n, x in holder.items():
            if isinstance(x, np.ndarray):
                holder[n] = dev(x)
    gen = torch.Generator(device="cuda").manual_seed(5)
    for holder, names in [(L, ("ln1", "ln2")) for L in w["self"] + w["cross"]] + [(w["kv"], ("ln",)), (w, ("final_ln",))]:
        for n in names:
            holder[n] = (1 + 0.2 * torch.randn(256, device="cuda", generator=gen)).bfloat16()
    return w


def request(st, toks):
    """Logits of a prompt's last row, of four token steps and of the early exit over all of it."""
    state = st.new_generation_state(48)
    out = [st.prefill(toks[:30], state)] + [st.decode_step(t, state) for t in toks[30:34]]
    return torch.cat(out + [st.forward_early_exit(toks[:34])[0]]).float()


def as_torch_ops(w):
    """The same stack in torch ops, on weights of its own."""
    import copy

    from paper_2405_05254_amd.stack import YocoStack
    st = YocoStack(copy.deepcopy(w), torch.bfloat16, glue_dtype=torch.bfloat16)
    st._native = None
    return st


def close(got, ref):
    return ((got - ref).norm() / ref.norm()).item() < 1.5e-2          # as in test_bf16_stack_matches_the_torch_ops


@pytest.mark.parametrize("how", ["strided", "misaligned"])
def test_gains_of_any_stride_and_alignment(how):
    from paper_2405_05254_amd.stack import YocoStack
    w = weights_on_device()
    toks = torch.from_numpy(ys.tokens(1, 40, 200)).cuda()
    ref = request(as_torch_ops(w), toks)
    for holder, names in [(L, ("ln1", "ln2")) for L in w["self"] + w["cross"]] + [(w["kv"], ("ln",)), (w, ("final_ln",))]:
        for n in names:
            room = torch.zeros(256 * 2 + 1, dtype=torch.bfloat16, device="cuda")
            view = room[0:512:2] if how == "strided" else room[1:257]
            holder[n] = view.copy_(holder[n])
    st = YocoStack(w, torch.bfloat16, glue_dtype=torch.bfloat16)
    assert st._native is not None and close(request(st, toks), ref)


def test_stacks_without_a_native_step_run_as_torch_ops():
    """What torch ops take, or refuse only where it is used, does not keep a stack from being made or served."""
    from paper_2405_05254_amd.stack import YocoStack
    toks = torch.from_numpy(ys.tokens(1, 40, 200)).cuda()
    w = weights_on_device()
    w["cross"][1]["ln2"] = torch.full((1,), 1.25, dtype=torch.bfloat16, device="cuda")        # one gain for every column
    w["self"][0]["ln1"] = w["self"][0]["ln1"][None]
    st = YocoStack(w, torch.bfloat16, glue_dtype=torch.bfloat16)
    got = request(st, toks)
    w["cross"][1]["ln2"], w["self"][0]["ln1"] = w["cross"][1]["ln2"].expand(256), w["self"][0]["ln1"][0]
    assert close(request(YocoStack(w, torch.bfloat16, glue_dtype=torch.bfloat16), toks), got)
    w = weights_on_device()
    w["Hkv"] = 1                                                     # fewer heads than W_K of Eq. 2 has columns for
    st = YocoStack(w, torch.bfloat16, glue_dtype=torch.bfloat16)
    X = st.self_decoder(toks)                                        # the self-decoder does not mind
    with pytest.raises(RuntimeError):
        st.write_cache(X)
    w["Hkv"], w["kv"]["W_K"] = 2, w["kv"]["W_K"][:, :128].contiguous()    # a matrix that is too small for the native step to read
    st = YocoStack(w, torch.bfloat16, glue_dtype=torch.bfloat16)
    with pytest.raises(RuntimeError):
        st.decode_step(toks[0], st.new_generation_state(8))


def replaced(w, st, how):
    """Something else in the place of a weight or setting, in a stack and in the dict that its reference is made from."""
    gen = torch.Generator(device="cuda").manual_seed(9)

    def like(t, scale=1.0, shift=0.0):
        return (shift + scale * torch.randn(t.shape, device="cuda", generator=gen)).bfloat16()
    if how == "matrices":
        for mine, theirs, names in ((st.self_layers[0], w["self"][0], ("W_Q", "W_2")), (st.cross_layers[1], w["cross"][1], ("W_G",)), (st.kv, w["kv"], ("W_V",))):
            for n in names:
                mine[n] = theirs[n] = like(mine[n], 0.0625)
        st.W_out = w["W_out"] = like(st.W_out, 0.0625)
    elif how == "gains":
        for mine, theirs, n in ((st.self_layers[1], w["self"][1], "ln1"), (st.cross_layers[0], w["cross"][0], "ln2"), (st.kv, w["kv"], "ln")):
            mine[n] = theirs[n] = like(mine[n], 0.3, 1.0)
        st.final_ln = w["final_ln"] = like(st.final_ln, 0.3, 1.0)
    elif how == "transposed":                                        # the same memory, read the other way
        st.self_layers[1]["W_O"] = st.self_layers[1]["W_O"].t()
        w["self"][1]["W_O"] = w["self"][1]["W_O"].t()
    elif how == "data":                                              # the same tensor, other memory
        st.cross_layers[0]["W_Q"].data = w["cross"][0]["W_Q"] = like(st.cross_layers[0]["W_Q"], 0.0625)
    elif how == "layer":
        st.cross_layers[0] = dict(st.cross_layers[0], W_1=like(st.cross_layers[0]["W_1"], 0.0625))
        w["cross"][0] = dict(w["cross"][0], W_1=st.cross_layers[0]["W_1"].clone())
    elif how == "fewer layers":
        del st.cross_layers[0], w["cross"][0]
    elif how == "wider":
        for mine, theirs in zip(st.self_layers + st.cross_layers, w["self"] + w["cross"]):
            for n, shape in (("W_G", (256, 1408)), ("W_1", (256, 1408)), ("W_2", (1408, 256))):
                mine[n] = theirs[n] = like(torch.empty(shape), 0.0442)
    else:
        st.scale = 0.02


@pytest.mark.parametrize("how", ["matrices", "gains", "transposed", "data", "layer", "fewer layers", "wider", "setting"])
def test_what_was_replaced_after_construction_counts(how):
    """In prompts and token steps alike, also between the steps of a request."""
    from paper_2405_05254_amd.stack import YocoStack
    w = weights_on_device()
    toks = torch.from_numpy(ys.tokens(1, 40, 200)).cuda()
    st = YocoStack(w, torch.bfloat16, glue_dtype=torch.bfloat16)
    first = request(st, toks)
    replaced(w, st, how)
    other = as_torch_ops(w)
    if how == "setting":
        other.scale = st.scale
    ref = request(other, toks)
    assert not close(first, ref)                                     # it matters
    assert close(request(st, toks), ref) and st._native is not None
    w = weights_on_device()
    st, other = YocoStack(w, torch.bfloat16, glue_dtype=torch.bfloat16), as_torch_ops(w)
    steps = []
    for s in (st, other):
        state = s.new_generation_state(48)
        s.prefill(toks[:30], state)
        w2 = weights_on_device()
        replaced(w2, s, how)
        if how == "data":
            s.cross_layers[0]["W_Q"].data = s.cross_layers[0]["W_Q"].data.clone()
        steps.append(torch.cat([s.decode_step(t, state) for t in toks[30:34]]).float())
    assert close(*steps)


@pytest.mark.parametrize("how", ["deepcopy", "pickle", "copy"])
def test_a_stack_can_be_copied(how):
    import copy
    import pickle
    st = small_stack("swa")
    toks = torch.from_numpy(ys.tokens(1, 40, 200)).cuda()
    ref = request(st, toks)
    other = dict(deepcopy=copy.deepcopy, pickle=lambda x: pickle.loads(pickle.dumps(x)), copy=copy.copy)[how](st)
    assert other._native is not None and torch.equal(request(other, toks), ref)
    L = other.self_layers[0]
    assert L["W_Q"].data_ptr() == L["w_in"].data_ptr()               # one copy of each weight, here too
    if how != "copy":                                                # which shares the layers
        L["W_Q"].zero_()
    other.final_ln = other.final_ln * 2
    assert not close(request(other, toks), ref) and torch.equal(request(st, toks), ref)
    st._native = None                                                # torch ops stay torch ops
    assert copy.copy(st)._native is None and copy.deepcopy(st)._native is None


def test_a_cache_without_rows_is_attended_to():
    """Attention over no rows is zero; the rest of the layer runs."""
    st = small_stack("swa")
    X = st.self_decoder(torch.from_numpy(ys.tokens(1, 40, 200)).cuda())
    cache = st.write_cache(X)
    got = st.cross_decoder_decode(X[39:], cache, 0)
    st._native = None
    assert close(got.float(), st.cross_decoder_decode(X[39:], cache, 0).float())


@pytest.mark.parametrize("cap", [40, 64])
@pytest.mark.parametrize("cache", ["bf16", "int8"])
def test_steps_at_and_past_the_end_of_the_cache(cache, cap):
    """The last row of the cache is stored; past it nothing is, and the rows there are attended to."""
    import ctypes as C
    st = small_stack("swa")
    st.cache_dtype = torch.int8 if cache == "int8" else torch.bfloat16
    toks = torch.from_numpy(ys.tokens(1, cap + 2, 200)).cuda()
    logits, stored = [], []
    for native in (True, False):
        if not native:
            st._native = None
        assert (st._current() is not None) == native
        state = st.new_generation_state(cap)
        kv = state["cache"]
        guarded = torch.full((kv.bytes + 8192,), 0xA5, dtype=torch.uint8, device="cuda")
        kv.mem = guarded[4096:4096 + kv.bytes]
        kv.mem.zero_()
        assert yoco.lib().yoco_kv_cache_init(kv.mem.data_ptr(), kv.bytes, 1, 2, 128, cap, yoco.INT8 if cache == "int8" else yoco.BF16,
                                             C.byref(kv.desc)) == 0
        out = [st.prefill(toks[:cap - 1], state)]
        before = kv.mem.clone()
        for t in toks[cap - 1:]:
            out.append(st.decode_step(t, state))
            assert (guarded[:4096] == 0xA5).all() and (guarded[4096 + kv.bytes:] == 0xA5).all()
            if len(out) == 2:
                held = kv.mem.clone()
                assert not torch.equal(held, before)
            assert torch.equal(kv.mem, held)
        if cache == "bf16":
            rows = [p[:, :, :cap - 1] for p in kv.planes()]
            kv.mem = before
            assert all(torch.equal(a, b[:, :, :cap - 1]) for a, b in zip(rows, kv.planes()))
        logits.append(torch.cat(out).double())
        stored.append(held)
    assert logits[0].shape == (4, 200) and close(*logits)
    if cache == "bf16":
        assert close(*(h.view(torch.bfloat16).double() for h in stored))


@pytest.mark.parametrize("kind", ["swa", "gret"])
def test_errors_against_64_bits_are_those_of_the_torch_ops(kind):
    """Both chains round the same thirty or so intermediates to bf16, so their errors against the fp64 oracle are two draws
    of one size: over three stacks here, and over single rows of larger ones, they differ by 7 % at most. One rounding more
    in each layer half would add an eighth to it, so a quarter more is too much."""
    import oracle
    from paper_2405_05254_amd.stack import YocoStack
    errors = np.zeros(2)
    for seed in (3, 4, 5):
        w = ys.stack_weights(seed, stack_config(4, 4, 4, 512, 1408, 1001, kind), "bf16")
        if kind == "gret":
            for L in w["self"]:
                L["W_gamma"] = ys.round_to(L["W_gamma"] * 0.05, "bf16")
        toks = ys.tokens(seed, 76, 1001)
        ref = torch.from_numpy(oracle.yoco_stack(toks, w)[69:])
        for i in range(2):
            st = YocoStack(w, torch.bfloat16, glue_dtype=torch.bfloat16)
            if i:
                st._native = None
            state, on_gpu = st.new_generation_state(76), torch.from_numpy(toks).cuda()
            got = torch.cat([st.prefill(on_gpu[:70], state)] + [st.decode_step(t, state) for t in on_gpu[70:]]).cpu().double()
            errors[i] += ((got - ref).norm() / ref.norm()).item() ** 2
    print("error against fp64: %.3e, torch ops %.3e" % tuple((errors / 3) ** 0.5))
    assert errors[0] < 1.25 ** 2 * errors[1]
