"""The token step's matrix-vector kernels where one form gives way to the next: input rows held in registers up to 1024, 2048, 3072
and 6144 elements and in LDS beyond, outputs that are no multiple of a workgroup's, against the same stack as torch ops."""
import pytest

torch = pytest.importorskip("torch")

import paper_2405_05254_amd as yoco  # noqa: E402,F401

pytestmark = pytest.mark.gpu


def random_stack(Hq, dm, ffn, vocab):
    gen = torch.Generator(device="cuda").manual_seed(dm + ffn)

    def mat(*shape):
        return (torch.randn(shape, device="cuda", generator=gen) / shape[0] ** 0.5).bfloat16()

    def gain():
        return (1 + 0.2 * torch.randn(dm, device="cuda", generator=gen)).bfloat16()
    qd = 128 * Hq

    def rest():
        return dict(ln1=gain(), ln2=gain(), W_Q=mat(dm, qd), W_O=mat(qd, dm), W_G=mat(dm, ffn), W_1=mat(dm, ffn), W_2=mat(ffn, dm))
    return dict(Hq=Hq, Hkv_self=Hq, Hkv=Hq, d=128, window=64, eps=1e-6, embed=mat(vocab, dm), final_ln=gain(), W_out=mat(dm, vocab),
                self=[dict(W_K=mat(dm, qd), W_V=mat(dm, qd), **rest())], kv=dict(ln=gain(), W_K=mat(dm, qd), W_V=mat(dm, qd)), cross=[rest()])


@pytest.mark.parametrize("Hq,dm,ffn,vocab", [
    (1, 8, 8, 1),                  # one piece of a row, one output
    (8, 1024, 3072, 1001),         # the last element that each form takes
    (9, 1032, 3080, 1003),         # and one piece more
    (16, 2048, 6144, 16387),
    (17, 2056, 6152, 97),
])
def test_token_steps_where_the_kernels_change(Hq, dm, ffn, vocab):
    import copy

    from paper_2405_05254_amd.stack import YocoStack
    w = random_stack(Hq, dm, ffn, vocab)
    logits = []
    for native in (True, False):
        st = YocoStack(copy.deepcopy(w), torch.bfloat16, glue_dtype=torch.bfloat16)
        assert st._native is not None
        if not native:
            st._native = None
        state = st.new_generation_state(20)
        toks = torch.arange(20, device="cuda") % vocab
        logits.append(torch.cat([st.prefill(toks[:15], state)] + [st.decode_step(t, state) for t in toks[15:]]).double())
    got, ref = logits
    assert ((got - ref).norm() / ref.norm()).item() < 1.5e-2         # bf16 roundings that fall the other way, over four layer halves


@pytest.mark.parametrize("Hq,dm,ffn,vocab", [
    (1, 8, 8, 11),
    (1, 520, 8, 524),
    (2, 1024, 16, 1001),
    (2, 1032, 16, 1033),
    (2, 2048, 16, 16387),          # the classifier's two outputs a wavefront, three in its last workgroup
    (2, 2056, 16, 16385),
    (2, 4104, 16, 4110),
])
def test_a_token_is_normed_as_a_row_of_a_prompt(Hq, dm, ffn, vocab):
    """Layers that add nothing and a classifier that copies: the logits are the normed row itself, every one of them, so that a
    sum in another order (which moves 1 element in some 30000 by a bf16 step) and an output out of place both show."""
    from paper_2405_05254_amd import binding as yb
    from paper_2405_05254_amd.stack import YocoStack
    w = random_stack(Hq, dm, ffn, vocab)
    for L in w["self"] + w["cross"]:
        for n in ("W_O", "W_2"):
            L[n].zero_()
    at = torch.arange(vocab, device="cuda") % dm
    w["W_out"] = torch.zeros(dm, vocab, device="cuda").index_put_((at, torch.arange(vocab, device="cuda")), torch.ones((), device="cuda")).bfloat16()
    gen = torch.Generator(device="cuda").manual_seed(dm)
    steps = 400
    w["embed"] = (torch.randn(steps, dm, device="cuda", generator=gen) * torch.randn(steps, dm, device="cuda", generator=gen).exp()).bfloat16()
    st = YocoStack(w, torch.bfloat16, glue_dtype=torch.bfloat16)
    assert st._native is not None
    state = st.new_generation_state(steps)
    toks = torch.arange(steps, device="cuda")
    st.prefill(toks[:1], state)
    got = torch.cat([st.decode_step(t, state) for t in toks[1:]])
    want = yb.norm_rows(st.embed[1:], st.final_ln, st.eps)[:, at]
    assert torch.equal(got, want), (got != want).sum().item()


@pytest.mark.parametrize("cache,rows", [("bf16", 2944), ("bf16", 2945), ("int8", 5709), ("int8", 5710)])
def test_token_steps_over_caches_around_what_counts_as_short(cache, rows):
    """16 heads of up to 23 MB of rows: the cross-decoder's attention reads the weights behind it ahead; of a row more not."""
    import copy

    from paper_2405_05254_amd.stack import YocoStack
    w = random_stack(16, 256, 264, 500)
    gen = torch.Generator(device="cuda").manual_seed(rows)
    K, V = (torch.randn(rows, 16, 128, device="cuda", generator=gen).bfloat16() for _ in range(2))
    logits = []
    for native in (True, False):
        st = YocoStack(copy.deepcopy(w), torch.bfloat16, glue_dtype=torch.bfloat16, cache_dtype=torch.int8 if cache == "int8" else torch.bfloat16)
        if not native:
            st._native = None
        state = st.new_generation_state(rows)
        for c in state["rings"]:
            yoco.global_kv_write(c, K[:64], V[:64], 0, 0)
        yoco.global_kv_write(state["cache"], K, V, 0, 0)
        state["length"] = rows - 1                                     # the step stores the last row anew
        logits.append(st.decode_step(torch.tensor(7, device="cuda"), state).double())
    got, ref = logits
    assert ((got - ref).norm() / ref.norm()).item() < 1.5e-2
