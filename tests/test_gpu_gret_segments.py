"""Chunkwise gated retention at the edges of its chunks of 64 rows and of its segments, every combination of GroupNorm and
gate, and a carried state that is updated in place, against the fp64 oracle."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_2405_05254_amd as yoco  # noqa: E402
import yoco_synth as ys  # noqa: E402

pytestmark = pytest.mark.gpu
D = 128


@pytest.mark.parametrize("B,T,H,chunk,norm,gate,carry", [
    (1, 1, 1, 128, True, True, True),          # one row
    (3, 63, 2, 256, True, False, False),       # one chunk, one row short; one segment, no state before it
    (1, 64, 3, 128, False, True, True),
    (2, 65, 1, 256, True, True, True),         # one row in the second chunk
    (1, 257, 5, 128, False, False, True),      # four segments folded
    (1, 321, 2, 128, True, True, True),        # six chunks in six segments: the scan
    (1, 1100, 1, 1024, True, True, True),      # the workspace of large chunks holds few states: longer segments
    (2, 640, 130, 128, True, False, True),     # so many heads that a sequence is one segment
    (1, 129, 2, 128, True, False, True),       # three chunks in three segments, of which launch 3 folds two
    (4, 400, 24, 256, True, True, True),       # two segments of four chunks, the last of which is short of one
    (4, 300, 24, 256, False, True, True),      # five chunks that one launch walks
    (1, 700, 48, 256, True, True, False),      # a workgroup per CU for most of it
])
def test_edges(B, T, H, chunk, norm, gate, carry):
    scale = 1.0 / math.sqrt(D)
    q, k, v, lg = ys.gret_inputs(T + H, B, T, H, D, D, 1.0, "bf16", mean_log_decay=0.1)
    rng = np.random.default_rng(3)
    g = ys.normal(rng, (B, T, H, D), 1.0, "bf16")
    S0 = rng.standard_normal((B, H, D, D)).astype(np.float32)
    dev = lambda a: torch.from_numpy(a).cuda().to(torch.bfloat16)  # noqa: E731
    state = torch.from_numpy(S0).cuda() if carry else torch.full((B, H, D, D), float("nan"), device="cuda")
    ws = torch.full((yoco.gret_prefill_workspace(B, T, H, D, D, chunk, yoco.BF16),), 0xFF, dtype=torch.uint8, device="cuda")
    o = yoco.gret_prefill(dev(q), dev(k), dev(v), torch.from_numpy(lg).cuda(), scale, chunk=chunk, group_norm=norm, eps=1e-6,
                          state_in=state if carry else None, state_out=state, workspace=ws, gate=dev(g) if gate else None)
    o, state = o.float().cpu().numpy().astype(np.float64), state.cpu().numpy().astype(np.float64)
    for b in range(B):
        ref, S = oracle.gret_recurrent(q[b], k[b], v[b], np.exp(lg[b].astype(np.float64)), scale,
                                       np.swapaxes(S0[b], -1, -2).astype(np.float64) if carry else None)
        S = np.swapaxes(S, -1, -2)
        if norm:
            ref = oracle.group_norm_heads(ref, 1e-6)
        if gate:
            ref = ref * g[b] / (1.0 + np.exp(-g[b].astype(np.float64)))
        for got, want, (most, mean) in ((o[b], ref, (2e-2, 2e-3)), (state[b], S, (2e-3, 1e-3))):
            unit = max(1.0, float(np.abs(want).max()))
            st = ys.error_stats(got / unit, want / unit)
            assert np.isfinite(got).all() and st["max_abs"] <= most and st["mean_rel"] <= mean, (b, st)


@pytest.mark.parametrize("T", [64, 129])         # the outputs' launch alone; the launch that adds up the first of three segments
def test_what_is_split_is_the_rounded_product(T):
    """Row j of the first chunk has a dim of K to itself, so that its row of the state is the high and the low part of v times its weight,
    which is the same in all heads: there is one float32 weight by which all 128 x 16 of them are bf16(x) + bf16(x - bf16(x)) of the
    rounded x = v w."""
    H, rng = 16, np.random.default_rng(T)
    bf16 = lambda x: torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(torch.bfloat16).float().numpy()  # noqa: E731
    k, v = np.zeros((1, T, H, D), np.float32), bf16(rng.standard_normal((1, T, H, D)))
    k[0, np.arange(64), :, np.arange(64)] = 1.0
    lg = np.zeros((1, T, H), np.float32)
    lg[0, :64] = -rng.exponential(0.04, (64, 1))
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    state = torch.empty((1, H, D, D), dtype=torch.float32, device="cuda")
    ws = torch.empty(yoco.gret_prefill_workspace(1, T, H, D, D, 256, yoco.BF16), dtype=torch.uint8, device="cuda")
    kd, vd = dev(k).to(torch.bfloat16), dev(v).to(torch.bfloat16)
    yoco.gret_prefill(kd, kd, vd, dev(lg), 1.0, chunk=256, state_out=state, workspace=ws)
    state = state.cpu().numpy()                                  # [.., dv, dk]
    of_both = 0
    for j in range(63):
        got, x = state[0, :, :, j], v[0, j]
        w0 = np.float32(np.exp(lg[0, j + 1:64, 0].astype(np.float64).sum()))
        found = False
        for ulps in sorted(range(-64, 65), key=abs):             # sums of 63 logarithms in fp32, below 8 in size: some 1e-6 of w
            w = (w0.view(np.int32) + np.int32(ulps)).view(np.float32)
            rounded, exact = x * w, x.astype(np.float64) * np.float64(w)
            hi = bf16(rounded)
            if np.array_equal(got, hi + bf16(rounded - hi)):
                found = True
                fused = (exact - hi).astype(np.float32)          # what a fused multiply-add gives
                of_both += int((bf16(fused) != bf16(rounded - hi)).sum())
                break
        assert found, j
    assert of_both > 20                                          # two formulas that agreed everywhere would prove nothing
