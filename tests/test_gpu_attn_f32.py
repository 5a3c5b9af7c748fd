"""The fp32 matrix-core prefill kernel at the edges of its tiles of 16 keys and 16 or 32 query rows, both storage types,
against the fp64 oracle."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_2405_05254_amd as yoco  # noqa: E402
import yoco_synth as ys  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,T,Hq,Hkv,d,window,scale", [
    ("f32", 1, 1, 1, 1, 64, 1, None),
    ("f32", 2, 15, 4, 2, 128, 3, None),            # windows shorter than a tile: wavefronts without a visible key
    ("f32", 1, 17, 2, 1, 64, 17, None),
    ("f32", 1, 129, 3, 3, 128, 64, -0.7),          # a negative scale: the smallest products weigh most
    ("f32", 3, 337, 24, 8, 64, 100, None),         # 32-row workgroups, a ragged last one
    ("f32", 1, 2065, 8, 8, 128, 500, None),
    ("bf16", 1, 333, 6, 2, 64, 128, None),
    ("bf16", 2, 70, 2, 2, 128, 70, 0.0),           # no scale: plain means, bf16 storage
])
def test_edges(dtype, B, T, Hq, Hkv, d, window, scale):
    scale = 1.0 / math.sqrt(d) if scale is None else scale
    rng = np.random.default_rng(T + Hq)
    q, k, v = (ys.normal(rng, (B, T, h, d), 1.0, dtype) for h in (Hq, Hkv, Hkv))
    dev = lambda a: torch.from_numpy(a).cuda().to(torch.float32 if dtype == "f32" else torch.bfloat16)  # noqa: E731
    o = yoco.swa_prefill(dev(q), dev(k), dev(v), window, scale).float().cpu().numpy()
    pos0 = T - T // 3                              # the last third again, as rows that follow a cache
    cache = yoco.KVCache(1, Hkv, d, T, torch.float32 if dtype == "f32" else torch.bfloat16)
    yoco.global_kv_write(cache, dev(k[B - 1]), dev(v[B - 1]), 0, 0)
    rows = [None] if pos0 == T else [yoco.cross_attn_prefill(cache, dev(q[B - 1, pos0:]), 0, pos0, scale).float().cpu().numpy()]
    tol = ys.TOL[dtype]
    pairs = [(o[b], oracle.swa(q[b], k[b], v[b], window, scale)) for b in range(B)]
    if rows[0] is not None:
        pairs.append((rows[0], oracle.cross_attn(q[B - 1, pos0:], k[B - 1], v[B - 1], pos0, scale)))
    for got, ref in pairs:
        st = ys.error_stats(got, ref)
        assert np.isfinite(got).all() and st["max_abs"] <= tol["max_abs"] and st["mean_rel"] <= tol["mean_rel"], st


@pytest.mark.parametrize("d,T,H", [(64, 70, 2), (128, 70, 2), (64, 2065, 8)])     # 16- and 32-row workgroups
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_values_that_a_query_does_not_see_do_not_reach_it(d, T, H, value):
    window, at = 24, 37
    rng = np.random.default_rng(d + T)
    q, k, v = (ys.normal(rng, (1, T, H, d), 1.0, "f32") for _ in range(3))
    ref = oracle.swa(q[0], k[0], v[0], window, 1.0 / math.sqrt(d))
    v[0, at, :, 3] = value
    o = yoco.swa_prefill(*(torch.from_numpy(a).cuda() for a in (q, k, v)), window, 1.0 / math.sqrt(d))[0].cpu().numpy()
    sees = np.zeros((T, H, d), bool)
    sees[at:at + window, :, 3] = True
    assert not np.isfinite(o[sees]).any()
    st = ys.error_stats(o[~sees], ref[~sees])
    assert np.isfinite(o[~sees]).all() and st["max_abs"] <= ys.TOL["f32"]["max_abs"] and st["mean_rel"] <= ys.TOL["f32"]["mean_rel"], st


@pytest.mark.parametrize("dtype,d,T,H", [("f32", 128, 70, 2), ("bf16", 64, 70, 3), ("f32", 64, 2065, 8)])     # 16- and 32-row workgroups
def test_outputs_in_the_place_of_the_queries(dtype, d, T, H):
    """Also where an infinite value has rows done again: bit for bit what a fresh output gets."""
    g = torch.Generator(device="cuda")
    g.manual_seed(T + d)
    q, k, v = (torch.randn(1, T, H, d, device="cuda", generator=g).to(torch.float32 if dtype == "f32" else torch.bfloat16) for _ in range(3))
    v[0, 37, :, 3] = float("inf")
    ref = yoco.swa_prefill(q, k, v, 24, 0.1)
    got = yoco.swa_prefill(q, k, v, 24, 0.1, out=q)
    assert got is q and torch.equal(got.nan_to_num(nan=7.0), ref.nan_to_num(nan=7.0))
