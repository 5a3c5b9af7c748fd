"""Prefill over a cache with the keys of a query tile shared out over several workgroups, whose partial results a second
launch merges, against the fp64 oracle."""
import math
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_2405_05254_amd as yoco  # noqa: E402
import yoco_synth as ys  # noqa: E402

D = 128
SCALE = 1.0 / math.sqrt(D)
PIECE = (128 * 128 + 2 * 128) * 4          # bytes of one piece's partial result


def plan(cache, q_pos0, Tq, Hq):
    """Pieces that a call is cut into: what it can make use of, in partial results of its query tiles."""
    return yoco.cross_attn_prefill_workspace(cache, q_pos0, Tq, Hq, SCALE) // (PIECE * Hq * ((Tq + 127) // 128)) or 1


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,q_pos0,Tq,pieces", [
    (24, 8, 1482, 23, 8),        # one query tile, three of its wavefronts without rows
    (2, 2, 3000, 129, 0),        # the last tile has one row
    (1, 1, 0, 1000, 0),          # the first query tiles see fewer key tiles than there are pieces
    (3, 1, 64 * 60 - 9, 9, 0),   # the fewest rows that are not a decode step
    (16, 2, 5000, 256, 0),       # whole tiles
    (4, 4, 1, 1600, 0),
    (24, 8, 10, 30, 1),          # too short to cut
])
def test_pieces_of_the_keys_match_the_oracle(Hq, Hkv, q_pos0, Tq, pieces):
    N, rng = q_pos0 + Tq, np.random.default_rng(Tq)
    cache = yoco.KVCache(2, Hkv, D, N + 3, torch.bfloat16)
    cache.mem.fill_(0xFF)                                       # NaN wherever nothing is written
    K, V = (ys.normal(rng, (N, Hkv, D), 1.0, "bf16") for _ in range(2))
    q = ys.normal(rng, (Tq, Hq, D), 1.0, "bf16")
    dev = lambda a: torch.from_numpy(a).cuda().to(torch.bfloat16)  # noqa: E731
    yoco.global_kv_write(cache, dev(K), dev(V), 1, 0)
    n = plan(cache, q_pos0, Tq, Hq)
    assert n == pieces or (pieces == 0 and n > 1)
    nbytes = yoco.cross_attn_prefill_workspace(cache, q_pos0, Tq, Hq, SCALE)
    own = yoco.cross_attn_prefill(cache, dev(q), 1, q_pos0, SCALE)
    ref = oracle.cross_attn(q, K, V, q_pos0, SCALE)
    tol = ys.TOL["bf16"]
    st = ys.error_stats(own.float().cpu().numpy(), ref)
    assert st["max_abs"] <= tol["max_abs"] and st["mean_rel"] <= tol["mean_rel"], st
    if n == 1:
        return
    ws = torch.full((nbytes // 4,), float("nan"), dtype=torch.float32, device="cuda")
    given = yoco.cross_attn_prefill(cache, dev(q), 1, q_pos0, SCALE, workspace=ws)
    assert torch.equal(own, given)                              # whatever the scratch held before
    for part in (nbytes // 2, 1024):                            # fewer pieces, and no room for two
        ws = torch.full((part // 4 + 64,), float("nan"), dtype=torch.float32, device="cuda")
        o = yoco.cross_attn_prefill(cache, dev(q), 1, q_pos0, SCALE, workspace=ws[:part // 4])
        assert torch.isnan(ws[part // 4:]).all()
        st = ys.error_stats(o.float().cpu().numpy(), ref)
        assert st["max_abs"] <= tol["max_abs"] and st["mean_rel"] <= tol["mean_rel"], (part, st)


@pytest.mark.gpu
@pytest.mark.parametrize("B,T,Hq,Hkv,window", [
    (1, 700, 8, 8, 1024),        # a head per XCD, a CU per query tile
    (4, 333, 6, 2, 200),         # grouped heads, windows shorter than the prompt
    (8, 130, 3, 1, 4000),
    (2, 129, 32, 4, 1),          # walks of one length: one KV head after another
    (3, 260, 3, 1, 500),         # heads that eight XCDs do not share evenly
    (1, 2500, 8, 8, 3000),       # long walks
    (9, 300, 24, 24, 1024),      # more KV heads than stay side by side, in two rounds; in more than two rounds
    (26, 260, 16, 16, 1024),
    (5, 900, 12, 6, 1024),       # 30 KV heads: not shared evenly; two query heads on each of 32
    (4, 900, 16, 8, 1024),
    (2, 800, 32, 8, 1024),       # four on each: one KV head after another
    (3, 700, 32, 8, 1024),       # ... but not where an XCD has three KV heads
    (2, 2500, 16, 16, 3000),     # long walks, more of them than CUs
    (6, 300, 24, 24, 1024),      # three query tiles a head that fill nearly a round
    (2, 1400, 24, 8, 1024),      # shared tiles of two KV heads an XCD, just over a round
    (9, 480, 24, 8, 1024),       # ... of nine, in nearly two
])
def test_window_prefill_whichever_tiles_go_first(B, T, Hq, Hkv, window):
    rng = np.random.default_rng(T)
    q = ys.normal(rng, (B, T, Hq, D), 1.0, "bf16")
    k, v = (ys.normal(rng, (B, T, Hkv, D), 1.0, "bf16") for _ in range(2))
    dev = lambda a: torch.from_numpy(a).cuda().to(torch.bfloat16)  # noqa: E731
    o = yoco.swa_prefill(dev(q), dev(k), dev(v), window, SCALE).float().cpu().numpy()
    for b in range(B):
        st = ys.error_stats(o[b], oracle.swa(q[b], k[b], v[b], window, SCALE))
        assert st["max_abs"] <= ys.TOL["bf16"]["max_abs"] and st["mean_rel"] <= ys.TOL["bf16"]["mean_rel"], (b, st)


@pytest.mark.gpu
@pytest.mark.parametrize("B,T,Hq,Hkv,window", [
    (1, 128, 3, 1, 1024),        # whole tiles: 384 columns
    (2, 299, 3, 1, 64),          # a column behind one, windows of a key tile
    (1, 213, 9, 3, 1),           # a column before one, rows that see themselves
    (3, 77, 5, 1, 40),           # wavefronts that begin in a row's heads, one without columns
    (12, 204, 24, 8, 512),       # more workgroups than places, which a head each would need two rounds of
    (1, 131, 64, 1, 1000),       # two rows a tile
    (1, 140, 387, 3, 100),       # 129 heads: a row is more than a tile
    (4, 1500, 14, 2, 512),       # windows of whole tiles
    (8, 331, 16, 8, 300),        # heavier tiles first
    (1, 290, 16, 4, 1024),       # a head each: its last rows are on two wavefronts
    (1, 1100, 32, 8, 2000),
])
def test_query_heads_that_share_a_tile_match_the_oracle(B, T, Hq, Hkv, window):
    rng = np.random.default_rng(T + Hq)
    q = ys.normal(rng, (B, T, Hq, D), 1.0, "bf16")
    k, v = (ys.normal(rng, (B, T, Hkv, D), 1.0, "bf16") for _ in range(2))
    dev = lambda a: torch.from_numpy(a).cuda().to(torch.bfloat16)  # noqa: E731
    out = torch.full((B * T * Hq * D + 4096,), float("nan"), dtype=torch.bfloat16, device="cuda")
    o = yoco.swa_prefill(dev(q), dev(k), dev(v), window, SCALE, out=out[:-4096].view(B, T, Hq, D)).float().cpu().numpy()
    assert torch.isnan(out[-4096:]).all()
    for b in range(B):
        st = ys.error_stats(o[b], oracle.swa(q[b], k[b], v[b], window, SCALE))
        assert st["max_abs"] <= ys.TOL["bf16"]["max_abs"] and st["mean_rel"] <= ys.TOL["bf16"]["mean_rel"], (b, st)


@pytest.mark.gpu
@pytest.mark.parametrize("B,T,Hq,Hkv,window", [
    (5, 131, 64, 1, 1000),       # two rows a tile: 640 workgroups of a head each, more than a round
    (52, 140, 5, 1, 40),         # wavefronts that begin in a row's heads, a last one with 28 columns
    (65, 100, 7, 1, 1),          # rows that see themselves; the second tile begins in a row's third head
])
def test_heads_share_tiles_beyond_a_round(B, T, Hq, Hkv, window):
    test_query_heads_that_share_a_tile_match_the_oracle(B, T, Hq, Hkv, window)


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,q_pos0,Tq", [
    (24, 8, 20000, 43),          # 129 columns: the second tile has one
    (24, 8, 20000, 42),          # 126
    (5, 1, 30000, 128),          # whole tiles, in as many pieces as there can be
    (64, 8, 9000, 151),
    (7, 1, 0, 700),              # the first tiles see fewer key tiles than there are pieces
    (130, 1, 3000, 9),           # a row is more than a tile
])
def test_query_heads_that_share_a_tile_in_pieces(Hq, Hkv, q_pos0, Tq):
    test_pieces_of_the_keys_match_the_oracle(Hq, Hkv, q_pos0, Tq, 0 if plan_of(Hq, Hkv, q_pos0, Tq) > 1 else 1)


def plan_of(Hq, Hkv, q_pos0, Tq):
    return plan(yoco.KVCache(2, Hkv, D, q_pos0 + Tq + 3, torch.bfloat16), q_pos0, Tq, Hq)


def on_256_cus():
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the counts are those of 256 CUs")


def written(ws):
    """Partial results that hold something."""
    return int((~torch.isnan(ws.view(-1, PIECE // 4))).any(1).sum())


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,q_pos0,Tq,parts", [
    (24, 8, 1482, 23, 24 * 8),          # a tile a head: 23 rows on one wavefront
    (24, 8, 517, 60, 24 * 5),           # 60 rows on two; of shared tiles one would have all four
    (24, 8, 20000, 42, 8 * 32),         # many key tiles: shared, 126 columns
    (24, 8, 20000, 43, 16 * 32),        # ... 129
    (64, 8, 9000, 151, 80 * 6),
    (16, 16, 18145, 29, 16 * 32),       # two workgroups on a CU, whatever trips the merge takes
    (16, 4, 154, 2447, 320 * 3),        # as many pieces of a head each as of shared tiles, which save 4 %
    (16, 4, 585, 1464, 184 * 4),        # shared, which a cut fits better
    (32, 8, 368, 1965, 0),              # as good as uncut, and so it stays
    (24, 8, 14000, 2000, 384 * 4),
])
def test_which_tiles_a_call_is_cut_into(Hq, Hkv, q_pos0, Tq, parts):
    on_256_cus()
    cache = yoco.KVCache(1, Hkv, D, q_pos0 + Tq, torch.bfloat16)
    cache.mem.zero_()
    q = torch.zeros((Tq, Hq, D), dtype=torch.bfloat16, device="cuda")
    nbytes = yoco.cross_attn_prefill_workspace(cache, q_pos0, Tq, Hq, SCALE)
    assert nbytes >= parts * PIECE and (nbytes > 0) == (parts > 0)
    if parts:
        ws = torch.full((nbytes // 4,), float("nan"), dtype=torch.float32, device="cuda")
        yoco.cross_attn_prefill(cache, q, 0, q_pos0, SCALE, workspace=ws)
        assert written(ws) == parts


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,Tq,tiles,pieces,parts,parts_of_half", [
    (2, 1, 1000, 16, 8, 100, 58),       # rows over themselves: the first tile has one key tile, for one of its pieces
    (3, 1, 513, 13, 9, 65, 35),         # the last tile has a row
    (5, 1, 385, 16, 7, 61, 0),          # half as many pieces are not worth it
    (12, 4, 770, 76, 3, 212, 0),
])
def test_shared_tiles_with_fewer_key_tiles_than_pieces(Hq, Hkv, Tq, tiles, pieces, parts, parts_of_half):
    on_256_cus()
    rng = np.random.default_rng(Tq)
    cache = yoco.KVCache(2, Hkv, D, Tq + 3, torch.bfloat16)
    cache.mem.fill_(0xFF)                                       # NaN wherever nothing is written
    K, V = (ys.normal(rng, (Tq, Hkv, D), 1.0, "bf16") for _ in range(2))
    q = ys.normal(rng, (Tq, Hq, D), 1.0, "bf16")
    dev = lambda a: torch.from_numpy(a).cuda().to(torch.bfloat16)  # noqa: E731
    yoco.global_kv_write(cache, dev(K), dev(V), 1, 0)
    ref, tol = oracle.cross_attn(q, K, V, 0, SCALE), ys.TOL["bf16"]
    assert yoco.cross_attn_prefill_workspace(cache, 0, Tq, Hq, SCALE) >= tiles * pieces * PIECE
    for held, expected in ((tiles * pieces, parts), (tiles * pieces // 2, parts_of_half), (2 * tiles - 1, 0)):
        ws = torch.full((held * PIECE // 4 + 64,), float("nan"), dtype=torch.float32, device="cuda")
        o = yoco.cross_attn_prefill(cache, dev(q), 1, 0, SCALE, workspace=ws[:-64])
        assert written(ws[:-64]) == expected and torch.isnan(ws[-64:]).all()
        st = ys.error_stats(o.float().cpu().numpy(), ref)
        assert st["max_abs"] <= tol["max_abs"] and st["mean_rel"] <= tol["mean_rel"], (held, st)


@pytest.mark.gpu
def test_under_capture_a_call_takes_no_scratch_of_its_own():
    cache, q, pos0, nbytes = _few_tiles(Tq=40, Hq=8)
    kv = [p[0].transpose(0, 1).float().cpu().numpy() for p in cache.planes()]
    ref, tol = oracle.cross_attn(q.float().cpu().numpy(), *kv, pos0, SCALE), ys.TOL["bf16"]
    ws, small = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in (nbytes, 1024))
    cut = yoco.cross_attn_prefill(cache, q, 0, pos0, SCALE, workspace=ws)
    whole = yoco.cross_attn_prefill(cache, q, 0, pos0, SCALE, workspace=small)       # no room for two pieces
    assert torch.equal(yoco.cross_attn_prefill(cache, q, 0, pos0, SCALE), cut) and not torch.equal(cut, whole)
    for o in (cut, whole):                                      # other low-order bits, the same error
        st = ys.error_stats(o.float().cpu().numpy(), ref)
        assert st["max_abs"] <= tol["max_abs"] and st["mean_rel"] <= tol["mean_rel"], st
    for given, out, want in ((None, None, whole), (None, torch.empty_like(q), whole), (ws, torch.empty_like(q), cut)):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            o = yoco.cross_attn_prefill(cache, q, 0, pos0, SCALE, out=out, workspace=given)
        for _ in range(3):
            o.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(o, want)


def _desc(dtype, Hkv, N, d=D):
    import ctypes as C

    from paper_2405_05254_amd import binding as yb
    c = yb._Cache()
    assert yoco.lib().yoco_kv_cache_init(0x7f0000000000, yoco.kv_cache_bytes(1, Hkv, d, N, dtype), 1, Hkv, d, N, dtype, C.byref(c)) == 0
    return c, C


def test_scratch_is_asked_for_where_it_is_of_use_and_bounded():
    L = yoco.lib()
    for dtype, d, Hkv, Hq, pos0, Tq, want in [
            (yoco.BF16, D, 8, 24, 14000, 2000, True), (yoco.BF16, D, 8, 24, 24000, 4096, True), (yoco.BF16, D, 1, 1, 500000, 9, True),
            (yoco.BF16, D, 8, 24, 14000, 8, False),             # few rows use the decode workspace
            (yoco.BF16, D, 8, 24, 0, 300, False), (yoco.BF16, D, 8, 64, 20000, 8192, False),
            (yoco.F32, D, 8, 24, 14000, 2000, False), (yoco.BF16, 64, 8, 24, 14000, 2000, False), (yoco.INT8, D, 8, 24, 14000, 2000, False)]:
        c, C = _desc(dtype, Hkv, pos0 + Tq, d)
        n = C.c_size_t(1)
        assert L.yoco_cross_attn_prefill_workspace(C.byref(c), pos0, Tq, Hq, SCALE, C.byref(n)) == 0
        assert (n.value > 0) == want and n.value <= 1536 * PIECE, (pos0, Tq, n.value)
    assert L.yoco_cross_attn_prefill_workspace(C.byref(c), 14001, 2000, 24, SCALE, C.byref(n)) != 0
    assert L.yoco_cross_attn_prefill_workspace(C.byref(c), 0, 2000, 9, SCALE, C.byref(n)) != 0
    assert L.yoco_cross_attn_prefill_workspace(C.byref(c), 0, 2000, 24, SCALE, None) != 0


def _few_tiles(Tq=64, Hq=16, Hkv=2, N=4000):
    """A call that is cut into pieces: cache, queries, their position and the scratch that the pieces take."""
    cache = yoco.KVCache(1, Hkv, D, N, torch.bfloat16)
    for i, p in enumerate(cache.planes()):
        p.copy_(ys.device_normal(p.shape, i, 1.0, torch.bfloat16, "cuda"))
    q = ys.device_normal((Tq, Hq, D), 2, 1.0, torch.bfloat16, "cuda")
    nbytes = yoco.cross_attn_prefill_workspace(cache, N - Tq, Tq, Hq, SCALE)
    assert plan(cache, N - Tq, Tq, Hq) > 1 and nbytes > 8 << 20
    return cache, q, N - Tq, nbytes


def _taken():
    s = torch.cuda.memory_stats()
    return s["allocation.all.allocated"], s["reserved_bytes.all.current"], s["num_ooms"], s["num_alloc_retries"]


@pytest.mark.gpu
def test_a_call_that_is_given_its_output_allocates_nothing():
    cache, q, pos0, _ = _few_tiles()
    o = torch.empty_like(q)
    before = _taken()
    assert yoco.cross_attn_prefill(cache, q, 0, pos0, SCALE, out=o) is o
    assert _taken() == before
    own = yoco.cross_attn_prefill(cache, q, 0, pos0, SCALE)
    assert _taken()[0] == before[0] + 2                         # the output and the scratch
    assert torch.allclose(o.float(), own.float(), atol=2e-3, rtol=2e-2)


@pytest.mark.gpu
def test_short_memory_costs_a_call_its_scratch_and_nothing_else():
    cache, q, pos0, nbytes = _few_tiles()
    whole = yoco.cross_attn_prefill(cache, q, 0, pos0, SCALE, out=torch.empty_like(q))
    torch.cuda.empty_cache()
    blocks = [torch.empty(512 << 10, dtype=torch.uint8, device="cuda") for _ in range(64)]
    del blocks                                                  # cached in a pool of small blocks, where the scratch does not fit
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + nbytes // 2) / total)
    try:
        before = _taken()
        o = yoco.cross_attn_prefill(cache, q, 0, pos0, SCALE)
        after = _taken()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert after == (before[0] + 1,) + before[1:]               # the output alone; the cached blocks are still there
    assert torch.equal(o, whole)


@pytest.mark.gpu
def test_scratch_leaves_the_capture_of_another_thread_alone():
    cache, q, pos0, _ = _few_tiles()
    side, own, x = torch.cuda.Stream(), [], torch.ones(1000, device="cuda")
    with torch.cuda.stream(side):
        ref = yoco.cross_attn_prefill(cache, q, 0, pos0, SCALE)
        kept = ref.clone()
        del ref
    torch.cuda.synchronize()
    torch.cuda.empty_cache()                                    # the next scratch is the driver's to give

    def other():
        with torch.cuda.stream(side):
            own.append(yoco.cross_attn_prefill(cache, q, 0, pos0, SCALE))

    with torch.cuda.stream(side):
        room = torch.empty_like(q)                              # the next output is not
    del room
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="global"):
        y = x * 2
        t = threading.Thread(target=other)
        t.start()
        t.join()
        y = y + 1
    for _ in range(3):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, torch.full_like(y, 3.0)) and torch.equal(own[0], kept)


@pytest.mark.gpu
def test_a_large_batch_takes_no_longer_a_prompt_than_a_small_one():
    """Prompts of 1900 rows x 24 heads, window 1024: the key tiles of a head stay in the L2 for its query tiles also where a
    launch has 59 of them (26 us a prompt and 28 at four of them; walked side by side 37)."""
    def us_a_prompt(B):
        q, k, v = (torch.zeros(B, 1900, 24, D, dtype=torch.bfloat16, device="cuda") for _ in range(3))
        o, best = torch.empty_like(q), float("inf")
        for _ in range(6):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(4):
                yoco.swa_prefill(q, k, v, 1024, SCALE, out=o)
            end.record()
            end.synchronize()
            best = min(best, start.elapsed_time(end) * 1e3 / (4 * B))
        return best

    assert us_a_prompt(59) < 1.2 * us_a_prompt(4)
