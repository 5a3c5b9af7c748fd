"""The end of a split decode step: splits that meet in the caller's workspace without anything having been cleared or are
left for a merge launch, and ragged batches whose sequences get different numbers of splits, against the fp64 oracle."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_2405_05254_amd as yoco  # noqa: E402
import yoco_synth as ys  # noqa: E402

pytestmark = pytest.mark.gpu
D = 128
SCALE = 1.0 / math.sqrt(D)


@pytest.mark.parametrize("dtype,Hq,Hkv,N_cap,lens", [
    ("bf16", 2, 1, 300, [300, 1, 129]),                     # 1 .. 3 splits of one step each
    ("bf16", 6, 2, 1100, [1100, 1024]),                     # 9 splits: the wider merge
    ("bf16", 4, 1, 2048, [2048]),                           # 16 splits of 4 heads: the most that meet in one launch
    ("bf16", 3, 1, 2300, [2300]),                           # 18 splits: a merge launch
    ("bf16", 16, 2, 1024, [1024, 130]),                     # 8 splits of 8 heads: one launch
    ("bf16", 8, 1, 1100, [1100, 0, 900]),                   # 9 splits of 8 heads: a merge launch, an empty sequence
    ("bf16", 9, 1, 500, [500, 1]),                          # 9 heads: a merge launch however few the splits
    ("int8", 12, 3, 9000, [9000, 12, 0]),                   # 18 splits of 512 rows would need a merge launch: as many of 256 as fill the chip
    ("int8", 5, 1, 4000, [4000, 2000]),                     # 8 splits of 5: one launch
    ("int8", 8, 1, 5000, [5000, 513, 0]),                   # 10 splits of 8, a merge launch: 20 of 256 rows
    ("int8", 16, 1, 513, [513, 512]),                       # 3 splits of 16 heads for a merge launch; one row less is one split
    ("int8", 16, 1, 512, [512, 257]),
    ("int8", 4, 1, 8192, [8192, 300]),                      # 16 splits of 512 rows meet: no finer
    ("int8", 4, 1, 8193, [8193, 300]),                      # 33 of 256
    ("int8", 4, 1, 16384, [16384]),                         # 64 of 256
    ("int8", 4, 1, 16385, [16385]),                         # 33 of 512, not 65
    ("bf16", 16, 1, 9000, [9000, 0, 7, 4400, 128, 127]),    # 16 heads in one workgroup, an empty sequence among long ones
    ("bf16", 9, 3, 1500, [1500, 1, 1499, 700, 0, 800, 129, 1400, 2]),     # many sequences and few units: every one in splits of a step
    ("bf16", 24, 8, 3000, [3000, 375, 0, 2999, 1600, 128, 2100, 900]),    # ... splits to spare from 700 rows on, a CU for each
    ("bf16", 16, 8, 1400, [1400, 200, 1300, 5, 1399, 700, 0, 1, 1200, 300, 1100, 128, 129, 256, 1024, 900, 640]),   # ... of two, at the line
    ("bf16", 16, 8, 1399, [1399, 200, 1300, 5, 1398, 700, 0, 1, 1200, 300, 1100, 128, 129, 256, 1024, 900, 640]),   # ... below it
    ("int8", 24, 8, 3079, [3079, 400, 3000, 0, 257, 1900, 513, 2500, 256]),
    ("int8", 64, 8, 4751, [4751, 600, 3000, 1]),
    ("int8", 8, 8, 1963, [1963, 250, 1500, 0, 1000, 1900, 300, 512, 513, 1200, 800, 64, 1800, 1700]),
    ("bf16", 8, 8, 21000, [20999, 2500, 300, 17, 9000]),    # splits to spare: the long sequences are cut finer than the short
    ("bf16", 12, 12, 1100, [1100, 1100, 1090, 1100, 1100, 1100, 1100]),   # 84 units of equal lengths: 3 splits, not 4
    ("bf16", 12, 12, 1100, [1100, 1100, 900, 1100, 1100, 1100, 1100]),    # ... just past what counts as equal
    ("bf16", 16, 16, 9000, [9000, 1300, 0]),                # 16 places for the splits of three sequences: a CU for each
    ("bf16", 8, 8, 9000, [0, 9000, 5, 8000, 2500, 127]),    # ... of 6, two of them without a split to spare
    ("bf16", 32, 8, 2600, [2600, 1, 1900, 600, 2500, 0, 2570, 1200, 130, 2000, 700, 2599]),
    ("int8", 8, 8, 9000, [9000, 513, 0, 7777]),
    ("bf16", 2, 2, 900, [(i * 379) % 901 for i in range(70)]),            # more sequences than a wavefront has lanes
    ("bf16", 34, 17, 4200, [4200] * 8),                     # 136 units: three splits, on half as many CUs as two rounds have
    ("bf16", 17, 17, 1000, [1000] * 9),                     # 153 units: unsplit, in a workspace for two
    ("int8", 3, 3, 5700, [5700] * 8),                       # 24 units: 10 splits, not 11
    ("int8", 4, 2, 1500, [1500, 513, 64]),
    ("int8", 13, 1, 3000, [2999, 1]),
])
@pytest.mark.parametrize("garbage", [0x00, 0xFF, 0x3F])
def test_splits_meet_in_an_uncleared_workspace(dtype, Hq, Hkv, N_cap, lens, garbage):
    B, rng = len(lens), np.random.default_rng(N_cap)
    cache = yoco.KVCache(B, Hkv, D, N_cap, torch.int8 if dtype == "int8" else torch.bfloat16)
    cache.mem.zero_()
    K, V = (ys.normal(rng, (B, N_cap, Hkv, D), 1.0, "bf16") for _ in range(2))
    q = ys.normal(rng, (B, Hq, D), 1.0, "bf16")
    dev = lambda a: torch.from_numpy(a).cuda().to(torch.bfloat16)  # noqa: E731
    for b in range(B):
        yoco.global_kv_write(cache, dev(K[b]), dev(V[b]), b, 0)
    nbytes, splits = yoco.cross_attn_decode_workspace(cache, Hq)
    ws = torch.full((nbytes,), garbage, dtype=torch.uint8, device="cuda")
    ln = torch.tensor(lens, dtype=torch.int64, device="cuda")
    first = yoco.cross_attn_decode(cache, dev(q), ln, SCALE, ws)
    again = yoco.cross_attn_decode(cache, dev(q), ln, SCALE, ws)         # over what the first call left behind
    assert torch.equal(first, again)
    attend = oracle.cross_attn_int8 if dtype == "int8" else oracle.cross_attn
    tol = ys.TOL["bf16"]
    for b, n in enumerate(lens):
        got = first[b].float().cpu().numpy()
        if n == 0:
            assert not got.any()
            continue
        st = ys.error_stats(got, attend(q[b:b + 1], K[b, :n], V[b, :n], n - 1, SCALE)[0])
        assert st["max_abs"] <= tol["max_abs"] and st["mean_rel"] <= tol["mean_rel"], (b, n, splits, st)


def test_a_workspace_without_splits_to_spare_is_enough():
    """Splits to spare for a ragged batch of short sequences are used where the workspace holds them; half of it holds the others,
    and nothing behind that half is touched."""
    B, Hkv, Hq, N = 8, 8, 24, 3000
    rng = np.random.default_rng(5)
    cache = yoco.KVCache(B, Hkv, D, N, torch.bfloat16)
    for plane in cache.planes():
        plane.copy_(torch.from_numpy(ys.normal(rng, tuple(plane.shape), 1.0, "bf16")))
    q = torch.from_numpy(ys.normal(rng, (B, Hq, D), 1.0, "bf16")).cuda().to(torch.bfloat16)
    lens = [3000, 375, 0, 2999, 1600, 128, 2100, 900]
    ln = torch.tensor(lens, dtype=torch.int64, device="cuda")
    nbytes, splits = yoco.cross_attn_decode_workspace(cache, Hq)
    if splits % 2:
        pytest.skip("no splits to spare on this many CUs")
    K, V = (p.float().cpu().numpy().transpose(0, 2, 1, 3) for p in cache.planes())
    ws = torch.full((nbytes,), 0x5A, dtype=torch.uint8, device="cuda")
    for held in (nbytes // 2, nbytes):
        o = yoco.cross_attn_decode(cache, q, ln, SCALE, ws[:held])
        assert (ws[held:] == 0x5A).all()
        for b, n in enumerate(lens):
            if n == 0:
                assert not o[b].any()
                continue
            st = ys.error_stats(o[b].float().cpu().numpy(), oracle.cross_attn(q[b:b + 1].float().cpu().numpy(), K[b, :n], V[b, :n], n - 1, SCALE)[0])
            assert st["max_abs"] <= ys.TOL["bf16"]["max_abs"] and st["mean_rel"] <= ys.TOL["bf16"]["mean_rel"], (held, b, n, st)
    with pytest.raises(yoco.YocoError):
        yoco.cross_attn_decode(cache, q, ln, SCALE, ws[:nbytes // 2 - 16])


@pytest.mark.parametrize("dtype,Hq,Hkv,d,N_cap,splits,lens", [
    ("int8", 24, 8, 128, 6000, 4, [5999, 6000, 3001] + [(i * 379) % 700 for i in range(14)]),    # 136 units of 8 bits: from 3000 rows a split on
    ("int8", 24, 8, 128, 5999, 2, [5999, 3001] + [(i * 379) % 700 for i in range(15)]),          # ... a row less
    ("bf16", 16, 1, 128, 22400, 62, [22400, 700, 0, 9000, 128, 1, 1400, 350]),                   # for a merge launch, which reads splits without rows too;
    ("int8", 16, 1, 128, 22400, 62, [22400, 700, 0, 9000, 256, 1, 1400, 350]),                   # ... not 64: as many as the static scratch holds
    ("bf16", 9, 1, 128, 22400, 64, [22400, 700, 0, 9000, 128, 1, 1400, 350]),
    ("bf16", 24, 8, 64, 3000, 8, [3000, 0, 1, 2999, 129, 1500, 375, 8]),                         # kernels that cut every length alike
])
def test_splits_to_spare(dtype, Hq, Hkv, d, N_cap, splits, lens):
    B, rng = len(lens), np.random.default_rng(N_cap + Hq)
    cache = yoco.KVCache(B, Hkv, d, N_cap, torch.int8 if dtype == "int8" else torch.bfloat16)
    cache.mem.zero_()
    dev = lambda a: torch.from_numpy(a).cuda().to(torch.bfloat16)  # noqa: E731
    rows = [[ys.normal(rng, (n, Hkv, d), 1.0, "bf16") for _ in range(2)] for n in lens]
    for b, (k, v) in enumerate(rows):
        yoco.global_kv_write(cache, dev(k), dev(v), b, 0)
    q = ys.normal(rng, (B, Hq, d), 1.0, "bf16")
    nbytes, n_splits = yoco.cross_attn_decode_workspace(cache, Hq)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert n_splits == splits
    ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
    o = yoco.cross_attn_decode(cache, dev(q), torch.tensor(lens, dtype=torch.int64, device="cuda"), 1 / math.sqrt(d), ws)
    attend = oracle.cross_attn_int8 if dtype == "int8" else oracle.cross_attn
    for b, n in enumerate(lens):
        got = o[b].float().cpu().numpy()
        if n == 0:
            assert not got.any()
            continue
        st = ys.error_stats(got, attend(q[b:b + 1], *rows[b], n - 1, 1 / math.sqrt(d))[0])
        assert st["max_abs"] <= ys.TOL["bf16"]["max_abs"] and st["mean_rel"] <= ys.TOL["bf16"]["mean_rel"], (b, n, st)


@pytest.mark.parametrize("dtype,Hq,Hkv,N_cap,lens", [
    ("bf16", 33, 33, 640, [640] * 8),                                  # 264 units on 256 CUs: eight of them in five splits of a step
    ("bf16", 33, 33, 640, [640, 1, 0, 639, 129, 384, 385, 640]),       # ... the sequences that are over have other lengths
    ("bf16", 33, 33, 700, [0, 700, 1, 700, 128, 256, 257, 512]),       # ... the first, of which eight units are split, is empty
    ("bf16", 86, 43, 1024, [1024] * 7 + [1023]),                       # 344 units: 88 in two
    ("bf16", 86, 43, 1023, [1023] * 8),                                # ... a row less
    ("bf16", 51, 17, 1000, [1000] * 15 + [3]),
    ("bf16", 264, 33, 1100, [1100] * 8),                               # 8 query heads: as many splits as meet in the launch
    ("bf16", 297, 33, 1100, [1100] * 8),                               # 9: none do
    ("bf16", 4, 4, 700, [700 - i for i in range(70)]),                 # more sequences than a wavefront has lanes
    ("int8", 36, 36, 1024, [1024] * 8),                                # 288 units in eighths, of which a length has as many as it has steps
    ("int8", 36, 36, 1024, [257, 1024, 0, 513, 1, 256, 1000, 64]),
    ("int8", 36, 36, 1023, [1023] * 8),
    ("int8", 96, 48, 1100, [1100] * 8),                                # 384 units: half of what is over, each
])
def test_units_that_are_over_are_split(dtype, Hq, Hkv, N_cap, lens):
    B, rng = len(lens), np.random.default_rng(N_cap + Hq)
    cache = yoco.KVCache(B, Hkv, D, N_cap, torch.int8 if dtype == "int8" else torch.bfloat16)
    cache.mem.zero_()
    dev = lambda a: torch.from_numpy(a).cuda().to(torch.bfloat16)  # noqa: E731
    rows = [[ys.normal(rng, (n, Hkv, D), 1.0, "bf16") for _ in range(2)] for n in lens]
    for b, (k, v) in enumerate(rows):
        yoco.global_kv_write(cache, dev(k), dev(v), b, 0)
    q = ys.normal(rng, (B, Hq, D), 1.0, "bf16")
    ln = torch.tensor(lens, dtype=torch.int64, device="cuda")
    nbytes, splits = yoco.cross_attn_decode_workspace(cache, Hq)
    assert splits == 1 or torch.cuda.get_device_properties(0).multi_processor_count != 256      # the partials of a few units fit one split of all
    ws = torch.full((nbytes + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
    o = yoco.cross_attn_decode(cache, dev(q), ln, SCALE, ws[:nbytes])
    assert torch.equal(o, yoco.cross_attn_decode(cache, dev(q), ln, SCALE, ws[:nbytes]))
    assert torch.equal(o, yoco.cross_attn_decode_noalloc(cache, dev(q), ln, SCALE, torch.empty_like(o)))
    assert (ws[nbytes:] == 0xFF).all()
    attend = oracle.cross_attn_int8 if dtype == "int8" else oracle.cross_attn
    for b, n in enumerate(lens):
        got = o[b].float().cpu().numpy()
        if n == 0:
            assert not got.any()
            continue
        st = ys.error_stats(got, attend(q[b:b + 1], *rows[b], n - 1, SCALE)[0])
        assert st["max_abs"] <= ys.TOL["bf16"]["max_abs"] and st["mean_rel"] <= ys.TOL["bf16"]["mean_rel"], (b, n, st)


@pytest.mark.parametrize("dtype,Hq,Hkv,N_cap,lens,cut", [
    ("bf16", 33, 33, 640, [640] * 8, True),                            # 264 units on 256 CUs, the eight that are over in five parts
    ("bf16", 33, 33, 639, [639] * 8, False),
    ("bf16", 33, 33, 700, [0] + [700] * 7, False),                     # what would be cut is empty
    ("bf16", 33, 33, 700, [384] + [700] * 7, False),                   # ... saves two steps
    ("bf16", 33, 33, 1000, [640] + [700] * 6 + [376], True),           # a CU's two units: 1016 rows, 92 more than 224 over the longest
    ("bf16", 33, 33, 1000, [640] + [700] * 6 + [375], False),          # ... of which a seventh of 640 is more than 91
    ("bf16", 33, 33, 1000, [1000] + [128] * 7, False),                 # the long one is the first
    ("bf16", 24, 24, 1024, [1024] * 11 + [700], True),                 # 288 units: a CU's two are heads of sequences 10 or 11 apart
    ("bf16", 86, 43, 1024, [1024] * 8, True),                          # two parts
    ("bf16", 86, 43, 1023, [1023] * 8, False),
    ("bf16", 32, 32, 1024, [1024] * 8, False),                         # a CU each
    ("bf16", 4, 4, 700, [700 - i for i in range(70)], True),           # more sequences than a wavefront has lanes
    ("bf16", 4, 4, 700, [100] * 70, False),
    ("bf16", 264, 33, 1100, [1100] * 8, True),                         # 8 query heads: parts that meet in the launch
    ("bf16", 297, 33, 1100, [1100] * 8, False),
    ("int8", 36, 36, 1024, [1024] * 8, True),
    ("int8", 36, 36, 1024, [512] * 8, False),                          # two steps of 256
    ("int8", 36, 36, 1024, [1024, 300, 200, 400, 200, 200, 300, 128], True),       # 1152 rows, an eighth of the first over the longest
    ("int8", 36, 36, 1024, [1024, 300, 200, 400, 200, 200, 300, 127], False),
])
def test_the_lengths_say_whether_units_that_are_over_are_cut(dtype, Hq, Hkv, N_cap, lens, cut):
    """Only parts write to the workspace."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the cases are made for 256 CUs")
    B, rng = len(lens), np.random.default_rng(N_cap + Hq)
    cache = yoco.KVCache(B, Hkv, D, N_cap, torch.int8 if dtype == "int8" else torch.bfloat16)
    cache.mem.zero_()
    dev = lambda a: torch.from_numpy(a).cuda().to(torch.bfloat16)  # noqa: E731
    rows = [[ys.normal(rng, (n, Hkv, D), 1.0, "bf16") for _ in range(2)] for n in lens]
    for b, (k, v) in enumerate(rows):
        yoco.global_kv_write(cache, dev(k), dev(v), b, 0)
    q = ys.normal(rng, (B, Hq, D), 1.0, "bf16")
    ln = torch.tensor(lens, dtype=torch.int64, device="cuda")
    nbytes, splits = yoco.cross_attn_decode_workspace(cache, Hq)
    assert splits == 1
    ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
    o = yoco.cross_attn_decode(cache, dev(q), ln, SCALE, ws)
    assert bool((ws != 0xFF).any()) == cut
    attend = oracle.cross_attn_int8 if dtype == "int8" else oracle.cross_attn
    for b, n in enumerate(lens):
        got = o[b].float().cpu().numpy()
        if n == 0:
            assert not got.any()
            continue
        st = ys.error_stats(got, attend(q[b:b + 1], *rows[b], n - 1, SCALE)[0])
        assert st["max_abs"] <= ys.TOL["bf16"]["max_abs"] and st["mean_rel"] <= ys.TOL["bf16"]["mean_rel"], (b, n, st)


def test_few_rows_of_a_batch_use_what_the_documented_workspace_holds():
    """A batch of more (sequence, head) units than CUs has one split per unit: its workspace serves the few-row call of
    one sequence, whose own split count would be larger."""
    cache = yoco.KVCache(40, 8, D, 2600, torch.int8)
    cache.mem.zero_()
    rng = np.random.default_rng(1)
    k, v = (torch.from_numpy(ys.normal(rng, (2600, 8, D), 1.0, "bf16")).cuda().to(torch.bfloat16) for _ in range(2))
    yoco.global_kv_write(cache, k, v, 39, 0)
    q = torch.from_numpy(ys.normal(rng, (1, 8, D), 1.0, "bf16")).cuda().to(torch.bfloat16)
    ws = torch.empty(yoco.cross_attn_decode_workspace(cache, 8)[0], dtype=torch.uint8, device="cuda")
    o = yoco.cross_attn_prefill(cache, q, 39, 2599, SCALE, workspace=ws)
    ref = oracle.cross_attn_int8(q.float().cpu().numpy(), k.float().cpu().numpy(), v.float().cpu().numpy(), 2599, SCALE)
    st = ys.error_stats(o.float().cpu().numpy(), ref)
    assert st["max_abs"] <= 2e-2 and st["mean_rel"] <= 2e-3, st


@pytest.mark.parametrize("dtype,Hq,Hkv,N_cap", [("bf16", 264, 264, 1100), ("bf16", 600, 300, 600), ("int8", 288, 288, 1030)])
def test_few_rows_over_more_heads_than_compute_units_are_whole(dtype, Hq, Hkv, N_cap):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the cases are made for 256 CUs")
    cache = yoco.KVCache(2, Hkv, D, N_cap, torch.int8 if dtype == "int8" else torch.bfloat16)
    cache.mem.zero_()
    rng = np.random.default_rng(N_cap)
    dev = lambda a: torch.from_numpy(a).cuda().to(torch.bfloat16)  # noqa: E731
    k, v = (ys.normal(rng, (N_cap, Hkv, D), 1.0, "bf16") for _ in range(2))
    yoco.global_kv_write(cache, dev(k), dev(v), 1, 0)
    q = ys.normal(rng, (3, Hq, D), 1.0, "bf16")
    ws = torch.full((yoco.cross_attn_decode_workspace(cache, Hq)[0],), 0xFF, dtype=torch.uint8, device="cuda")
    o = yoco.cross_attn_prefill(cache, dev(q), 1, N_cap - 3, SCALE, workspace=ws)
    assert (ws == 0xFF).all()
    attend = oracle.cross_attn_int8 if dtype == "int8" else oracle.cross_attn
    st = ys.error_stats(o.float().cpu().numpy(), attend(q, k, v, N_cap - 3, SCALE))
    assert st["max_abs"] <= ys.TOL["bf16"]["max_abs"] and st["mean_rel"] <= ys.TOL["bf16"]["mean_rel"], st


@pytest.mark.parametrize("Hq,Hkv,N_cap,tokens", [
    (1, 1, 2048, [5000, 3, 0]),       # the vector-ALU step, 16 splits in one launch
    (2, 1, 2200, [2200, 9000]),       # ... 18, with a merge launch
    (12, 4, 2048, [2048, 1]),         # the matrix-core step
    (4, 1, 2200, [100000, 700, 0]),
    (16, 16, 1500, [5000, 3, 0, 700, 1499, 1500, 1501, 900]),       # splits to spare, the vector-ALU step
    (24, 8, 3000, [2999, 3000, 3001, 1, 128, 1700, 375, 9000]),     # ... the matrix-core step
    (16, 1, 700, [699, 701]),         # more than 8 heads per KV head
    (33, 33, 512, [512, 5000, 3, 0, 511, 513, 256, 700]),           # 264 units: the eight that are over in splits
    (86, 43, 1024, [5000, 1024, 1023, 1, 2000, 0, 129, 1025]),      # ... 88 of 344 in two, two query heads each
    (99, 33, 640, [640, 639, 641, 0, 1, 384, 385, 6400]),           # ... the matrix-core step
])
def test_rings_that_are_split_store_the_new_row_and_attend_to_it(Hq, Hkv, N_cap, tokens):
    B, rng = len(tokens), np.random.default_rng(N_cap)
    rows = lambda n: torch.from_numpy(ys.normal(rng, (B, n, Hkv, D), 1.0, "bf16")).cuda().to(torch.bfloat16)  # noqa: E731
    K, V, kn, vn = rows(N_cap), rows(N_cap), rows(1), rows(1)
    fused, apart = (yoco.KVCache(B, Hkv, D, N_cap, torch.bfloat16) for _ in range(2))
    for c in (fused, apart):
        c.mem.zero_()
        for b in range(B):
            yoco.global_kv_write(c, K[b], V[b], b, 0)
    q = torch.from_numpy(ys.normal(rng, (B, Hq, D), 1.0, "bf16")).cuda().to(torch.bfloat16)
    ln = torch.tensor(tokens, dtype=torch.int64, device="cuda")
    ws = torch.full((yoco.cross_attn_decode_workspace(fused, Hq)[0],), 0xFF, dtype=torch.uint8, device="cuda")
    got = yoco.swa_decode(fused, q, ln, SCALE, ws, k_new=kn[:, 0], v_new=vn[:, 0])
    yoco.kv_cache_append(apart, kn[:, 0], vn[:, 0], ln - 1, True)
    ref = yoco.swa_decode(apart, q, ln, SCALE, ws)
    assert torch.equal(fused.mem, apart.mem)
    for b, n in enumerate(tokens):
        if n == 0:
            assert not got[b].any() and not ref[b].any()
            continue
        k, v = (p[b, :, :min(n, N_cap)].float().cpu().numpy().transpose(1, 0, 2) for p in apart.planes())
        want = oracle.cross_attn(q[b:b + 1].float().cpu().numpy(), k, v, k.shape[0] - 1, SCALE)[0]
        for o in (got, ref):
            st = ys.error_stats(o[b].float().cpu().numpy(), want)
            assert st["max_abs"] <= ys.TOL["bf16"]["max_abs"] and st["mean_rel"] <= ys.TOL["bf16"]["mean_rel"], (b, n, st)


@pytest.mark.parametrize("dtype,Hq,Hkv,N_cap", [
    ("bf16", 16, 16, 3000),           # 16 splits that meet in the launch
    ("bf16", 12, 4, 3000),            # 24, with a merge launch
    ("int8", 12, 4, 3000),            # 12 splits of a step of 256 rows
    ("int8", 16, 2, 2000),            # 8 heads: 8 splits
])
def test_lengths_of_one_sequence_around_the_steps_of_its_splits(dtype, Hq, Hkv, N_cap):
    rng = np.random.default_rng(N_cap + Hq)
    cache = yoco.KVCache(1, Hkv, D, N_cap, torch.int8 if dtype == "int8" else torch.bfloat16)
    cache.mem.zero_()
    K, V = (ys.normal(rng, (N_cap, Hkv, D), 1.0, "bf16") for _ in range(2))
    q = ys.normal(rng, (1, Hq, D), 1.0, "bf16")
    dev = lambda a: torch.from_numpy(a).cuda().to(torch.bfloat16)  # noqa: E731
    yoco.global_kv_write(cache, dev(K), dev(V), 0, 0)
    ws = torch.full((yoco.cross_attn_decode_workspace(cache, Hq)[0],), 0xFF, dtype=torch.uint8, device="cuda")
    attend = oracle.cross_attn_int8 if dtype == "int8" else oracle.cross_attn
    for n in (1, 127, 128, 129, 256, 257, 384, 385, 512, 513, 640, 641, 768, 769, 1025, 2000, N_cap):
        o = yoco.cross_attn_decode(cache, dev(q), torch.tensor([n], dtype=torch.int64, device="cuda"), SCALE, ws)
        st = ys.error_stats(o.float().cpu().numpy(), attend(q, K[:n], V[:n], n - 1, SCALE))
        assert st["max_abs"] <= ys.TOL["bf16"]["max_abs"] and st["mean_rel"] <= ys.TOL["bf16"]["mean_rel"], (n, st)


@pytest.mark.parametrize("splits", [17, 32, 33, 64, 65, 256])
def test_merge_launches_of_every_width(splits):
    N, Hq = 128 * splits - 5, 3
    cache = yoco.KVCache(1, 1, D, N, torch.bfloat16)
    rng = np.random.default_rng(splits)
    K, V = (ys.normal(rng, (N, 1, D), 1.0, "bf16") for _ in range(2))
    q = ys.normal(rng, (1, Hq, D), 1.0, "bf16")
    dev = lambda a: torch.from_numpy(a).cuda().to(torch.bfloat16)  # noqa: E731
    yoco.global_kv_write(cache, dev(K), dev(V), 0, 0)
    nbytes, n = yoco.cross_attn_decode_workspace(cache, Hq)
    assert n == splits
    ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
    for length in (N, N // 2, 1, 0):                                     # splits without rows among them, and nothing but those
        o = yoco.cross_attn_decode(cache, dev(q), torch.tensor([length], dtype=torch.int64, device="cuda"), SCALE, ws)
        got = o.float().cpu().numpy()
        if length == 0:
            assert not got.any()
            continue
        st = ys.error_stats(got, oracle.cross_attn(q, K[:length], V[:length], length - 1, SCALE))
        assert st["max_abs"] <= ys.TOL["bf16"]["max_abs"] and st["mean_rel"] <= ys.TOL["bf16"]["mean_rel"], (length, st)
