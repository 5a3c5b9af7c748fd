// C ABI of libyoco: argument validation and dispatch. No kernels here; the one device object is the static scratch
// array of yoco_cross_attn_decode_noalloc.
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <sys/random.h>

#include <atomic>
#include <chrono>
#include <mutex>

#include "yoco_common.h"

int yoco::compute_units() {
  static const int cus = [] {                     // initialised once, thread-safe
    int dev = 0, n = 0;
    const bool ok = hipGetDevice(&dev) == hipSuccess &&
                    hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0;
    (void)hipGetLastError();
    return ok ? n : 256;                          // no device visible (host-only sizing): MI355X has 256 CUs
  }();
  return cus;
}

namespace {

thread_local char g_err[256] = "";

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

int hip_result(hipError_t e, const char* what) {
  if (e == hipSuccess) return YOCO_OK;
  return fail(YOCO_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

bool aligned16(const void* p) { return (((uintptr_t)p) & 15u) == 0; }
size_t elem_bytes(int dtype) { return dtype == YOCO_F32 ? 4 : 2; }
bool dtype_ok(int dtype) { return dtype == YOCO_F32 || dtype == YOCO_BF16; }                 // tensors
bool cache_dtype_ok(int dtype) { return dtype_ok(dtype) || dtype == YOCO_INT8; }             // cache planes
int io_dtype(const yoco_kv_cache& c) { return c.dtype == YOCO_INT8 ? YOCO_BF16 : c.dtype; }  // of q and o on this cache
// Bytes of one sequence's share of a plane (all its KV heads).
size_t plane_bytes_per_seq(const yoco_kv_cache& c) {
  if (c.dtype == YOCO_INT8) return (size_t)c.Hkv * yoco::i8_plane_bytes(c.N_cap);
  return (size_t)c.Hkv * c.N_cap * c.d * elem_bytes(c.dtype);
}

int check_cache(const yoco_kv_cache* c) {
  if (!c) return fail(YOCO_ERR_INVALID_ARG, "cache descriptor is null");
  if (!c->k || !c->v) return fail(YOCO_ERR_INVALID_ARG, "cache planes are null");
  if (c->B <= 0 || c->Hkv <= 0 || c->N_cap <= 0) return fail(YOCO_ERR_INVALID_ARG, "cache has a non-positive size");
  if (!cache_dtype_ok(c->dtype)) return fail(YOCO_ERR_UNSUPPORTED, "cache dtype %d", c->dtype);
  if (c->d <= 0 || c->d > 256) return fail(YOCO_ERR_UNSUPPORTED, "head_dim %d not in [8, 256]", c->d);
  if (c->dtype == YOCO_INT8 && !yoco::cache_i8_supported(c->d))
    return fail(YOCO_ERR_UNSUPPORTED, "an 8-bit cache needs head_dim 128, not %d", c->d);
  if (c->d % 8) return fail(YOCO_ERR_ALIGNMENT, "head_dim %d is not a multiple of 8", c->d);
  if (!aligned16(c->k) || !aligned16(c->v)) return fail(YOCO_ERR_ALIGNMENT, "cache planes are not 16-byte aligned");
  return YOCO_OK;
}

int check_heads(int Hq, int Hkv) {
  if (Hq <= 0 || Hkv <= 0) return fail(YOCO_ERR_INVALID_ARG, "non-positive head count");
  if (Hq % Hkv) return fail(YOCO_ERR_INVALID_ARG, "Hq %d is not a multiple of Hkv %d", Hq, Hkv);
  if (Hq > 65535) return fail(YOCO_ERR_UNSUPPORTED, "Hq %d exceeds the grid limit", Hq);
  return YOCO_OK;
}

// Splits of the decode pass. Streaming reads on MI355X are fastest with few, long, contiguous streams: one workgroup per
// CU (measured: 6.9 TB/s at 256 workgroups, 6.0 TB/s at 2048; 8 KV heads x 16384 rows 17.7 us at 256, 19.6 at 512).
// `even`: the splits a sequence gets on average (a batch of equal lengths possibly fewer: inv_even). A split of a bf16
// cache has at least 128 rows, one step of its four wavefronts: a launch over few rows is latency, and a step more costs
// more than the workgroups saved (16 heads x 2016 rows: 13.4 us at 4 splits of 512 rows, 7.7 us at 16 of 128). Of an
// 8-bit cache it has at least 256, a step again, where that many meet in the launch (4 x 4 heads: 1500 rows 8.6 us at 3
// splits, 7.5 at 6; 4096 rows 9.2 at 8, 8.1 at 16) or a merge launch is there in any case (16:4 heads x 16000 rows 9.6 us at
// 32 splits, 8.2 at 63; 64:8 x 8000 9.7 at 16, 8.7 at 32; 16:1 x 700 9.7 at 2, 8.4 at 3) and has no more than 64 to read
// for a head (6:2 x 30000 9.5 at 59, 10.1 at 118; 16:1 x 20000 10.1 at 40, 10.8 at 79). Else it has 512: a merge launch for finer
// splits gains where the cache is full (24:8 x 8192 rows 9.3 us at 16, 8.0 at 32) and loses where it is not (300 rows of
// them 6.3 and 7.5).
// An fp32 cache has 512.
// `most`: what the workspace holds and the grid launches. Twice as many where a split of `even` has rows enough (2560)
// to be worth halving, so that the long sequences of a ragged batch can be split finer than the short ones (the kernel
// decides, from the lengths on the device; 5 x 2500..20000 rows x 8 heads: 45 us instead of 52, but 32 x 125..1000 rows
// 21 instead of 17). From four sequences on 700 rows are enough, up to three quarters as many units as CUs: there the long
// sequences are what a launch waits for (us, means over ten draws of lengths from an eighth of the capacity to all of it, without
// and with; bf16 21 x 8:64 heads x 4768 rows 50.2 and 41.3, 12 x 8:24 x 3000 19.4 and 18.0, 24 x 8:24 x 2000 24.8 and 24.0, 8 x 8:24 x
// 3000 14.1 and 13.95; 8 bits, which had none to spare, 11 x 16 x 16614 89.6 and 69.7, 9 x 8:24 x 3079 13.2 and 11.3). At
// three quarters a step of rows more can turn it: 24 x 8:64 x 1420 20.1 and 19.95, x 1600 21.6 and 22.5, x 1800 24.25 and 24.0; beyond,
// 232 units x 3141 35.8 and 36.1, 30 x 8 x 1000 16.8 and 18.8. From 500 to 700 rows it is one or the other (bf16 20 x 8:24 x 1200
// 16.1 and 14.65, 9 x 8:24 x 2400 13.65 and 13.0, but 8 x 16 x 1200 13.4 and 13.65, 4 x 8:24 x 4500 12.15 and 12.55; 8 bits 12 x 8:24 x
// 1800 10.8 and 10.7, 5 x 8:24 x 4000 10.5 and 10.8), and of two sequences 64:8 heads x 13668 take 15.1 and 16.4. Three or
// four times as many give no more. In 8 bits only up to half as many units as CUs, or from 3000 rows a split on, because the
// workgroups that a batch of equal lengths leaves without rows cost it (24 x 8 x 2000 17.8 and 18.7, x 4000 31.6 and 32.2, x 6000
// 46.5 and 46.85). Not where the splits are then too many to meet in the launch. The kernels of other head dimensions, and of more
// than 16 heads a KV head, share out the capacity and not the lengths; in bf16 the same rule is theirs, and theirs is the most to
// gain, with a wavefront a head and little in flight in each (8 x 8:24 heads of 64 x 3000 rows 84.7 and 52.8 at equal, 77.4 and
// 45.8 at ragged lengths, 5 x 8 of 64 x 8000 122 and 65.8, 12 x 4 of 256 x 6000 550 and 337).
// `least`: the same without that, which a workspace has to hold; one that holds no more gets no more. A pure function of the
// cache shape, the query heads and the device: the workspace query and the decode call agree.
struct Splits {
  int even, most, least;
  float inv_ragged, inv_even;   // 1 / how many workgroups a batch of ragged, of equal lengths should make
  int alike;                    // splits of each sequence of one length
  int split, parts;             // the first `split` pairs of sequence and KV head are split into `parts`, where no other is
  int places;                   // ragged: splits, over the batch, that have a CU of their own for each KV head; 0: not asked
};

// Rows from which on the units that are over are split into more than two parts: window caches, whose rows seldom differ, and others.
constexpr int64_t kRingPartRows = 512, kPartRows = 640;

Splits decode_splits(const yoco_kv_cache* c, int Hq) {
  const int cus = yoco::compute_units();
  const int64_t units = (int64_t)c->B * c->Hkv;
  auto clamp = [](int64_t s, int64_t hi) { return s > hi ? hi : s < 1 ? 1 : s; };
  const int64_t wanted = (cus + units - 1) / units;
  auto count = [&](int64_t rows) { return (int)clamp(clamp(wanted, (c->N_cap + rows - 1) / rows), 256); };
  auto meets = [&](int splits) { return yoco::decode_meets_in_launch(Hq / c->Hkv, splits); };
  const bool finer = c->dtype == YOCO_INT8 && (meets(count(256)) || (!meets(count(512)) && count(256) <= 64));
  const int min_rows = c->dtype == YOCO_BF16 ? 128 : finer ? 256 : 512;
  int64_t s = clamp(clamp(wanted, (c->N_cap + min_rows - 1) / min_rows), 256);
  // Splits of a bf16 cache have to save three steps of 128 rows to be worth the meeting at the end (240 units of 355 rows:
  // 10.1 us unsplit, 12.0 in two; 16 units of 400: 9.2 unsplit, 7.6 in four), of an 8-bit one two of 256 (32 units of 500
  // rows: 6.9 unsplit, 7.5 in two; of 700 8.3 and 7.4 in three).
  const int64_t saves = c->dtype == YOCO_BF16 ? 3 : 2;
  if ((c->dtype == YOCO_BF16 || finer) && (c->N_cap + min_rows - 1) / min_rows - (c->N_cap + min_rows * s - 1) / (min_rows * s) < saves) s = 1;
  // More (sequence, KV head) units than CUs, and not a multiple of them: the workgroups of a ragged last round run
  // with part of the chip idle (384 units on 256 CUs measured 5.7 TB/s at 4096 rows). Two to four splits per unit
  // make the count a multiple again, as long as a split keeps at least 1024 rows (384 units of 1024 rows: 35.9 us
  // unsplit, 36.7 at two).
  // Else, up to twice as many units as CUs, only the units that are over are split, into as many parts as give every CU one whole
  // unit and at most one part, up to eight of 128 rows or more (us a layer, unsplit and so: window caches 12 x 24 heads x 1024 rows
  // 33.2 and 27.2, 16 x 24 36.0 and 34.0, 12 x 24 x 512, ragged, 17.8 and 15.3; bf16 33 x 8:24 x 2000 65.5 and 44.7, 40 x 8:24 x 3000, ragged,
  // 83.8 and 60.1; 8 bits 33 x 8:24 x 1024 20.7 and 16.2, 48 x 8 x 1024 22.2 and 20.8). Two parts of fewer than 512 rows lose (24 x 16 x 512
  // 19.5 and 20.8), and so do 8 bits below 1024 rows (40 x 8 x 512 12.2 and 12.8) and more units (80 x 8 x 1024, 8 bits, 63 and 71). Of a
  // ragged batch the kernel looks at the lengths first (split_rows); caches below 640 rows have too little to gain for that.
  int64_t split = 0, parts = 1;
  if (s == 1 && units > cus && units % cus != 0) {
    for (int64_t t = 2; t <= 4; ++t)
      if ((units * t) % cus == 0 && c->N_cap / t >= 1024) { s = t; break; }
    if (s == 1 && units < 2 * cus && (c->dtype == YOCO_BF16 || c->dtype == YOCO_INT8) && c->d == 128 && Hq / c->Hkv <= 16) {
      parts = clamp(clamp(cus / (units % cus), 8), c->N_cap / 128);
      while (parts > 1 && !meets((int)parts)) --parts;
      if (parts > 1 && c->N_cap >= (c->dtype == YOCO_BF16 && parts > 2 ? kRingPartRows : 1024)) split = units % cus;
    }
  }
  // What fitted the static scratch with splits of 512 rows still does.
  const int64_t coarse = clamp(clamp(wanted, (c->N_cap + 511) / 512), 256);
  const int64_t fits = (int64_t)(YOCO_NOALLOC_SCRATCH_BYTES / ((size_t)c->B * Hq * yoco::partial_stride(c->d) * sizeof(float)));
  auto bounded = [&](int64_t x) { return x > fits ? (fits > coarse ? fits : coarse) : x; };
  if (s > coarse) s = bounded(s);
  int64_t most = s, least = s;
  if ((c->dtype == YOCO_BF16 || finer) && units <= cus && s > 1 && s <= 128) {
    const int64_t twice = bounded(2 * s) > s ? bounded(2 * s) : s;
    if (c->dtype == YOCO_BF16 && c->N_cap / s >= 2560) most = least = twice;
    const bool few = 4 * units <= 3 * cus && (c->dtype == YOCO_BF16 || 2 * units <= cus || c->N_cap / s >= 3000);
    if (most == s && c->N_cap / s >= 700 && c->B >= yoco::kManySequences && few && meets((int)twice) == meets((int)s)) most = twice;
  }
  // Equal lengths: no more workgroups than CUs where the count is no multiple, because a workgroup or two too many share
  // a CU and the launch waits for them (24 units x 32768 rows: 264 workgroups 47.6 us in 8 bits and 87.4 in bf16, 240 36.2
  // and 64.1; 200 units x 8192: 400 workgroups 74.7 and 144, 200 63.6 and 136; rolling caches, 160 units x 2048: 36.9
  // -> 31.1). Where that leaves a quarter of the CUs without one, two rounds' worth is better for a bf16 cache (160 units x
  // 16384: 160 workgroups 258 us, 320 268, 480 203; in 8 bits 107, 130, 108), if it makes at least one and a half (200 x 2
  // does not) of splits of 1024 rows or more. Ragged lengths keep the larger count, of which short sequences take less
  // (200 units of 1000 to 8192 rows: 88 us, at 200 workgroups 137), unless the kernel finds shares that fit (split_rows).
  int64_t n = s;
  if (units < cus && units * s > cus) {
    n = cus / units;
    const int64_t twice = 2 * cus / units;
    if (c->dtype == YOCO_BF16 && 4 * units * n < 3 * cus && 2 * units * twice >= 3 * cus && twice <= least && c->N_cap / twice >= 1024) n = twice;
  }
  return {(int)s, (int)most, (int)least, 1.f / (float)(units * s), 1.f / (float)(units * n), (int)n, (int)split, (int)parts, units <= cus ? cus / c->Hkv : 0};
}

size_t partial_bytes(const yoco_kv_cache& c, int Hq, int splits) {
  return (size_t)c.B * Hq * splits * yoco::partial_stride(c.d) * sizeof(float);
}
// The splits of a decode call with `held` bytes of workspace.
int plan_decode(const yoco_kv_cache& c, int Hq, size_t held, Splits* plan, bool ring) {
  *plan = decode_splits(&c, Hq);
  if (held < partial_bytes(c, Hq, plan->most)) plan->most = plan->least;
  if (!ring && c.N_cap < kPartRows) plan->split = 0;
  const size_t need = partial_bytes(c, Hq, plan->most);
  return held < need ? fail(YOCO_ERR_WORKSPACE, "workspace %zu < %zu bytes", held, need) : YOCO_OK;
}

// The tag a decode launch marks its published splits with: never 0, never the same twice in a process (a bijection of a
// counter), and nothing that other data is likely to look like.
unsigned long long next_tag() {
  static std::atomic<uint64_t> n{[] {                // nothing here throws: callers are C
    uint64_t start = 0;
    if (getrandom(&start, sizeof(start), GRND_NONBLOCK) != (ssize_t)sizeof(start)) start = (uint64_t)(uintptr_t)&start;
    return start ^ (uint64_t)std::chrono::steady_clock::now().time_since_epoch().count();
  }()};
  uint64_t z;
  do {
    z = n.fetch_add(1, std::memory_order_relaxed) * 0x9E3779B97F4A7C15ull;
    z ^= z >> 29;
  } while (z == 0);
  return z;
}

// Split-KV attention of one query token per sequence of `c`: one launch, or one for the splits and one for their merge.
// `lens` (device) or, when it is null, `fixed_len` (host) gives the visible rows.
// k_new / v_new (both null or both rows [B,Hkv,d] of the cache dtype): the new token's row is stored at slot
// lens[b] - 1 (ring: modulo the capacity) by the same call and attended to.
int run_decode(const yoco_kv_cache& c, const void* q, void* o, const int64_t* lens, int64_t fixed_len, int Hq, float scale,
               float* ws, Splits sp, hipStream_t s, const char* what, const void* k_new = nullptr, const void* v_new = nullptr,
               int ring = 0, const yoco::ReadAhead& ahead = {}) {
  hipError_t e;
  if (!lens) sp.split = 0;                           // the kernel decides by the lengths
  if (sp.split) sp.most = sp.parts;                  // where every pair has room for one split: no more than CUs, which are fewer
  const unsigned long long tag = yoco::decode_meets_in_launch(Hq / c.Hkv, sp.most) ? next_tag() : 0;
  if (c.dtype == YOCO_INT8) {
    if (!yoco::decode_i8_supported(c, Hq))
      return fail(YOCO_ERR_UNSUPPORTED, "%s: an 8-bit cache serves up to 16 query heads per KV head, not %d", what, Hq / c.Hkv);
    if (k_new) return fail(YOCO_ERR_UNSUPPORTED, "%s: no fused append into an 8-bit cache", what);
    e = yoco::launch_decode_i8(c, q, lens, fixed_len, Hq, scale, ws, sp.most, sp.inv_ragged, sp.inv_even, sp.alike, sp.split, sp.places, tag, o, ahead, s);
    if (tag) return hip_result(e, what);
  } else if (yoco::decode_bf16_supported(c, Hq)) {
    e = yoco::launch_decode_bf16(c, q, lens, fixed_len, Hq, scale, ws, sp.most, sp.inv_ragged, sp.inv_even, sp.alike, sp.split, sp.places, tag, o, k_new, v_new, ring, ahead, s);
    if (tag) return hip_result(e, what);
  } else {
    if (k_new) {                                      // no fused path for this shape: append, then attend
      e = yoco::launch_kv_append(c, k_new, v_new, lens, lens ? -1 : fixed_len - 1, ring, c.dtype, s);
      if (e != hipSuccess) return hip_result(e, what);
    }
    e = yoco::launch_decode_generic(c, q, lens, fixed_len, Hq, scale, ws, sp.most, s);
  }
  if (e != hipSuccess) return hip_result(e, what);
  return hip_result(yoco::launch_decode_merge(ws, o, c.B, Hq, c.d, sp.most, io_dtype(c), s), what);
}

int check_gret_shape(int B, int64_t T, int H, int dk, int dv, int dtype) {
  if (B <= 0 || H <= 0 || T < 0) return fail(YOCO_ERR_INVALID_ARG, "non-positive B or H, or negative T");
  if (B > 65535 || H > 65535) return fail(YOCO_ERR_UNSUPPORTED, "B %d or H %d exceeds the grid limit", B, H);
  if (!dtype_ok(dtype)) return fail(YOCO_ERR_UNSUPPORTED, "dtype %d", dtype);
  if (dk <= 0 || dv <= 0 || dk > 256 || dv > 256) return fail(YOCO_ERR_UNSUPPORTED, "head dims %d, %d not in [8, 256]", dk, dv);
  if (dk % 8 || dv % 8) return fail(YOCO_ERR_ALIGNMENT, "head dims %d, %d are not multiples of 8", dk, dv);
  return YOCO_OK;
}

// ---- one token through a whole stack
typedef unsigned short bf16_raw;

int check_stack(const yoco_stack* st) {
  if (st->n_self < 0 || st->n_cross <= 0 || (st->n_self && !st->self) || !st->cross || !st->final_ln || !st->w_out || (st->n_self && (!st->kv_ln || !st->w_kv)))
    return fail(YOCO_ERR_INVALID_ARG, "stack: missing layers or weights");
  if (st->d_model <= 0 || st->ffn <= 0 || st->vocab <= 0 || !(st->tau > 0.f)) return fail(YOCO_ERR_INVALID_ARG, "stack: non-positive size");
  int rc = check_heads(st->Hq, st->Hkv);
  if (rc) return rc;
  if (st->n_self && !st->gret && (rc = check_heads(st->Hq, st->Hkv_self))) return rc;
  if (st->n_self && st->gret && st->Hkv_self != st->Hq) return fail(YOCO_ERR_UNSUPPORTED, "stack: gated retention has no grouped heads");
  if (st->d != 128) return fail(YOCO_ERR_UNSUPPORTED, "stack: head_dim %d, not 128", st->d);
  if (st->d_model % 8 || st->ffn % 8) return fail(YOCO_ERR_ALIGNMENT, "stack: widths must be multiples of 8");
  if (st->d_model > yoco::kGemvMaxK || st->ffn > yoco::kGemvMaxK || (int64_t)st->Hq * st->d > yoco::kGemvMaxK)
    return fail(YOCO_ERR_UNSUPPORTED, "stack: a width exceeds %d", yoco::kGemvMaxK);
  for (int i = 0; i < st->n_self + st->n_cross; ++i) {
    const yoco_stack_layer& L = i < st->n_self ? st->self[i] : st->cross[i - st->n_self];
    if (!L.ln1 || !L.w_in || !L.w_o || !L.ln2 || !L.w_gu || !L.w_2) return fail(YOCO_ERR_INVALID_ARG, "stack: layer %d has a null pointer", i);
    if (!aligned16(L.ln1) || !aligned16(L.w_in) || !aligned16(L.w_o) || !aligned16(L.ln2) || !aligned16(L.w_gu) || !aligned16(L.w_2))
      return fail(YOCO_ERR_ALIGNMENT, "stack: layer %d has a pointer that is not 16-byte aligned", i);
  }
  if (!aligned16(st->kv_ln) || !aligned16(st->w_kv) || !aligned16(st->final_ln) || !aligned16(st->w_out))
    return fail(YOCO_ERR_ALIGNMENT, "stack: pointer not 16-byte aligned");
  return YOCO_OK;
}

// The activations of one token, carved out of the caller's scratch.
struct StackScratch {
  bf16_raw *x, *y, *in, *o, *h;
  float* log_gamma;
  size_t bytes;
  StackScratch(const yoco_stack& st, char* p) {
    char* const p0 = p;
    auto take = [&](size_t n) { char* r = p; p += (n + 255) & ~(size_t)255; return r; };
    const size_t qd = (size_t)st.Hq * st.d, kd = (size_t)(st.Hkv_self > st.Hkv ? st.Hkv_self : st.Hkv) * st.d;
    x = (bf16_raw*)take(2 * (size_t)st.d_model);
    y = (bf16_raw*)take(2 * (size_t)st.d_model);
    in = (bf16_raw*)take(2 * (2 * qd + 2 * kd));
    o = (bf16_raw*)take(2 * qd);
    h = (bf16_raw*)take(2 * (size_t)st.ffn);
    log_gamma = (float*)take(4 * (size_t)st.Hq);
    bytes = (size_t)(p - p0);
  }
};

// The weights that the launches behind a layer's attention stream, as far as kAheadBytes go: W_O, then the SwiGLU pair (four rows of
// either half for a workgroup of launch_gemv). A token step of 4 + 4 layers of 2048 over 1900 rows 273.0 us, 268.0 with it, over
// 200 rows 265.2 and 259.5, of 1024-wide layers over 500 rows 169.3 and 165.3; with 8, 24 or 32 MB 270, 270 and 277. Only for
// attention over a short cache: a longer one pushes the weights out of the L2s (32 MB in all) again, and its launch has less
// bandwidth to spare. The line lies behind where the two sides cross, the cross-decoder's launches not reading ahead and reading,
// of 16 heads: 2200 rows (18 MB) 274.5 and 272.0, 2600 (21 MB) 274.7 and 274.7, 3000 (24.6 MB) 275.1 and 277.0, 3500 277.1 and
// 280.7; of 8-bit rows 5500 (23.2 MB) 284.7 and 282.9.
constexpr int64_t kAheadBytes = 16 << 20, kShortCache = 23 << 20;
yoco::ReadAhead weights_ahead(const yoco_stack& st, const yoco_stack_layer& L, const yoco_kv_cache& c, int64_t rows) {
  yoco::ReadAhead a = {};
  if (rows > c.N_cap) rows = c.N_cap;
  if (rows * c.Hkv * (c.dtype == YOCO_INT8 ? 264 : 512) > kShortCache) return a;
  int64_t left = kAheadBytes;
  auto part = [&](int m, const void* w, int64_t rows, int64_t width, int halves) {
    const int64_t bytes = 4 * width * 2;
    int64_t pieces = left / (bytes * halves);
    if (pieces > rows / 4) pieces = rows / 4;
    a.part[m] = {w, rows * width * 2, (int)bytes, (int)pieces, halves};
    left -= pieces * bytes * halves;
  };
  part(0, L.w_o, st.d_model, (int64_t)st.Hq * st.d, 1);
  part(1, L.w_gu, st.ffn, st.d_model, 2);
  a.workgroups = yoco::compute_units();
  return a;
}

// ---- static scratch for callers that cannot allocate (yoco_cross_attn_decode_noalloc). Every GPU the library
// runs on holds its own copy of the array, at its own address, until the process ends. In host code the array's name is
// only a handle for hipGetSymbolAddress; kernels and copies get the per-device address looked up below.
constexpr size_t kScratchBytes = YOCO_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mutex;

// Device address of `scratch` on the current device, looked up once per device with that device current.
int scratch_of_current_device(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_result(e, "hipGetDevice");
  if (dev < 0 || dev >= kMaxDevices) return fail(YOCO_ERR_UNSUPPORTED, "device index %d outside [0, %d)", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_result(e, "hipGetSymbolAddress(scratch)");
    if (!p) return fail(YOCO_ERR_HIP, "hipGetSymbolAddress(scratch) returned a null address");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return YOCO_OK;
}

constexpr int64_t kFewRows = 8;   // query rows up to which the prefill call splits over the cache like decode

// Tq query rows over one sequence of a cache, without the tensors.
yoco::AttnView cross_view(const yoco_kv_cache& c, int64_t q_pos0, int64_t Tq, int Hq, float scale) {
  yoco::AttnView a = {};
  a.q_stride_t = (int64_t)Hq * c.d;
  a.kv_stride_n = c.d;
  a.kv_stride_h = c.N_cap * c.d;
  a.Tq = Tq; a.q_pos0 = q_pos0;
  a.window = q_pos0 + Tq;          // every earlier row is visible
  a.Hq = Hq; a.Hkv = c.Hkv; a.d = c.d; a.B = 1; a.scale = scale;
  return a;
}

}  // namespace

#pragma GCC visibility push(default)
extern "C" {

int yoco_version(void) { return 100; }

const char* yoco_last_error_string(void) { return g_err; }

int yoco_kv_cache_bytes(int B, int Hkv, int d, int64_t N_cap, int dtype, size_t* bytes) {
  if (!bytes) return fail(YOCO_ERR_INVALID_ARG, "bytes is null");
  if (B <= 0 || Hkv <= 0 || d <= 0 || N_cap <= 0) return fail(YOCO_ERR_INVALID_ARG, "non-positive size");
  if (!cache_dtype_ok(dtype)) return fail(YOCO_ERR_UNSUPPORTED, "dtype %d", dtype);
  if (d % 8) return fail(YOCO_ERR_ALIGNMENT, "head_dim %d is not a multiple of 8", d);
  if (d > 256) return fail(YOCO_ERR_UNSUPPORTED, "head_dim %d exceeds 256", d);
  if (dtype == YOCO_INT8) {
    if (!yoco::cache_i8_supported(d)) return fail(YOCO_ERR_UNSUPPORTED, "an 8-bit cache needs head_dim 128, not %d", d);
    *bytes = (size_t)2 * B * Hkv * (size_t)yoco::i8_plane_bytes(N_cap);
    return YOCO_OK;
  }
  *bytes = (size_t)2 * B * Hkv * (size_t)N_cap * d * elem_bytes(dtype);
  return YOCO_OK;
}

int yoco_kv_cache_init(void* mem, size_t bytes, int B, int Hkv, int d, int64_t N_cap, int dtype, yoco_kv_cache* out) {
  if (!out) return fail(YOCO_ERR_INVALID_ARG, "out is null");
  if (!mem) return fail(YOCO_ERR_INVALID_ARG, "mem is null");
  size_t need = 0;
  int rc = yoco_kv_cache_bytes(B, Hkv, d, N_cap, dtype, &need);
  if (rc) return rc;
  if (bytes < need) return fail(YOCO_ERR_WORKSPACE, "cache memory %zu < %zu bytes", bytes, need);
  if (((uintptr_t)mem) & 255u) return fail(YOCO_ERR_ALIGNMENT, "cache memory is not 256-byte aligned");
  out->k = mem;
  out->v = (char*)mem + need / 2;
  out->B = B;
  out->Hkv = Hkv;
  out->d = d;
  out->dtype = dtype;
  out->N_cap = N_cap;
  return YOCO_OK;
}

int yoco_swa_prefill(const void* q, const void* k, const void* v, void* o, int B, int64_t T, int Hq, int Hkv, int d,
                     int64_t window, float scale, int dtype, void* stream) {
  if (!q || !k || !v || !o) return fail(YOCO_ERR_INVALID_ARG, "null tensor pointer");
  if (B <= 0 || T <= 0 || window <= 0) return fail(YOCO_ERR_INVALID_ARG, "non-positive B, T or window");
  if (B > 65535) return fail(YOCO_ERR_UNSUPPORTED, "B %d exceeds the grid limit", B);
  int rc = check_heads(Hq, Hkv);
  if (rc) return rc;
  if (!dtype_ok(dtype)) return fail(YOCO_ERR_UNSUPPORTED, "dtype %d", dtype);
  if (d <= 0 || d > 256) return fail(YOCO_ERR_UNSUPPORTED, "head_dim %d not in [8, 256]", d);
  if (d % 8) return fail(YOCO_ERR_ALIGNMENT, "head_dim %d is not a multiple of 8", d);
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o))
    return fail(YOCO_ERR_ALIGNMENT, "tensor pointer not 16-byte aligned");
  yoco::AttnView a;
  a.q = q; a.k = k; a.v = v; a.o = o;
  a.q_stride_t = (int64_t)Hq * d;
  a.q_stride_b = T * a.q_stride_t;
  a.kv_stride_n = (int64_t)Hkv * d;
  a.kv_stride_h = d;
  a.kv_stride_b = T * a.kv_stride_n;
  a.Tq = T; a.q_pos0 = 0;
  a.window = window > T ? T : window;
  a.Hq = Hq; a.Hkv = Hkv; a.d = d; a.B = B; a.scale = scale;
  if (yoco::swa_mfma_supported(a, dtype)) return hip_result(yoco::launch_swa_mfma(a, nullptr, 0, (hipStream_t)stream), "swa_prefill");
  if (yoco::attn_f32_supported(a)) return hip_result(yoco::launch_attn_f32(a, dtype, (hipStream_t)stream), "swa_prefill");
  return hip_result(yoco::launch_attn_generic(a, dtype, (hipStream_t)stream), "swa_prefill");
}

int yoco_global_kv_write_scaled(const yoco_kv_cache* c, const void* k, const void* v, const float* row_scale, int b, int64_t pos0,
                                int64_t n, int src_dtype, void* stream) {
  int rc = check_cache(c);
  if (rc) return rc;
  if (n < 0) return fail(YOCO_ERR_INVALID_ARG, "negative row count");
  if (b < 0 || b >= c->B) return fail(YOCO_ERR_INVALID_ARG, "sequence %d outside [0, %d)", b, c->B);
  if (pos0 < 0 || pos0 + n > c->N_cap)
    return fail(YOCO_ERR_INVALID_ARG, "rows [%lld, %lld) outside the cache capacity %lld", (long long)pos0,
                (long long)(pos0 + n), (long long)c->N_cap);
  if (!dtype_ok(src_dtype)) return fail(YOCO_ERR_UNSUPPORTED, "source dtype %d", src_dtype);
  if (n == 0) return YOCO_OK;
  if (!k || !v) return fail(YOCO_ERR_INVALID_ARG, "null row pointer");
  if (!aligned16(k) || !aligned16(v)) return fail(YOCO_ERR_ALIGNMENT, "row pointer not 16-byte aligned");
  if (row_scale && (((uintptr_t)row_scale) & 3u)) return fail(YOCO_ERR_ALIGNMENT, "row_scale is not 4-byte aligned");
  if (c->dtype == YOCO_INT8) {
    if (n * c->Hkv > (int64_t)1 << 32) return fail(YOCO_ERR_UNSUPPORTED, "too many rows for one call");
    if (c->Hkv > 65535) return fail(YOCO_ERR_UNSUPPORTED, "Hkv %d exceeds the grid limit", c->Hkv);
    return hip_result(yoco::launch_kv_code_i8(*c, k, v, row_scale, b, pos0, n, nullptr, src_dtype, (hipStream_t)stream), "global_kv_write");
  }
  return hip_result(yoco::launch_kv_write(*c, k, v, row_scale, b, pos0, 0, n, src_dtype, (hipStream_t)stream), "global_kv_write");
}

int yoco_global_kv_write(const yoco_kv_cache* c, const void* k, const void* v, int b, int64_t pos0, int64_t n,
                         int src_dtype, void* stream) {
  return yoco_global_kv_write_scaled(c, k, v, nullptr, b, pos0, n, src_dtype, stream);
}

int yoco_swa_cache_write(const yoco_kv_cache* ring, const void* k, const void* v, int b, int64_t pos0, int64_t n,
                         int src_dtype, void* stream) {
  int rc = check_cache(ring);
  if (rc) return rc;
  if (ring->dtype == YOCO_INT8) return fail(YOCO_ERR_UNSUPPORTED, "a rolling window cache cannot be 8-bit");
  if (n < 0) return fail(YOCO_ERR_INVALID_ARG, "negative row count");
  if (b < 0 || b >= ring->B) return fail(YOCO_ERR_INVALID_ARG, "sequence %d outside [0, %d)", b, ring->B);
  if (pos0 < 0) return fail(YOCO_ERR_INVALID_ARG, "negative position %lld", (long long)pos0);
  if (pos0 > INT64_MAX - n) return fail(YOCO_ERR_INVALID_ARG, "positions overflow");
  if (!dtype_ok(src_dtype)) return fail(YOCO_ERR_UNSUPPORTED, "source dtype %d", src_dtype);
  if (n == 0) return YOCO_OK;
  if (!k || !v) return fail(YOCO_ERR_INVALID_ARG, "null row pointer");
  if (!aligned16(k) || !aligned16(v)) return fail(YOCO_ERR_ALIGNMENT, "row pointer not 16-byte aligned");
  const int64_t r0 = n > ring->N_cap ? n - ring->N_cap : 0;     // earlier rows would be overwritten by later ones
  return hip_result(yoco::launch_kv_write(*ring, k, v, nullptr, b, pos0, r0, n, src_dtype, (hipStream_t)stream), "swa_cache_write");
}

int yoco_kv_cache_append(const yoco_kv_cache* c, const void* k, const void* v, const int64_t* pos, int ring,
                         int src_dtype, void* stream) {
  int rc = check_cache(c);
  if (rc) return rc;
  if (!dtype_ok(src_dtype)) return fail(YOCO_ERR_UNSUPPORTED, "source dtype %d", src_dtype);
  if (!k || !v || !pos) return fail(YOCO_ERR_INVALID_ARG, "null pointer");
  if (!aligned16(k) || !aligned16(v)) return fail(YOCO_ERR_ALIGNMENT, "row pointer not 16-byte aligned");
  if (((uintptr_t)pos) & 7u) return fail(YOCO_ERR_ALIGNMENT, "pos is not 8-byte aligned");
  if (c->dtype == YOCO_INT8) {
    if (ring) return fail(YOCO_ERR_UNSUPPORTED, "a rolling window cache cannot be 8-bit");
    return hip_result(yoco::launch_kv_code_i8(*c, k, v, nullptr, 0, 0, c->B, pos, src_dtype, (hipStream_t)stream), "kv_cache_append");
  }
  return hip_result(yoco::launch_kv_append(*c, k, v, pos, 0, ring, src_dtype, (hipStream_t)stream), "kv_cache_append");
}

int yoco_cross_attn_prefill(const yoco_kv_cache* c, const void* q, void* o, int b, int64_t q_pos0, int64_t Tq, int Hq,
                            float scale, void* workspace, size_t workspace_bytes, void* stream) {
  int rc = check_cache(c);
  if (rc) return rc;
  rc = check_heads(Hq, c->Hkv);
  if (rc) return rc;
  if (!q || !o) return fail(YOCO_ERR_INVALID_ARG, "null tensor pointer");
  if (!aligned16(q) || !aligned16(o)) return fail(YOCO_ERR_ALIGNMENT, "tensor pointer not 16-byte aligned");
  if (b < 0 || b >= c->B) return fail(YOCO_ERR_INVALID_ARG, "sequence %d outside [0, %d)", b, c->B);
  if (Tq <= 0 || q_pos0 < 0) return fail(YOCO_ERR_INVALID_ARG, "non-positive Tq or negative q_pos0");
  if (q_pos0 + Tq > c->N_cap)
    return fail(YOCO_ERR_INVALID_ARG, "query positions up to %lld exceed the cache capacity %lld",
                (long long)(q_pos0 + Tq), (long long)c->N_cap);
  const size_t eb = elem_bytes(io_dtype(*c));
  const size_t seq_bytes = plane_bytes_per_seq(*c);
  if (workspace && !aligned16(workspace)) return fail(YOCO_ERR_ALIGNMENT, "workspace not 16-byte aligned");
  if (workspace && Tq <= kFewRows) {
    // A few rows cannot fill the chip one workgroup per query tile: treat each
    // row as a decode step of a one-sequence cache, split over the rows it sees.
    yoco_kv_cache one = *c;
    one.B = 1;
    one.k = (char*)c->k + (size_t)b * seq_bytes;
    one.v = (char*)c->v + (size_t)b * seq_bytes;
    const size_t per_split = (size_t)Hq * yoco::partial_stride(c->d) * sizeof(float);
    Splits splits = decode_splits(&one, Hq);
    splits.most = splits.even;                                          // one sequence: nothing is ragged
    const size_t whole = (size_t)c->B * decode_splits(c, Hq).least;     // what the documented workspace holds
    const size_t held = workspace_bytes / per_split;
    if (held >= (whole < (size_t)splits.even ? whole : (size_t)splits.even)) {
      if (held < (size_t)splits.most) splits.most = (int)held;
      for (int64_t i = 0; i < Tq; ++i) {
        rc = run_decode(one, (const char*)q + (size_t)i * Hq * c->d * eb, (char*)o + (size_t)i * Hq * c->d * eb, nullptr,
                        q_pos0 + i + 1, Hq, scale, (float*)workspace, splits, (hipStream_t)stream, "cross_attn_prefill (split)");
        if (rc) return rc;
      }
      return YOCO_OK;
    }
  }
  if (c->dtype == YOCO_INT8)
    return fail(YOCO_ERR_UNSUPPORTED, "cross_attn_prefill over an 8-bit cache serves up to %d rows and needs the decode workspace",
                (int)kFewRows);
  yoco::AttnView a = cross_view(*c, q_pos0, Tq, Hq, scale);
  a.q = q; a.o = o;
  a.k = (const char*)c->k + (size_t)b * seq_bytes;
  a.v = (const char*)c->v + (size_t)b * seq_bytes;
  if (yoco::swa_mfma_supported(a, c->dtype))
    return hip_result(yoco::launch_swa_mfma(a, Tq > kFewRows ? workspace : nullptr, workspace_bytes, (hipStream_t)stream), "cross_attn_prefill");
  if (yoco::attn_f32_supported(a)) return hip_result(yoco::launch_attn_f32(a, c->dtype, (hipStream_t)stream), "cross_attn_prefill");
  return hip_result(yoco::launch_attn_generic(a, c->dtype, (hipStream_t)stream), "cross_attn_prefill");
}

int yoco_cross_attn_prefill_workspace(const yoco_kv_cache* c, int64_t q_pos0, int64_t Tq, int Hq, float scale, size_t* bytes) {
  if (!c || !bytes) return fail(YOCO_ERR_INVALID_ARG, "null argument");
  if (c->B <= 0 || c->Hkv <= 0 || c->N_cap <= 0 || c->d <= 0) return fail(YOCO_ERR_INVALID_ARG, "cache has a non-positive size");
  int rc = check_heads(Hq, c->Hkv);
  if (rc) return rc;
  if (Tq <= 0 || q_pos0 < 0 || Tq > c->N_cap || q_pos0 > c->N_cap - Tq)
    return fail(YOCO_ERR_INVALID_ARG, "query positions outside the cache capacity %lld", (long long)c->N_cap);
  const yoco::AttnView a = cross_view(*c, q_pos0, Tq, Hq, scale);
  *bytes = Tq > kFewRows && yoco::swa_mfma_supported(a, c->dtype) ? yoco::swa_mfma_workspace(a) : 0;
  return YOCO_OK;
}

int yoco_cross_attn_decode_workspace(const yoco_kv_cache* c, int Hq, size_t* bytes, int* splits) {
  if (!c || !bytes || !splits) return fail(YOCO_ERR_INVALID_ARG, "null argument");
  if (c->B <= 0 || c->Hkv <= 0 || c->N_cap <= 0 || c->d <= 0) return fail(YOCO_ERR_INVALID_ARG, "cache has a non-positive size");
  int rc = check_heads(Hq, c->Hkv);
  if (rc) return rc;
  const int s = decode_splits(c, Hq).most;
  *splits = s;
  *bytes = partial_bytes(*c, Hq, s);
  return YOCO_OK;
}

int yoco_cross_attn_decode(const yoco_kv_cache* c, const void* q, void* o, const int64_t* lens, int Hq, float scale,
                           void* workspace, size_t workspace_bytes, void* stream) {
  int rc = check_cache(c);
  if (rc) return rc;
  rc = check_heads(Hq, c->Hkv);
  if (rc) return rc;
  if (!q || !o || !lens || !workspace) return fail(YOCO_ERR_INVALID_ARG, "null pointer");
  if (!aligned16(q) || !aligned16(o) || !aligned16(workspace))
    return fail(YOCO_ERR_ALIGNMENT, "pointer not 16-byte aligned");
  if (c->B > 65535) return fail(YOCO_ERR_UNSUPPORTED, "B %d exceeds the grid limit", c->B);
  Splits plan;
  rc = plan_decode(*c, Hq, workspace_bytes, &plan, false);
  if (rc) return rc;
  return run_decode(*c, q, o, lens, 0, Hq, scale, (float*)workspace, plan, (hipStream_t)stream, "cross_attn_decode");
}

int yoco_cross_attn_decode_noalloc(const yoco_kv_cache* c, const void* q, void* o, const int64_t* lens, int Hq, float scale,
                                   void* stream) {
  // Validate the shape and the size first: a call that is too large must fail before anything touches the device.
  int rc = check_cache(c);
  if (rc) return rc;
  if (!q || !o || !lens) return fail(YOCO_ERR_INVALID_ARG, "null pointer");
  rc = check_heads(Hq, c->Hkv);
  if (rc) return rc;
  const size_t need = partial_bytes(*c, Hq, decode_splits(c, Hq).least);
  if (need > kScratchBytes)
    return fail(YOCO_ERR_WORKSPACE, "cross_attn_decode_noalloc: the partial results need %zu bytes, the static scratch holds %zu",
                need, kScratchBytes);
  void* ptr = nullptr;
  rc = scratch_of_current_device(&ptr);
  if (rc) return rc;
  // A merge reads only what the same call has put there (splits published under its tag, or every partial of the generic
  // kernels' first launch), so nothing in the array has to be cleared between calls.
  return yoco_cross_attn_decode(c, q, o, lens, Hq, scale, ptr, kScratchBytes, stream);
}

int yoco_swa_decode(const yoco_kv_cache* ring, const void* q, const void* k_new, const void* v_new, void* o,
                    const int64_t* lens, int Hq, float scale, void* workspace, size_t workspace_bytes, void* stream) {
  // The ring holds exactly the rows the window admits and a softmax-weighted
  // sum does not depend on the order of its terms, so a decode step over the
  // ring, with lens clamped to its capacity (the kernels do), is Eq. 8.
  int rc = check_cache(ring);
  if (rc) return rc;
  if (ring->dtype == YOCO_INT8) return fail(YOCO_ERR_UNSUPPORTED, "a rolling window cache cannot be 8-bit");
  rc = check_heads(Hq, ring->Hkv);
  if (rc) return rc;
  if (!q || !o || !lens || !workspace) return fail(YOCO_ERR_INVALID_ARG, "null pointer");
  if (!aligned16(q) || !aligned16(o) || !aligned16(workspace))
    return fail(YOCO_ERR_ALIGNMENT, "pointer not 16-byte aligned");
  if (ring->B > 65535) return fail(YOCO_ERR_UNSUPPORTED, "B %d exceeds the grid limit", ring->B);
  if ((k_new == nullptr) != (v_new == nullptr)) return fail(YOCO_ERR_INVALID_ARG, "k_new and v_new must both be given or both be null");
  if (k_new && (!aligned16(k_new) || !aligned16(v_new))) return fail(YOCO_ERR_ALIGNMENT, "new row pointer not 16-byte aligned");
  Splits plan;
  rc = plan_decode(*ring, Hq, workspace_bytes, &plan, true);
  if (rc) return rc;
  return run_decode(*ring, q, o, lens, 0, Hq, scale, (float*)workspace, plan, (hipStream_t)stream, "swa_decode", k_new, v_new, 1);
}

int yoco_gret_prefill_workspace(int B, int64_t T, int H, int dk, int dv, int chunk, int dtype, size_t* bytes) {
  if (!bytes) return fail(YOCO_ERR_INVALID_ARG, "bytes is null");
  int rc = check_gret_shape(B, T, H, dk, dv, dtype);
  if (rc) return rc;
  if (chunk <= 0) return fail(YOCO_ERR_INVALID_ARG, "non-positive chunk");
  *bytes = yoco::gret_chunk_supported(B, T, H, dk, dv, chunk, dtype) ? yoco::gret_chunk_workspace(B, T, H, chunk) : 0;
  return YOCO_OK;
}

int yoco_gret_prefill(const void* q, const void* k, const void* v, const float* log_gamma, const void* gate, void* o,
                      const float* state_in, float* state_out, int B, int64_t T, int H, int dk, int dv, int chunk,
                      float scale, int group_norm, float eps, int dtype, void* workspace, size_t workspace_bytes,
                      void* stream) {
  int rc = check_gret_shape(B, T, H, dk, dv, dtype);
  if (rc) return rc;
  if (chunk <= 0) return fail(YOCO_ERR_INVALID_ARG, "non-positive chunk");
  if (!(eps >= 0.f)) return fail(YOCO_ERR_INVALID_ARG, "negative eps");
  if (state_in && !aligned16(state_in)) return fail(YOCO_ERR_ALIGNMENT, "state_in not 16-byte aligned");
  if (state_out && !aligned16(state_out)) return fail(YOCO_ERR_ALIGNMENT, "state_out not 16-byte aligned");
  if (workspace && (((uintptr_t)workspace) & 255u)) return fail(YOCO_ERR_ALIGNMENT, "workspace not 256-byte aligned");
  if (T == 0) {
    if (!state_out || state_out == state_in) return YOCO_OK;
    const size_t nb = (size_t)B * H * dk * dv * sizeof(float);
    if (state_in) return hip_result(hipMemcpyAsync(state_out, state_in, nb, hipMemcpyDeviceToDevice, (hipStream_t)stream), "gret_prefill");
    return hip_result(yoco::launch_fill_zero(state_out, nb / sizeof(float), (hipStream_t)stream), "gret_prefill");
  }
  if (!q || !k || !v || !log_gamma || !o) return fail(YOCO_ERR_INVALID_ARG, "null tensor pointer");
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || (gate && !aligned16(gate)) || (((uintptr_t)log_gamma) & 3u))
    return fail(YOCO_ERR_ALIGNMENT, "tensor pointer not aligned");
  yoco::GretView a;
  a.q = q; a.k = k; a.v = v; a.o = o; a.log_gamma = log_gamma; a.gate = gate;
  a.state_in = state_in; a.state_out = state_out;
  a.T = T; a.B = B; a.H = H; a.dk = dk; a.dv = dv;
  a.scale = scale; a.eps = eps; a.group_norm = group_norm != 0;
  if (workspace && yoco::gret_chunk_supported(B, T, H, dk, dv, chunk, dtype) &&
      workspace_bytes >= yoco::gret_chunk_workspace(B, T, H, chunk))
    return hip_result(yoco::launch_gret_chunk(a, chunk, workspace, (hipStream_t)stream), "gret_prefill (chunkwise)");
  if (!yoco::gret_recurrent_supported(a))
    return fail(YOCO_ERR_UNSUPPORTED, "gated retention: dk %d, dv %d have no kernel (at most 128)", dk, dv);
  return hip_result(yoco::launch_gret_recurrent(a, dtype, (hipStream_t)stream), "gret_prefill");
}

int yoco_gret_decode(const void* q, const void* k, const void* v, const float* log_gamma, const void* gate, void* o, float* state,
                     int B, int H, int dk, int dv, float scale, int group_norm, float eps, int dtype, void* stream) {
  int rc = check_gret_shape(B, 1, H, dk, dv, dtype);
  if (rc) return rc;
  if (!(eps >= 0.f)) return fail(YOCO_ERR_INVALID_ARG, "negative eps");
  if (!q || !k || !v || !log_gamma || !o || !state) return fail(YOCO_ERR_INVALID_ARG, "null pointer");
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(state) || (gate && !aligned16(gate)) ||
      (((uintptr_t)log_gamma) & 3u))
    return fail(YOCO_ERR_ALIGNMENT, "pointer not aligned");
  yoco::GretView a;
  a.q = q; a.k = k; a.v = v; a.o = o; a.log_gamma = log_gamma; a.gate = gate;
  a.state_in = state; a.state_out = state;
  a.T = 1; a.B = B; a.H = H; a.dk = dk; a.dv = dv;
  a.scale = scale; a.eps = eps; a.group_norm = group_norm != 0;
  if (!yoco::gret_recurrent_supported(a))
    return fail(YOCO_ERR_UNSUPPORTED, "gated retention: dk %d, dv %d have no kernel (at most 128)", dk, dv);
  return hip_result(yoco::launch_gret_recurrent(a, dtype, (hipStream_t)stream), "gret_decode");
}

int yoco_stack_step_scratch(const yoco_stack* st, size_t* bytes) {
  if (!st || !bytes) return fail(YOCO_ERR_INVALID_ARG, "null argument");
  int rc = check_stack(st);
  if (rc) return rc;
  *bytes = StackScratch(*st, nullptr).bytes;
  return YOCO_OK;
}

int yoco_stack_step(const yoco_stack* st, const void* x, const yoco_kv_cache* rings, float* const* states, const yoco_kv_cache* cache,
                    int64_t pos, void* x_out, void* logits, void* scratch, size_t scratch_bytes, void* workspace,
                    size_t workspace_bytes, void* stream) {
  if (!st || !x || !cache || !scratch || !workspace) return fail(YOCO_ERR_INVALID_ARG, "null argument");
  int rc = check_stack(st);
  if (rc) return rc;
  rc = check_cache(cache);
  if (rc) return rc;
  const bool self = rings || states;
  if (self && (st->gret ? !states : !rings)) return fail(YOCO_ERR_INVALID_ARG, "the self-decoder's caches do not match its kind");
  if (self && (!st->kv_ln || !st->w_kv)) return fail(YOCO_ERR_INVALID_ARG, "stack: missing weights of the global cache");
  if (cache->B != 1 || cache->Hkv != st->Hkv || cache->d != st->d || io_dtype(*cache) != YOCO_BF16)
    return fail(YOCO_ERR_INVALID_ARG, "the cache does not match the stack");
  if (cache->dtype == YOCO_INT8 && !yoco::decode_i8_supported(*cache, st->Hq))
    return fail(YOCO_ERR_UNSUPPORTED, "an 8-bit cache serves up to 16 query heads per KV head, not %d", st->Hq / cache->Hkv);
  if (pos < 0) return fail(YOCO_ERR_INVALID_ARG, "negative position %lld", (long long)pos);
  if (!aligned16(x) || !aligned16(x_out) || !aligned16(logits) || !aligned16(scratch) || !aligned16(workspace))
    return fail(YOCO_ERR_ALIGNMENT, "pointer not 16-byte aligned");
  const StackScratch t(*st, (char*)scratch);
  if (scratch_bytes < t.bytes) return fail(YOCO_ERR_WORKSPACE, "scratch %zu < %zu bytes", scratch_bytes, t.bytes);
  Splits plan, ring_plan;
  rc = plan_decode(*cache, st->Hq, workspace_bytes, &plan, false);
  if (rc) return rc;
  const bool in_rings = self && !st->gret && st->n_self > 0;
  if (self && st->gret) {
    if (!(st->eps >= 0.f)) return fail(YOCO_ERR_INVALID_ARG, "negative eps");
    for (int i = 0; i < st->n_self; ++i) {
      if (!states[i]) return fail(YOCO_ERR_INVALID_ARG, "state %d is null", i);
      if (!aligned16(states[i])) return fail(YOCO_ERR_ALIGNMENT, "state %d is not 16-byte aligned", i);
    }
  }
  if (in_rings) {
    for (int i = 0; i < st->n_self; ++i) {
      rc = check_cache(rings + i);
      if (rc) return rc;
      if (rings[i].B != 1 || rings[i].Hkv != st->Hkv_self || rings[i].d != st->d || rings[i].dtype != YOCO_BF16 ||
          rings[i].N_cap != rings[0].N_cap)
        return fail(YOCO_ERR_INVALID_ARG, "ring %d does not match the stack", i);
    }
    rc = plan_decode(rings[0], st->Hq, workspace_bytes, &ring_plan, true);
    if (rc) return rc;
  }

  hipStream_t s = (hipStream_t)stream;
  const int dm = st->d_model, qd = st->Hq * st->d, kd = st->Hkv_self * st->d, ckd = st->Hkv * st->d;
  hipError_t e = hipSuccess;
  auto gemv = [&](const void* in, const void* gain, const void* W, int N, int K, const void* res, int glu, void* out, int n_plain) {
    if (e != hipSuccess) return;
    yoco::GemvArgs g;
    g.x = in; g.gain = gain; g.W = W; g.res = res; g.out = out;
    g.log_gamma = t.log_gamma;
    g.N = N; g.K = K; g.n_plain = n_plain; g.glu = glu;
    g.eps = st->eps; g.inv_tau = 1.f / st->tau;
    e = yoco::launch_gemv(g, s);
  };
  const void* cur = x;
  // W_O, the residual and the SwiGLU half of Eq. 1; `last`: where the residual stream goes
  auto finish_layer = [&](const yoco_stack_layer& L, void* last) {
    gemv(t.o, nullptr, L.w_o, dm, qd, cur, 0, t.y, dm);
    gemv(t.y, L.ln2, L.w_gu, st->ffn, dm, nullptr, 1, t.h, st->ffn);
    gemv(t.h, nullptr, L.w_2, dm, st->ffn, t.y, 0, last, dm);
    cur = last;
  };
  if (self) {
    for (int i = 0; i < st->n_self; ++i) {
      const yoco_stack_layer& L = st->self[i];
      const int plain = qd + 2 * kd + (st->gret ? qd : 0);
      gemv(cur, L.ln1, L.w_in, plain + (st->gret ? st->Hq : 0), dm, nullptr, 0, t.in, plain);
      if (e != hipSuccess) return hip_result(e, "stack_step");
      bf16_raw *q = t.in, *k = q + qd, *v = k + kd, *gate = v + kd;
      if (st->gret) {
        rc = yoco_gret_decode(q, k, v, t.log_gamma, gate, t.o, states[i], 1, st->Hq, st->d, st->d, st->scale, 1, st->eps, YOCO_BF16, stream);
      } else {
        rc = run_decode(rings[i], q, t.o, nullptr, pos + 1, st->Hq, st->scale, (float*)workspace, ring_plan, s, "stack_step", k, v, 1, weights_ahead(*st, L, rings[i], pos + 1));
      }
      if (rc) return rc;
      finish_layer(L, t.x);
    }
    // Eq. 2 for the new row and the first cross-decoder layer's queries read the same input: one launch, which stores the row
    // in a bf16 cache itself (past the capacity nothing is stored, as in yoco_kv_cache_append)
    yoco::GemvPair g = {};
    g.x = cur; g.K = dm; g.eps = st->eps;
    g.gain = st->kv_ln; g.W = st->w_kv; g.N = g.n_plain = 2 * ckd; g.out = t.in + qd;
    g.gain2 = st->cross[0].ln1; g.W2 = st->cross[0].w_in; g.N2 = qd; g.out2 = t.in;
    if (cache->dtype == YOCO_BF16 && pos < cache->N_cap) {
      g.k_row = (bf16_raw*)cache->k + pos * st->d;
      g.v_row = (bf16_raw*)cache->v + pos * st->d;
      g.head_stride = cache->N_cap * st->d;
    }
    if (e == hipSuccess) e = yoco::launch_gemv_pair(g, s);
    if (e != hipSuccess) return hip_result(e, "stack_step");
    if (!g.k_row && pos < cache->N_cap) {
      rc = yoco_global_kv_write(cache, t.in + qd, t.in + qd + ckd, 0, pos, 1, YOCO_BF16, stream);
      if (rc) return rc;
    }
  }
  for (int i = 0; i < st->n_cross; ++i) {
    const yoco_stack_layer& L = st->cross[i];
    if (i > 0 || !self) gemv(cur, L.ln1, L.w_in, qd, dm, nullptr, 0, t.in, qd);
    if (e != hipSuccess) return hip_result(e, "stack_step");
    rc = run_decode(*cache, t.in, t.o, nullptr, pos + 1, st->Hq, st->scale, (float*)workspace, plan, s, "stack_step", nullptr, nullptr, 0, weights_ahead(*st, L, *cache, pos + 1));
    if (rc) return rc;
    finish_layer(L, i + 1 == st->n_cross && x_out ? x_out : t.x);
  }
  if (logits) gemv(cur, st->final_ln, st->w_out, st->vocab, dm, nullptr, 0, logits, st->vocab);
  return hip_result(e, "stack_step");
}

int yoco_norm_rows(const void* x, const void* add, void* y, const void* gain, void* xn, int64_t rows, int dim, float eps, void* stream) {
  if (!x || !gain || !xn || (add && !y)) return fail(YOCO_ERR_INVALID_ARG, "null pointer");
  if (rows < 0 || rows > INT32_MAX || dim <= 0) return fail(YOCO_ERR_INVALID_ARG, "rows or dim out of range");
  if (dim % 8 || !aligned16(x) || !aligned16(add) || !aligned16(y) || !aligned16(gain) || !aligned16(xn))
    return fail(YOCO_ERR_ALIGNMENT, "pointer not 16-byte aligned or dim not a multiple of 8");
  if (rows == 0) return YOCO_OK;
  return hip_result(yoco::launch_norm_rows(x, add, y, gain, xn, rows, dim, eps, (hipStream_t)stream), "norm_rows");
}

int yoco_glu_rows(const void* gu, void* h, int64_t rows, int ffn, void* stream) {
  if (!gu || !h) return fail(YOCO_ERR_INVALID_ARG, "null pointer");
  if (rows < 0 || ffn <= 0) return fail(YOCO_ERR_INVALID_ARG, "rows or ffn out of range");
  if (ffn % 8 || !aligned16(gu) || !aligned16(h)) return fail(YOCO_ERR_ALIGNMENT, "pointer not 16-byte aligned or ffn not a multiple of 8");
  if (rows == 0) return YOCO_OK;
  return hip_result(yoco::launch_glu_rows(gu, h, rows, ffn, (hipStream_t)stream), "glu_rows");
}

int yoco_ceiling_mfma(const void* seed, void* sink, int iters, int workgroups, void* stream) {
  if (!seed || !sink) return fail(YOCO_ERR_INVALID_ARG, "null pointer");
  if (!aligned16(seed)) return fail(YOCO_ERR_ALIGNMENT, "seed not 16-byte aligned");
  if (iters <= 0 || workgroups <= 0) return fail(YOCO_ERR_INVALID_ARG, "non-positive iters or workgroups");
  return hip_result(yoco::launch_mfma_ceiling(seed, sink, iters, workgroups, (hipStream_t)stream), "ceiling_mfma");
}

int yoco_ceiling_attn_loop(const void* seed, void* sink, int iters, int workgroups, int mode, void* stream) {
  if (!seed || !sink) return fail(YOCO_ERR_INVALID_ARG, "null pointer");
  if (!aligned16(seed)) return fail(YOCO_ERR_ALIGNMENT, "seed not 16-byte aligned");
  if (iters <= 0 || workgroups <= 0) return fail(YOCO_ERR_INVALID_ARG, "non-positive iters or workgroups");
  if (mode != 1 && mode != 2) return fail(YOCO_ERR_INVALID_ARG, "mode %d is neither 1 (LDS-fed products) nor 2 (with the softmax work)", mode);
  return hip_result(yoco::launch_attn_loop_ceiling(seed, sink, iters, workgroups, mode, (hipStream_t)stream), "ceiling_attn_loop");
}

int yoco_ceiling_stream_read(const void* buf, size_t bytes, void* sink, int workgroups, void* stream) {
  if (!buf || !sink) return fail(YOCO_ERR_INVALID_ARG, "null pointer");
  if (!aligned16(buf) || bytes % 16) return fail(YOCO_ERR_ALIGNMENT, "buffer not 16-byte aligned or size not a multiple of 16");
  if (bytes == 0 || workgroups <= 0) return fail(YOCO_ERR_INVALID_ARG, "empty buffer or non-positive workgroups");
  return hip_result(yoco::launch_stream_read(buf, bytes, sink, workgroups, (hipStream_t)stream), "ceiling_stream_read");
}

}  // extern "C"
#pragma GCC visibility pop
