// The end of a split-KV decode workgroup: merge its wavefronts, publish the split's partial results, and, where splits
// and heads are few (decode_meets_in_launch), merge the splits. A wavefront has every fourth head of the KV head to itself:
// it publishes its split of them, and merges those of which it finds every split published. One launch per decode step
// then, which saves up to a microsecond and 2.4 us of host time against a merge launch. That one wavefront's reading is
// a serial chain that grows with splits and heads, so the others are left for a merge launch, a workgroup per query head.
//
// Nothing has to be cleared beforehand. A split is published by writing the call's tag (64 bits, never used twice by a
// process, drawn around a random start) into the spare words of its partial; whoever sees all tags merges, and puts
// zeros back, so that a captured launch can be replayed. A wavefront publishes before it looks, and both go to the
// device-coherent level, so the last one to publish sees all tags; two that see them both write the same bits. None
// waits for another.
#pragma once
#include <type_traits>

#include "lanes.h"
#include "yoco_common.h"

namespace yoco {

constexpr int kMaxDecodeSplits = 256;
// Ragged batches get no more splits than CUs where a split has rows enough to pay for finding the shares (0.4 us) and the
// sequences are few enough that this leaves no more than a third of the CUs' places unused (760 ragged batches of 2 to 48
// sequences of 1500 to 44564 rows, 16 to 64 query heads, bf16 and 8-bit: a twentieth faster on the mean than shares of
// rows / CUs, which made up to a tenth more workgroups than CUs and launched those with rows among those without: 2 x 16
// heads x 44564 rows, lengths 0.88 of it, 147 us, now 103; 8 x 8 x 25000, 0.69, 136 and 93).
// From four sequences on 320 rows pay for it (5 x 8 heads x 5000 rows 16.3 us, now 14.7, 9 x 8 x 2833 17.3 and 15.8, 8 bits 14 x 8 x
// 1963 13.5 and 11.2; at 256 rows 8 x 8 x 1500 9.4 and 9.6); of two or three the plain shares are about as good (3 x 16 x 2713
// 11.9, 12.2 with the search).
constexpr int kLongSplit = 512, kLongSplitOfMany = 320;
constexpr float kGoodFit = 1.5f;
constexpr float kLn2 = 0.6931471805599453f;

struct SplitOut {
  float* ws;                 // [B][Hq][splits][128 + 4]: vector, max (log2 units), sum, tag
  bf16_t* o;                 // [B,Hq,128]
  int splits;                // the most a sequence can be split into
  float inv_ragged;          // 1 / how many workgroups the whole batch should make, when its lengths differ
  float inv_even;            // ... and when they do not
  int even;                  // that many for each sequence
  int places;                // how many (sequence, split) pairs have a CU of their own for each KV head; 0: do not ask
  unsigned long long tag;    // 0: the splits are left for a merge launch
};

// Which rows a workgroup takes. A sequence gets as many splits as its length asks for, so that a batch of ragged lengths
// ends together (8 sequences of 375 to 3000 rows x 8 KV heads: the longest no longer runs on as many workgroups as the
// shortest). GRAIN: what a split's rows are a multiple of (a step of each of its four wavefronts).
struct SplitRows {
  int b, g, sp;              // sequence, KV head and split
  int64_t lo, hi;            // rows of this split, lo >= hi: nothing to do
  int splits;                // of this sequence; 0: the sequence is empty, split 0 stores zeros
  float total;               // rows of the whole batch (of its capacity where nothing is split)
};

// Inclusive scan over the wavefront with 0 as the neutral element: within rows of 16 lanes, then a row's last value into
// the next one, then the lower half's into the upper half.
template <int CTRL, int ROWS, typename F>
__device__ __forceinline__ int dpp_step(int x, F f) { return f(x, __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xf, false)); }
template <typename F>
__device__ __forceinline__ int lane_scan(int x, F f) {
  x = dpp_step<0x111, 0xf>(x, f);    // row_shr:1
  x = dpp_step<0x112, 0xf>(x, f);    // row_shr:2
  x = dpp_step<0x114, 0xf>(x, f);    // row_shr:4
  x = dpp_step<0x118, 0xf>(x, f);    // row_shr:8
  x = dpp_step<0x142, 0xa>(x, f);    // row_bcast:15 into rows 1 and 3
  return dpp_step<0x143, 0xc>(x, f);  // row_bcast:31 into rows 2 and 3
}
__device__ __forceinline__ int last_lane(int x) { return __builtin_amdgcn_readlane(x, 63); }
__device__ __forceinline__ int lanes_max(int x) {           // of values that are not negative
  return last_lane(lane_scan(x, [](int a, int b) { return a > b ? a : b; }));
}
__device__ __forceinline__ int lanes_sum(int x) { return last_lane(lane_scan(x, [](int a, int b) { return a + b; })); }
__device__ __forceinline__ float lanes_sum(float x) {
  return __int_as_float(last_lane(lane_scan(__float_as_int(x), [](int a, int b) { return __float_as_int(__int_as_float(a) + __int_as_float(b)); })));
}
__device__ __forceinline__ float lanes_max(float x) {       // of values that are not negative
  return __int_as_float(last_lane(lane_scan(__float_as_int(x), [](int a, int b) { return a > b ? a : b; })));
}

// How many splits `len` rows ask for at 1 / inv_share rows a split (a tenth over is no reason for one more).
__device__ __forceinline__ int splits_for(float len, float inv_share, int most) {
  const int n = (int)ceilf(len * inv_share - 0.1f);
  return n < 1 ? 1 : n > most ? most : n;
}
// ceil(a / b), or one more, for positive whole numbers below 2^24.
__device__ __forceinline__ int about_ceil_div(int a, int b) {
  const int q = (int)((float)(a + b - 1) * __builtin_amdgcn_rcpf((float)b));
  return q * b < a ? q + 1 : q;
}
// How many splits of `each` steps hold `steps`, no more than the n that `each` was made for.
__device__ __forceinline__ int splits_of(int steps, int each, int n) {
  const int s = about_ceil_div(steps, each);
  return s < n ? s : n;
}

// One length alone: a step a split as far as there are splits, or none where that saves fewer than three steps (of 256 rows:
// two), because a meeting costs more (a merge launch there is in any case). us, 16 heads in bf16, a cache of 3000 rows: 200
// rows (2 steps) 6.8 in two, 5.7 whole; 260 (3 steps) 8.0 in two, 6.5 whole; 520 (5 steps) 8.0 in four, 6.6 in five.
template <int GRAIN>
__device__ __forceinline__ int one_length_splits(int len, int most, bool meets) {
  const int steps = (len + GRAIN - 1) / GRAIN, n = steps < most ? steps : most;
  return n > 1 && (!meets || steps - about_ceil_div(steps, n) >= (GRAIN < 256 ? 3 : 2)) ? n : 1;
}

// A decode kernel's last parameter, or none: ReadAhead, what the workgroups behind those of the splits read, or SplitFirst, that only
// the first pairs of sequence and KV head are split. (A parameter, and a kernel, of its own: as an argument that is never used
// either cost the others up to 3 %.)
template <typename... Last>
constexpr bool kSplitsFirst = (std::is_same<Last, SplitFirst>::value || ...);
template <int GRAIN, typename... Last>
__device__ __forceinline__ SplitRows split_rows(const SplitOut& out, const yoco_kv_cache& c, const int64_t* lens, int64_t fixed_len, const Last&... last) {
  // 32-bit arithmetic: 2^31 rows of 132 bytes and more do not fit any GPU this runs on
  auto clamp_len = [&](int64_t n) { return (int)(n < 0 ? 0 : n > c.N_cap ? c.N_cap : n); };
  const int B = c.B;
  SplitRows r;
  r.b = blockIdx.y;
  r.g = blockIdx.x;
  r.sp = blockIdx.z;
  int len, n = 1;
  r.total = (float)B * (float)c.N_cap;               // unsplit: nothing depends on the other lengths
  if constexpr (kSplitsFirst<Last...>) {
    // Whole, the launch lasts as long as the two units of a CU that has two, or as the longest sequence. Cut, it lasts as long as the longest
    // and a part of the first, and a meeting's time, some 224 rows in bf16; what is too short for parts only waits for their workgroups. So
    // the lengths decide, the same in all workgroups. 8-bit caches, whose walk waits more for the vector ALU than for memory, lose
    // nothing down to no rows at all (48 x 8:24 of 128 to 1024 rows, 166 rows more than the longest and a part, 17.0 whole, 16.0 cut). us,
    // whole, always cut, so: 12 x 24 heads of 128 to 1024 rows, the draws that are worst and best for a cut, 15.2, 17.6, 15.2 and 21.4, 16.5, 16.8; 33
    // x 8:24 x 500 to 4000 in 8 bits 30.0, 32.3, 30.2 and 44.1, 35.5, 36.2; 40 x 8:24 x 375 to 3000 56.5, 60.1, 57.0 and 88.0, 63.2, 63.6; all of
    // 100 rows 5.4, 6.3, 5.8. Looking at the lengths takes 0.2 to 0.5.
    const SplitFirst& f = (last, ...);
    asm volatile("" : : "s"(f.split), "s"(f.apart), "s"(f.apart_most), "s"(out.splits));    // not a trip for the arguments behind the branch
    int mine = 0, front = (int)c.N_cap;
    bool worth = true;                               // of many sequences some pair is long
    if (B <= 64) {                                   // a lane per sequence
      const int i = threadIdx.x & 63;
      const int64_t n_i = lens[i < B ? i : 0], n_x = lens[i + f.apart < B ? i + f.apart : 0], n_y = lens[i + f.apart_most < B ? i + f.apart_most : 0];
      mine = i < B ? clamp_len(n_i) : 0;
      const int x = clamp_len(n_x), y = i + f.apart_most < B ? clamp_len(n_y) : 0, first = i * c.Hkv < f.split ? mine : 0;
      const int pair = lanes_max(first ? first + (x > y ? x : y) : 0), longest = lanes_max(mine);
      front = lanes_max(first);
      worth = (pair - longest - (GRAIN < 256 ? 224 : 0)) * out.splits >= front;
    }
    const int id = r.b * c.Hkv + r.g, more = f.split * (out.splits - 1);
    int unit = id;
    bool split = false;
    if (worth && one_length_splits<GRAIN>(front, out.splits, true) > 1) {
      // The splits come first: of a CU's two workgroups the first is the faster one, and theirs have a meeting before them (16 x 24 heads x
      // 1024 rows, last, 35.9 us; first 34.3).
      auto quotient = [](int x, int by) { return __builtin_amdgcn_readfirstlane((int)(((float)x + 0.5f) * __builtin_amdgcn_rcpf((float)by))); };   // exact: x < 2^20
      split = id < f.split + more;
      unit = split ? quotient(id, out.splits) : id - more;
      r.b = quotient(unit, c.Hkv);
      r.g = unit - r.b * c.Hkv;
      if (split) r.sp = id - unit * out.splits;
    }
    if (unit >= B * c.Hkv) {                         // one to spare: a part of a sequence that has one
      r.b = 0;
      r.sp = 1;
    }
    len = B <= 64 ? __builtin_amdgcn_readlane(mine, r.b) : clamp_len(lens[r.b]);
    if (split) n = one_length_splits<GRAIN>(len, out.splits, true);
  } else if (out.splits == 1 || !lens || B == 1) {
    len = clamp_len(lens ? lens[r.b] : fixed_len);
    if (out.splits > 1) {
      r.total = (float)len * (float)B;
      n = one_length_splits<GRAIN>(len, out.even < out.splits ? out.even : out.splits, out.tag != 0);
    }
  } else {
    // The same float arithmetic in every workgroup: all agree on every sequence's splits.
    const int lane = threadIdx.x & 63;
    const int mine = lane < B ? clamp_len(lens[lane]) : 0;       // a lane per sequence, of the first 64
    float sum = (float)mine, longest = (float)mine;
    for (int i = lane + 64; i < B; i += 64) {
      const float n_i = (float)clamp_len(lens[i]);
      sum += n_i;
      longest = fmaxf(longest, n_i);
    }
    r.total = lanes_sum(sum);
    const bool ragged = lanes_max(longest) * (float)B * 16.f > r.total * 17.f;       // equal: the longest is within a sixteenth of the mean
    float share = fmaxf(r.total * (float)c.Hkv * (ragged ? out.inv_ragged : out.inv_even), (float)GRAIN);
    bool fits = false;
    const float fl = (float)mine;
    // Not where all splits that there can be have one anyway (8 x 8 heads x 2299 rows, four splits at most: 12.3 us, 12.6 with it).
    if (__builtin_expect(ragged && B * out.splits > out.places && 2 * B <= out.places && B <= 64 && share >= (float)(B < kManySequences ? kLongSplit : kLongSplitOfMany), 0)) {
      // The smallest share, nearly, with which every split has a CU of its own, because a CU with two makes the launch wait.
      float s = fmaxf(r.total / (float)out.places, (float)GRAIN);
      for (int i = 0; i < 32 && !fits; ++i) {
        const int over = lanes_sum(lane < B ? splits_for(fl, __builtin_amdgcn_rcpf(s), out.splits) : 0) - out.places;
        fits = over <= 0;
        if (!fits) s *= 1.f + fmaxf(0.03f, 0.5f * (float)over / (float)out.places);
      }
      fits = fits && s * (float)out.places < kGoodFit * r.total;       // not where sequences too short to fill a place waste many
      share = fits ? s : share;
    }
    const float inv_share = __builtin_amdgcn_rcpf(share);
    if (__builtin_expect(!fits, 1)) {
      len = B <= 64 ? __builtin_amdgcn_readlane(mine, r.b) : clamp_len(lens[r.b]);
      n = splits_for((float)len, inv_share, out.splits);
    } else {
      const int wanted = splits_for(fl, inv_share, out.splits), steps = (mine + GRAIN - 1) / GRAIN;
      const int live = lane < B ? (steps ? splits_of(steps, about_ceil_div(steps, wanted), wanted) : 1) : 0;   // an empty sequence has one, which stores zeros
      // Workgroups are dealt to the CUs in order, and those without rows leave at once: the ones with rows come first, so
      // that no CU gets two while another gets none.
      auto locate = [&](int count, int j) {          // the sequence that holds place j of all counts, and its place there
        const int upto = lane_scan(count, [](int a, int b) { return a + b; });
        r.b = __builtin_ctzll(__builtin_amdgcn_ballot_w64(j < upto) | (1ull << 63));
        r.sp = j - __builtin_amdgcn_readlane(upto - count, r.b);
      };
      const int j = (int)blockIdx.y + B * (int)blockIdx.z, all = lanes_sum(live);
      locate(live, j);
      if (j >= all) {                                // one of those without rows
        locate(lane < B ? out.splits - live : 0, j - all);
        r.sp += __builtin_amdgcn_readlane(live, r.b);
      }
      len = __builtin_amdgcn_readlane(mine, r.b);
      n = __builtin_amdgcn_readlane(wanted, r.b);
    }
  }
  n = __builtin_amdgcn_readfirstlane(n);
  const int steps = (len + GRAIN - 1) / GRAIN;
  int each = steps;                                  // even shares of this sequence
  r.splits = steps ? 1 : 0;
  if (n > 1) {
    each = about_ceil_div(steps, n);
    r.splits = steps ? splits_of(steps, each, n) : 0;
  }
  r.lo = (int64_t)r.sp * (each * GRAIN);
  r.hi = r.lo + each * GRAIN < len ? r.lo + each * GRAIN : len;
  return r;
}

// Device-coherent accesses (they bypass the per-XCD L2s).
__device__ __forceinline__ unsigned long long get_u64(const void* p) {
  return __hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_u64(void* p, unsigned long long x) {
  __hip_atomic_store((unsigned long long*)p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_pair(float* p, float x, float y) {
  put_u64(p, (unsigned long long)__float_as_uint(x) | ((unsigned long long)__float_as_uint(y) << 32));
}
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The merge of a head's S <= N published splits by one wavefront: o = sum_s 2^(m_s - M) o_s / sum_s 2^(m_s - M) l_s. Lane s
// takes the maximum and sum of split s, every lane owns a pair of dims of all vectors, and all of it is requested together:
// one trip to memory. Order and assignment are fixed: results are bit-reproducible whoever merges. Every lane used to take
// all maxima and sums: 16 splits x 3 heads of 2000 rows 7.2 us, now 6.7; 8 x 8 of 900 rows 8.6 and 7.6.
template <int N>
__device__ __forceinline__ void merge_head(const float* p, size_t stride, int S, bf16_t* o) {
  static_assert(N <= 64, "a lane a split");
  const int lane = threadIdx.x & 63, e = lane * 2;
  const unsigned long long ml = get_u64(p + (lane < S ? lane : S - 1) * stride + 128);
  unsigned long long x[N];
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = get_u64(p + (i < S ? i : S - 1) * stride + e);
  const float m = __uint_as_float((unsigned)ml), M = over64<LaneMax>(m);
  const float base = M == -INFINITY ? 0.f : M;                                         // empty splits only
  const float f = lane < S ? __builtin_amdgcn_exp2f(m - base) : 0.f;
  const float L = over64<LaneSum>(f * __uint_as_float((unsigned)(ml >> 32)));
  float a = 0.f, b = 0.f;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float fi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), i));
    a = fmaf(fi, __uint_as_float((unsigned)x[i]), a);
    b = fmaf(fi, __uint_as_float((unsigned)(x[i] >> 32)), b);
  }
  const float inv = L > 0.f ? 1.f / L : 0.f;                                           // no visible row -> zeros
  *(unsigned*)(o + e) = (unsigned)f32_to_bf16(a * inv) | ((unsigned)f32_to_bf16(b * inv) << 16);
}

// What the workgroups behind those of the splits do: read weights that the next launches will stream, so that these find them in
// the L2 of their XCD. A decode step over a short cache is latency and leaves most of the bandwidth idle. Workgroups are dealt to
// the 8 XCDs round robin, of this launch as of the next: piece i goes to an XCD that has workgroup i of the launch that reads it.
__device__ __forceinline__ void read_ahead(const ReadAhead& w, int splits) {
  const int before = gridDim.x * gridDim.y * splits, all = gridDim.x * gridDim.y * gridDim.z;
  const int me = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  const int first = (me & 7) + 8 * ((me - before) >> 3), step = (all - before) & ~7;
  for (int m = 0; m < 2; ++m)
    for (int i = first; i < w.part[m].pieces; i += step)
      for (int64_t at = (int64_t)i * w.part[m].bytes, half = 0; half < w.part[m].halves; ++half, at += w.part[m].to_second)
        for (int e = threadIdx.x * 16; e < w.part[m].bytes; e += 4 * 256 * 16) {
          unsigned x[4][4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int b = e + u * 256 * 16;
            const uint4 v = *(const uint4*)((const char*)w.part[m].from + at + (b < w.part[m].bytes ? b : e));
            x[u][0] = v.x; x[u][1] = v.y; x[u][2] = v.z; x[u][3] = v.w;
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) asm volatile("" : : "v"(x[u][0]), "v"(x[u][1]), "v"(x[u][2]), "v"(x[u][3]));
        }
}

// True for a workgroup that has read ahead and is done.
template <typename... Last>
__device__ __forceinline__ bool has_read_ahead(int splits, const Last&... last) {
  if constexpr ((std::is_same<Last, ReadAhead>::value || ...)) {
    if ((int)blockIdx.z < splits) return false;
    (read_ahead(last, splits), ...);
    return true;
  }
  return false;
}

// 256 threads, head_dim 128. red_o [4][GS][128] and red_ml [4][GS][2] (max in log2 units, sum) hold the wavefronts'
// states in LDS, complete behind a barrier; head0 = first query head of the KV head, in rows of o. From here on a
// wavefront has its heads to itself (every fourth): no barrier stands between the trips to memory, of which a meeting takes
// four, one after another (the partial's way out, the tag's, all tags back, all partials back).
template <int GS>
__device__ __forceinline__ void finish_split(const SplitOut& out, float (*red_o)[GS][128], float (*red_ml)[GS][2], int G, size_t head0, int sp,
                                             int S) {
  constexpr int kD = 128, kHeads = (GS + 3) / 4;             // heads of a wavefront
  constexpr int kMeetHeads = kHeads < 2 ? kHeads : 2;        // where splits meet: at most 8 heads, of more than 4 at most 8 splits
  const size_t stride = partial_stride(kD);
  const size_t per_head = out.splits * stride;
  const bool whole = out.tag ? S <= 1 : out.splits <= 1;     // a single split is the whole answer
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63, e = lane * 2;
#pragma unroll
  for (int i = 0; i < kHeads; ++i) {
    const int h = wave + 4 * i;
    if (h >= G) break;
    const float M = fmaxf(fmaxf(red_ml[0][h][0], red_ml[1][h][0]), fmaxf(red_ml[2][h][0], red_ml[3][h][0]));
    float l = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float f = __builtin_amdgcn_exp2f(red_ml[w][h][0] - M);
      l = fmaf(f, red_ml[w][h][1], l);
      o0 = fmaf(f, red_o[w][h][e], o0);
      o1 = fmaf(f, red_o[w][h][e + 1], o1);
    }
    if (whole) {
      *(unsigned*)(out.o + (head0 + h) * kD + e) =
          (unsigned)f32_to_bf16(l > 0.f ? o0 / l : 0.f) | ((unsigned)f32_to_bf16(l > 0.f ? o1 / l : 0.f) << 16);
      continue;
    }
    float* const p = out.ws + (head0 + h) * per_head + sp * stride;
    const float m = l > 0.f ? M : -INFINITY;
    if (!out.tag) {
      p[e] = o0;
      p[e + 1] = o1;
      if (lane == 0) {
        p[kD] = m * kLn2;                            // the merge launch works with natural exponents
        p[kD + 1] = l;
      }
      continue;
    }
    put_pair(p + e, o0, o1);
    if (lane == 0) put_pair(p + kD, m, l);
  }
  if (whole || !out.tag) return;
  wait_stores();                                             // this wavefront's heads are visible to the whole device
  float* const tags = out.ws + (head0 + wave) * per_head + kD + 2;           // head i, split s: tags + 4 i * per_head + s * stride
  if (lane < kMeetHeads && wave + 4 * lane < G) put_u64(tags + 4 * lane * per_head + sp * stride, out.tag);
  wait_stores();
  unsigned long long seen[kMeetHeads];                       // of all of its heads in one trip
#pragma unroll
  for (int i = 0; i < kMeetHeads; ++i)
    seen[i] = wave + 4 * i < G ? get_u64(tags + 4 * i * per_head + (lane < S ? lane : S - 1) * stride) : 0ull;
#pragma unroll
  for (int i = 0; i < kMeetHeads; ++i) {
    if (wave + 4 * i >= G) break;
    if (__builtin_amdgcn_ballot_w64(seen[i] != out.tag)) continue;
    float* const t = tags + 4 * i * per_head;
    const float* const p = t - (kD + 2);
    bf16_t* const o = out.o + (head0 + wave + 4 * i) * kD;
    if (S <= 4) merge_head<4>(p, stride, S, o);
    else if (kMeetHeads > 1 || S <= 8) merge_head<8>(p, stride, S, o);
    else merge_head<kMeetSplits>(p, stride, S, o);
    if (lane < S) put_u64(t + lane * stride, 0ull);
  }
}

}  // namespace yoco
