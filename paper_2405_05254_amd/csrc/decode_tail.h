// The end of a split-KV decode workgroup: merge its wavefronts, publish the split's partial result, and, where splits
// and heads are few (decode_meets_in_launch), let the workgroup that finds every split of its (sequence, KV head)
// published merge them. One launch per decode step then, which saves up to a microsecond and 3 us of host time against
// a merge launch. That one workgroup's reading is a serial chain that grows with splits and heads, so the others are left
// for a merge launch, a workgroup per query head.
//
// Nothing has to be cleared beforehand. A split is published by writing the call's tag (64 bits, never used twice by a
// process, drawn around a random start) into the spare words of its partial; whoever sees all tags merges, and puts
// zeros back, so that a captured launch can be replayed. A workgroup publishes before it looks, and both go to the
// device-coherent level, so the last one to publish sees all tags; two that see them both write the same bits. No
// workgroup waits for another.
#pragma once
#include "yoco_common.h"

namespace yoco {

constexpr int kMaxDecodeSplits = 256;
constexpr float kLn2 = 0.6931471805599453f;

struct SplitOut {
  float* ws;                 // [B][Hq][splits][128 + 4]: vector, max (log2 units), sum, tag
  bf16_t* o;                 // [B,Hq,128]
  int splits;                // the most a sequence can be split into
  float inv_ragged;          // 1 / how many workgroups the whole batch should make, when its lengths differ
  float inv_even;            // ... and when they do not
  unsigned long long tag;    // 0: the splits are left for a merge launch
};

// Which rows a workgroup takes. The batch's rows, times its KV heads, are shared out over `workgroups` workgroups: a
// sequence gets as many splits as its length asks for, so that a batch of ragged lengths ends together (8 sequences of
// 375 to 3000 rows x 8 KV heads: the longest no longer runs on as many workgroups as the shortest). GRAIN: what a
// split's rows are a multiple of (a step of each of its four wavefronts).
struct SplitRows {
  int64_t lo, hi;            // rows of this split, lo >= hi: nothing to do
  int splits;                // of this sequence; 0: the sequence is empty, split 0 stores zeros
  float total;               // rows of the whole batch (of its capacity where nothing is split)
};

template <int GRAIN>
__device__ __forceinline__ SplitRows split_rows(const SplitOut& out, const yoco_kv_cache& c, const int64_t* lens, int64_t fixed_len, int b, int sp) {
  // 32-bit arithmetic: 2^31 rows of 132 bytes and more do not fit any GPU this runs on
  auto clamp_len = [&](int64_t n) { return (unsigned)(n < 0 ? 0 : n > c.N_cap ? c.N_cap : n); };
  const unsigned len = clamp_len(lens ? lens[b] : fixed_len);
  unsigned n = 1;
  float total = (float)c.B * (float)c.N_cap;         // unsplit: nothing depends on the other lengths
  if (out.splits > 1) {
    total = (float)len;
    float inv = out.inv_even;
    if (lens && c.B > 1) {                           // the same float arithmetic in every workgroup: all agree on every sequence's splits
      total = 0.f;
      if (out.inv_ragged == out.inv_even) {
        for (int i = threadIdx.x & 63; i < c.B; i += 64) total += (float)clamp_len(lens[i]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) total += __shfl_xor(total, o);
      } else {
        float longest = 0.f;
        for (int i = threadIdx.x & 63; i < c.B; i += 64) {
          const float n_i = (float)clamp_len(lens[i]);
          total += n_i;
          longest = fmaxf(longest, n_i);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
          total += __shfl_xor(total, o);
          longest = fmaxf(longest, __shfl_xor(longest, o));
        }
        if (longest * (float)c.B * 16.f > total * 17.f) inv = out.inv_ragged;   // equal: the longest is within a sixteenth of the mean
      }
    }
    const float share = fmaxf(total * (float)c.Hkv * inv, (float)GRAIN);
    n = (unsigned)__builtin_amdgcn_readfirstlane((int)ceilf((float)len / share - 0.1f));
    n = n < 1 ? 1 : n > (unsigned)out.splits ? (unsigned)out.splits : n;
  }
  SplitRows r;
  const unsigned rows = ((len + n * GRAIN - 1) / (n * GRAIN)) * GRAIN;          // even shares of this sequence
  r.splits = rows ? (int)((len + rows - 1) / rows) : 0;
  r.lo = (int64_t)sp * rows;
  r.hi = r.lo + rows < len ? r.lo + rows : len;
  r.total = total;
  return r;
}

// Device-coherent accesses (they bypass the per-XCD L2s).
__device__ __forceinline__ void put_f32(float* p, float x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ unsigned long long get_u64(const void* p) {
  return __hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_u64(void* p, unsigned long long x) {
  __hip_atomic_store((unsigned long long*)p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The merge of S <= N published splits: o = sum_s 2^(m_s - M) o_s / sum_s 2^(m_s - M) l_s. Each thread owns a head's pair
// of dims and takes the splits' maxima and sums along with its part of their vectors: one trip to memory, no exchange
// between threads. Order and assignment are fixed: results are bit-reproducible whoever merges.
template <int N>
__device__ __forceinline__ void merge_splits(const SplitOut& out, int G, size_t head0, int S) {
  constexpr int kD = 128;
  const size_t stride = partial_stride(kD), per_head = out.splits * stride;
  for (int t = threadIdx.x; t < G * (kD / 2); t += 256) {
    const int h = t / (kD / 2), e = (t % (kD / 2)) * 2;
    const float* const p = out.ws + (head0 + h) * per_head;
    unsigned long long ml[N], x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int s = i < S ? i : S - 1;
      ml[i] = get_u64(p + s * stride + kD);
      x[i] = get_u64(p + s * stride + e);
    }
    float M = -INFINITY;
#pragma unroll
    for (int i = 0; i < N; ++i) M = fmaxf(M, __uint_as_float((unsigned)ml[i]));
    const float base = M == -INFINITY ? 0.f : M;                                       // empty splits only
    float L = 0.f, a = 0.f, b = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const float f = i < S ? __builtin_amdgcn_exp2f(__uint_as_float((unsigned)ml[i]) - base) : 0.f;
      L = fmaf(f, __uint_as_float((unsigned)(ml[i] >> 32)), L);
      a = fmaf(f, __uint_as_float((unsigned)x[i]), a);
      b = fmaf(f, __uint_as_float((unsigned)(x[i] >> 32)), b);
    }
    const float inv = L > 0.f ? 1.f / L : 0.f;                                         // no visible row -> zeros
    *(unsigned*)(out.o + (head0 + h) * kD + e) = (unsigned)f32_to_bf16(a * inv) | ((unsigned)f32_to_bf16(b * inv) << 16);
  }
}

// 256 threads, head_dim 128. red_o [4][GS][128] and red_ml [4][GS][2] (max in log2 units, sum) hold the wavefronts'
// states in LDS, complete behind a barrier; head0 = first query head of the KV head, in rows of o.
template <int GS>
__device__ __forceinline__ void finish_split(const SplitOut& out, float (*red_o)[GS][128], float (*red_ml)[GS][2], int G, size_t head0, int sp,
                                             int S) {
  constexpr int kD = 128;
  const size_t stride = partial_stride(kD);
  const size_t per_head = out.splits * stride;
  const bool whole = out.tag ? S <= 1 : out.splits <= 1;     // a single split is the whole answer
  for (int t = threadIdx.x; t < G * kD; t += 256) {
    const int h = t / kD, e = t % kD;
    const float M = fmaxf(fmaxf(red_ml[0][h][0], red_ml[1][h][0]), fmaxf(red_ml[2][h][0], red_ml[3][h][0]));
    float l = 0.f, o = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float f = __builtin_amdgcn_exp2f(red_ml[w][h][0] - M);
      l = fmaf(f, red_ml[w][h][1], l);
      o = fmaf(f, red_o[w][h][e], o);
    }
    if (whole) {
      out.o[(head0 + h) * kD + e] = f32_to_bf16(l > 0.f ? o / l : 0.f);
      continue;
    }
    float* p = out.ws + (head0 + h) * per_head + sp * stride;
    if (!out.tag) {
      p[e] = o;
      if (e == 0) {
        p[kD] = l > 0.f ? M * kLn2 : -INFINITY;    // the merge launch works with natural exponents
        p[kD + 1] = l;
      }
      continue;
    }
    put_f32(p + e, o);
    if (e == 0) {
      put_f32(p + kD, l > 0.f ? M : -INFINITY);
      put_f32(p + kD + 1, l);
    }
  }
  if (whole || !out.tag) return;
  wait_stores();                                   // this wavefront's part is visible to the whole device
  __syncthreads();                                 // ... and everyone else's
  float* const tags = out.ws + head0 * per_head + kD + 2;                  // split s: tags + s * stride
  int seen = 1;
  if (threadIdx.x < 64) {
    if (threadIdx.x == 0) put_u64(tags + sp * stride, out.tag);
    wait_stores();
    if (threadIdx.x < S) seen = get_u64(tags + threadIdx.x * stride) == out.tag;
  }
  if (!__syncthreads_and(seen)) return;            // uniform over the workgroup

  if (S <= 4) merge_splits<4>(out, G, head0, S);
  else if (S <= 8) merge_splits<8>(out, G, head0, S);
  else merge_splits<kMeetSplits>(out, G, head0, S);
  if (threadIdx.x < S) put_u64(tags + threadIdx.x * stride, 0ull);
}

}  // namespace yoco
