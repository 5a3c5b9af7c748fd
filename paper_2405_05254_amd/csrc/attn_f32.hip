// Attention prefill in fp32 arithmetic on the matrix cores (v_mfma_f32_16x16x4_f32), head_dim 64 or 128: fp32 storage, and
// bf16 storage where the bf16 kernel has no path (head_dim 64, scale <= 0). Serves yoco_swa_prefill and
// yoco_cross_attn_prefill: a query at absolute position p sees keys j with p - C < j <= p.
//
// Bound by the fp32 matrix rate (157 TFLOP/s) for long windows, by latency for the short prompts it mostly meets. So a
// workgroup has few query rows (16, or 32 where that alone gives every CU four workgroups) and its four wavefronts take
// turns at the 16-key tiles, with a merge at the end; and no operand passes through LDS: S^T = K Q^T and O^T = V^T P^T,
// with the dims of a product dealt to the lanes so that a lane's operands are what 128-bit loads of the rows deliver, and
// the scores' accumulator registers are the second product's operand as they stand. K of the next tile is requested
// behind the first product, V behind the second. Measured against one wavefront per query row on the vector ALU, which it
// replaces at these head dims: 512 rows x 4 heads of 64, window 128: 14.1 -> 6.0 us (launch and latency); 2 x 1455 rows x
// 4 heads of 128, window 1024: 650 -> 83 us; 2 x 2048 x 8 heads of 128: 1854 -> 186 us (69 TFLOP/s).
#include "attend_range.h"
#include "yoco_common.h"

namespace yoco {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kKeys = 16;        // keys per tile
constexpr int kWaves = 4;

__device__ __forceinline__ f32x4 load4(const float* p) { return *(const f32x4*)p; }
__device__ __forceinline__ f32x4 load4(const bf16_t* p) {
  const u32x2 w = *(const u32x2*)p;
  return {__uint_as_float(w[0] << 16), __uint_as_float(w[0] & 0xffff0000u), __uint_as_float(w[1] << 16), __uint_as_float(w[1] & 0xffff0000u)};
}
__device__ __forceinline__ void store4(float* p, const f32x4& x) { *(f32x4*)p = x; }
__device__ __forceinline__ void store4(bf16_t* p, const f32x4& x) {
  *(u32x2*)p = {(unsigned)f32_to_bf16(x[0]) | ((unsigned)f32_to_bf16(x[1]) << 16), (unsigned)f32_to_bf16(x[2]) | ((unsigned)f32_to_bf16(x[3]) << 16)};
}
__device__ __forceinline__ bool not_finite(float x) {
  unsigned u = __float_as_uint(x);
  asm("" : "+v"(u));                                  // the compiler is told to expect no NaN from arithmetic
  return (u & 0x7f800000u) == 0x7f800000u;
}
__device__ __forceinline__ float finite_or_zero(float m) { return m == -INFINITY ? 0.f : m; }     // the base of an empty row's exponents

// Lane (n, qg) = (lane % 16, lane / 16). First product, step (i, e): K row n and Q row n, dim 16 i + 4 qg + e. Scores: query n,
// keys 4 qg + i. Second product, step i: V row 4 qg + i, dims 64 g + 4 n + j for output block (g, j); output: query n, dims
// 64 g + 16 qg + 4 r + j in register r of block (g, j).
template <typename T, int D, int QB>
__global__ void __launch_bounds__(64 * kWaves, QB == 1 ? 3 : 2) attn_f32_kernel(AttnView a) {
  constexpr int kRows = 16 * QB, kPieces = D / 16, kGroups = D / 64;
  __shared__ __attribute__((aligned(16))) float red_o[kWaves][kRows][D];
  __shared__ float red_m[kWaves][kRows], red_l[kWaves][kRows];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, qg = lane >> 4;
  const int h = blockIdx.y, b = blockIdx.z, kvh = h / (a.Hq / a.Hkv);
  const int64_t i0 = (int64_t)blockIdx.x * kRows;
  const int64_t last_q = i0 + kRows < a.Tq ? i0 + kRows - 1 : a.Tq - 1;
  const int64_t lo = a.q_pos0 + i0 - a.window + 1 > 0 ? a.q_pos0 + i0 - a.window + 1 : 0, hi = a.q_pos0 + last_q;
  const T* kb = (const T*)a.k + b * a.kv_stride_b + kvh * a.kv_stride_h;
  const T* vb = (const T*)a.v + b * a.kv_stride_b + kvh * a.kv_stride_h;
  const T* qb0 = (const T*)a.q + b * a.q_stride_b + (int64_t)h * D;

  f32x4 kf[kPieces], vf[kKeys / 4][kGroups];
  auto load_k = [&](int64_t j0) {
    int64_t row = j0 + n;
    row = row < hi ? row : hi;                            // rows past the last visible one repeat it (masked)
    const T* p = kb + row * a.kv_stride_n + qg * 4;
#pragma unroll
    for (int i = 0; i < kPieces; ++i) kf[i] = load4(p + 16 * i);
  };
  auto load_v = [&](int64_t j0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int64_t row = j0 + 4 * qg + i;
      row = row < hi ? row : hi;
#pragma unroll
      for (int g = 0; g < kGroups; ++g) vf[i][g] = load4(vb + row * a.kv_stride_n + 64 * g + 4 * n);
    }
  };
  const int64_t first = lo / kKeys * kKeys + wave * kKeys;
  if (first <= hi) {
    load_k(first);
    load_v(first);
  }
  f32x4 qf[QB][kPieces];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    int64_t row = i0 + qb * 16 + n;
    row = row < a.Tq ? row : a.Tq - 1;
#pragma unroll
    for (int i = 0; i < kPieces; ++i) qf[qb][i] = load4(qb0 + row * a.q_stride_t + qg * 4 + 16 * i);
  }

  float m[QB], l[QB];
  f32x4 o[QB][kGroups][4];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    m[qb] = -INFINITY;
    l[qb] = 0.f;
#pragma unroll
    for (int g = 0; g < kGroups; ++g)
#pragma unroll
      for (int j = 0; j < 4; ++j) o[qb][g][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float c = a.scale * kLog2e;
  for (int64_t j0 = first; j0 <= hi; j0 += kWaves * kKeys) {
    f32x4 s[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) s[qb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < kPieces; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) s[qb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i][e], qf[qb][i][e], s[qb], 0, 0, 0);
    const bool more = j0 + kWaves * kKeys <= hi;
    if (more) load_k(j0 + kWaves * kKeys);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const int64_t ahead = a.q_pos0 + i0 + qb * 16 + n - j0 - 4 * qg;      // this lane's query minus its first key
      float mx = m[qb];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s[qb][i] = ahead - i >= 0 && ahead - i < a.window ? s[qb][i] * c : -INFINITY;
        mx = fmaxf(mx, s[qb][i]);
      }
      mx = over_rows<LaneMax>(mx);
      const float base = finite_or_zero(mx), alpha = __builtin_amdgcn_exp2f(m[qb] - base);
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s[qb][i] = __builtin_amdgcn_exp2f(s[qb][i] - base);
        sum += s[qb][i];
      }
      l[qb] = l[qb] * alpha + sum;
      if (__builtin_amdgcn_ballot_w64(mx != m[qb])) {
#pragma unroll
        for (int g = 0; g < kGroups; ++g)
#pragma unroll
          for (int j = 0; j < 4; ++j) o[qb][g][j] *= alpha;
      }
      m[qb] = mx;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int g = 0; g < kGroups; ++g)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) o[qb][g][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[i][g][j], s[qb][i], o[qb][g][j], 0, 0, 0);
    if (more) load_v(j0 + kWaves * kKeys);
  }

#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    l[qb] = over_rows<LaneSum>(l[qb]);
    const int row = qb * 16 + n;
#pragma unroll
    for (int g = 0; g < kGroups; ++g)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        *(f32x4*)&red_o[wave][row][64 * g + 16 * qg + 4 * r] = f32x4{o[qb][g][0][r], o[qb][g][1][r], o[qb][g][2][r], o[qb][g][3][r]};
    if (qg == 0) {
      red_m[wave][row] = m[qb];
      red_l[wave][row] = l[qb];
    }
  }
  __syncthreads();
  T* ob = (T*)a.o + b * a.q_stride_b + (int64_t)h * D;
  bool bad = false;
  for (int t = threadIdx.x; t < kRows * (D / 4); t += 64 * kWaves) {
    const int row = t / (D / 4), e = (t % (D / 4)) * 4;
    if (i0 + row >= a.Tq) continue;
    const float M = finite_or_zero(fmaxf(fmaxf(red_m[0][row], red_m[1][row]), fmaxf(red_m[2][row], red_m[3][row])));
    float L = 0.f;
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float f = __builtin_amdgcn_exp2f(red_m[w][row] - M);
      L = fmaf(f, red_l[w][row], L);
      x += f * *(const f32x4*)&red_o[w][row][e];
    }
    x *= 1.f / L;
    bad |= not_finite(x[0]) | not_finite(x[1]) | not_finite(x[2]) | not_finite(x[3]);
    store4(ob + (i0 + row) * a.q_stride_t + e, x);
  }

  // Keys that a query of these rows does not see were weighed with 0, and 0 * inf is NaN: where anything came out infinite
  // or NaN, the rows are done again over the keys that each of them sees. Q comes from registers: o may be its memory.
  if (!__syncthreads_or(bad)) return;
  float* const q_s = &red_o[wave][0][0];
  float* const p_s = q_s + D;
  for (int row = wave; row < kRows && i0 + row < a.Tq; row += kWaves) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
      if (row == qb * 16 + n) {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) *(f32x4*)(q_s + qg * 4 + 16 * i) = qf[qb][i];
      }
    lds_wave_sync();
    const int64_t pos = a.q_pos0 + i0 + row, j_lo = pos - a.window + 1 > 0 ? pos - a.window + 1 : 0;
    float m1 = -INFINITY, l1 = 0.f, acc[4] = {0.f, 0.f, 0.f, 0.f};
    attend_range<T>(kb, vb, a.kv_stride_n, j_lo, pos, D, a.scale, q_s, p_s, m1, l1, acc);
#pragma unroll
    for (int t = 0; t < D / 64; ++t) Elem<T>::store(ob + (i0 + row) * a.q_stride_t + lane + 64 * t, acc[t] * (1.f / l1));
  }
}

template <typename T, int D>
hipError_t launch(const AttnView& a, hipStream_t s) {
  const int64_t small = (a.Tq + 15) / 16;
  // 32 rows halve what the caches deliver per product (2 x 2048 rows x 8 heads: 186 us against 202); 16 keep more CUs busy
  // on short prompts (2 x 1455 rows x 4 heads: 83 us against 91)
  if (small * a.Hq * a.B >= 1024)
    hipLaunchKernelGGL((attn_f32_kernel<T, D, 2>), dim3((unsigned)((a.Tq + 31) / 32), a.Hq, a.B), dim3(64 * kWaves), 0, s, a);
  else
    hipLaunchKernelGGL((attn_f32_kernel<T, D, 1>), dim3((unsigned)small, a.Hq, a.B), dim3(64 * kWaves), 0, s, a);
  return hipGetLastError();
}

}  // namespace

bool attn_f32_supported(const AttnView& a) { return a.d == 64 || a.d == 128; }

hipError_t launch_attn_f32(const AttnView& a, int dtype, hipStream_t s) {
  if (dtype == YOCO_F32) return a.d == 64 ? launch<float, 64>(a, s) : launch<float, 128>(a, s);
  return a.d == 64 ? launch<bf16_t, 64>(a, s) : launch<bf16_t, 128>(a, s);
}

}  // namespace yoco
