// What stands between the attention calls of a whole stack (section 2.1, Eq. 1: RMSNorm, the projections, SwiGLU, the
// residual stream), bf16 weights and activations, for one token at a time and row-wise for prompts.
//
// One token: a step is a walk over every weight matrix once, so it is bound by HBM (0.9 GB of weights per token on a
// 4 + 4-layer stack of 2048-wide layers: 0.13 ms at the rate of a streaming read) and, with matrices of 8 to 46 MB,
// by what surrounds each stream: launches, and the latency of the first loads. Hence one launch per matrix with
// everything around it folded in (the norm before, the residual or the SwiGLU product behind), the first weights
// requested before the norm of the input is formed, and enough wavefronts that the whole matrix is in flight at once.
// The roundings are those of the unfused chain: every named intermediate is rounded to bf16 where it used to be stored.
#include <type_traits>

#include "lanes.h"
#include "mfma_util.h"
#include "yoco_common.h"

namespace yoco {

namespace {

__device__ __forceinline__ float dot2(unsigned a, unsigned b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
}
__device__ __forceinline__ float lo_f(unsigned x) { return __uint_as_float(x << 16); }
__device__ __forceinline__ float hi_f(unsigned x) { return __uint_as_float(x & 0xffff0000u); }
__device__ __forceinline__ float round_bf16(float x) { return bf16_to_f32(f32_to_bf16(x)); }

__device__ __forceinline__ float block_total(float x, float* red) {     // 256 threads; red: 4 floats, used once
  x = over64<LaneSum>(x);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}
__device__ __forceinline__ float swish(float g) { return g / (1.f + __expf(-g)); }

// ---- y = W x for one row x. W is [N][K] (a row per output), so a wavefront owns kRows outputs and its lanes run along
// K with 128-bit loads. GLU: output n takes rows n and N + n (the two halves of W): swish(first) * second.
enum Epilogue { kPlain, kResidual, kGlu };
constexpr int kStep = 2048;                       // elements of K per trip: 4 loads of 16 bytes per lane and row

// Args: GemvArgs, or GemvPair for two matrices, the second's workgroups behind the first's (N is a multiple of a workgroup's
// outputs).
template <int ROWS, bool NORM, Epilogue EPI, typename Args>
__global__ void __launch_bounds__(256) gemv_kernel(Args g) {
  constexpr bool kPair = std::is_same<Args, GemvPair>::value;
  constexpr int NR = EPI == kGlu ? 2 * ROWS : ROWS;
  extern __shared__ __attribute__((aligned(16))) unsigned char x_lds[];      // the input row (normalised), bf16
  __shared__ float red[4];
  const int tid = threadIdx.x, lane = tid & 63;
  int row0 = (blockIdx.x * 4 + (tid >> 6)) * ROWS;
  bool second = false;
  if constexpr (kPair) {
    second = (int)blockIdx.x * 4 * ROWS >= g.N;
    if (second) {
      row0 -= g.N;
      g.gain = g.gain2;
      g.W = g.W2;
      g.out = g.out2;
      g.n_plain = g.N = g.N2;
    }
  }
  const bf16_t* wp[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    int row = row0 + (EPI == kGlu ? r >> 1 : r);
    row = row < g.N ? row : g.N - 1;                                         // surplus rows repeat the last one, nothing is stored
    if (EPI == kGlu && (r & 1)) row += g.N;
    wp[r] = (const bf16_t*)g.W + (int64_t)row * g.K;
  }
  u32x4 w[NR][4];
  auto load = [&](int k0) {
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int k = k0 + c * 512 + lane * 8;
        w[r][c] = u32x4{0, 0, 0, 0};
        if (k < g.K) w[r][c] = __builtin_nontemporal_load((const u32x4*)(wp[r] + k));
      }
  };
  // The input row is requested before the weights (loads return in order): its norm is formed while they arrive.
  constexpr int kKeep = NORM ? 2 : 4;                                         // pieces per thread held in registers
  const u32x4* xp = (const u32x4*)g.x;
  const u32x4* gp = (const u32x4*)g.gain;
  const int pieces = g.K >> 3;
  u32x4 xv[kKeep], gv[kKeep];
#pragma unroll
  for (int i = 0; i < kKeep; ++i) {
    xv[i] = gv[i] = u32x4{0, 0, 0, 0};
    if (tid + i * 256 < pieces) {
      xv[i] = xp[tid + i * 256];
      if (NORM) gv[i] = gp[tid + i * 256];
    }
  }
  load(0);

  auto square = [](const u32x4& v, float ss) {
#pragma unroll
    for (int i = 0; i < 4; ++i) ss = fmaf(lo_f(v[i]), lo_f(v[i]), fmaf(hi_f(v[i]), hi_f(v[i]), ss));
    return ss;
  };
  float rstd = 0.f;
  if (NORM) {
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < kKeep; ++i) ss = square(xv[i], ss);
    for (int p = tid + kKeep * 256; p < pieces; p += 256) ss = square(xp[p], ss);
    rstd = rsqrtf(block_total(ss, red) / (float)g.K + g.eps);
  }
  auto put = [&](int p, const u32x4& v, const u32x4& gn) {
    u32x4 y = v;
    if (NORM) {
#pragma unroll
      for (int i = 0; i < 4; ++i) y[i] = pack_bf16(lo_f(v[i]) * rstd * lo_f(gn[i]), hi_f(v[i]) * rstd * hi_f(gn[i]));
    }
    ((u32x4*)x_lds)[p] = y;
  };
#pragma unroll
  for (int i = 0; i < kKeep; ++i)
    if (tid + i * 256 < pieces) put(tid + i * 256, xv[i], gv[i]);
  for (int p = tid + kKeep * 256; p < pieces; p += 256) put(p, xp[p], NORM ? gp[p] : xp[p]);
  __syncthreads();

  float acc[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) acc[r] = 0.f;
  for (int k0 = 0; k0 < g.K; k0 += kStep) {
    u32x4 cur[NR][4];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) cur[r][c] = w[r][c];
    if (k0 + kStep < g.K) load(k0 + kStep);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int p = (k0 >> 3) + c * 64 + lane;
      if (p < pieces) {
        const u32x4 x = ((const u32x4*)x_lds)[p];
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[r] = dot2(cur[r][c][i], x[i], acc[r]);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) acc[r] = over64<LaneSum>(acc[r]);
  bf16_t* out = (bf16_t*)g.out;
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    const int n = row0 + r;
    if (lane != r || n >= g.N) continue;
    if (EPI == kGlu) {
      out[n] = f32_to_bf16(round_bf16(swish(round_bf16(acc[2 * r]))) * round_bf16(acc[2 * r + 1]));
    } else if (EPI == kResidual) {
      out[n] = f32_to_bf16(round_bf16(acc[r]) + bf16_to_f32(((const bf16_t*)g.res)[n]));
    } else if (n >= g.n_plain) {                                             // ln(gamma) of Eq. 4: logsigmoid(x W_gamma) / tau, fp32
      const float a = acc[r];
      g.log_gamma[n - g.n_plain] = (fminf(a, 0.f) - log1pf(__expf(-fabsf(a)))) * g.inv_tau;
    } else {
      bf16_t* to = out + n;
      if constexpr (kPair) {
        const int heads = g.N >> 8, head = n >> 7;
        if (!second && g.k_row) to = (bf16_t*)(head < heads ? g.k_row : g.v_row) + (head < heads ? head : head - heads) * g.head_stride + (n & 127);
      }
      *to = f32_to_bf16(acc[r]);
    }
  }
}

// ---- prompts: the row-wise passes between the matrix products. One workgroup per row.
// y = x (+ add), stored when y != null; xn = RMSNorm(y) * gain
__global__ void __launch_bounds__(256) norm_rows_kernel(const u32x4* __restrict__ x, const u32x4* __restrict__ add, u32x4* __restrict__ y,
                                                        const u32x4* __restrict__ gain, u32x4* __restrict__ xn, int pieces, float eps) {
  __shared__ float red[4];
  const int64_t row = (int64_t)blockIdx.x * pieces;
  constexpr int kKeep = 2;                                   // pieces per thread held in registers: rows up to 4096
  u32x4 keep[kKeep];
  float ss = 0.f;
  int it = 0;
  for (int p = threadIdx.x; p < pieces; p += 256, ++it) {
    u32x4 v = x[row + p];
    if (add) {
      const u32x4 a = add[row + p];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = pack_bf16(lo_f(v[i]) + lo_f(a[i]), hi_f(v[i]) + hi_f(a[i]));
      y[row + p] = v;
    }
    if (it == 0) keep[0] = v;
    if (it == 1) keep[1] = v;
#pragma unroll
    for (int i = 0; i < 4; ++i) ss = fmaf(lo_f(v[i]), lo_f(v[i]), fmaf(hi_f(v[i]), hi_f(v[i]), ss));
  }
  const float rstd = rsqrtf(block_total(ss, red) / (float)(pieces * 8) + eps);
  it = 0;
  for (int p = threadIdx.x; p < pieces; p += 256, ++it) {
    const u32x4 v = it == 0 ? keep[0] : it == 1 ? keep[1] : (add ? y : x)[row + p];   // later pieces: written by this thread above
    const u32x4 gn = gain[p];
    u32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = pack_bf16(lo_f(v[i]) * rstd * lo_f(gn[i]), hi_f(v[i]) * rstd * hi_f(gn[i]));
    xn[row + p] = o;
  }
}

// h = swish(gu[:, :ffn]) * gu[:, ffn:]; gu is [rows][2 ffn]
__global__ void __launch_bounds__(256) glu_rows_kernel(const u32x4* __restrict__ gu, u32x4* __restrict__ h, int pieces, int64_t total) {
  for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
    const int64_t row = idx / pieces;
    const int p = (int)(idx - row * pieces);
    const u32x4 a = gu[row * 2 * pieces + p], b = gu[row * 2 * pieces + pieces + p];
    u32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      o[i] = pack_bf16(round_bf16(swish(lo_f(a[i]))) * lo_f(b[i]), round_bf16(swish(hi_f(a[i]))) * hi_f(b[i]));
    h[idx] = o;
  }
}

template <int ROWS, bool NORM, Epilogue EPI, typename Args>
hipError_t launch(const Args& g, int rows, hipStream_t s) {
  const int per_wg = 4 * ROWS;
  hipLaunchKernelGGL((gemv_kernel<ROWS, NORM, EPI, Args>), dim3((unsigned)((rows + per_wg - 1) / per_wg)), dim3(256), (unsigned)g.K * 2u, s, g);
  return hipGetLastError();
}

}  // namespace

// One output per wavefront (two for the classifier, whose outputs are tens of workgroups per CU anyway): more wavefronts
// with less each measured faster down the line, with 2 / 1 outputs 6.9 / 6.3 us for 2048 x 5632 (23 MB), 4.3 / 4.0 us for
// 2048 x 2048; 6144 x 2048 6.9 us, SwiGLU 2 x 5632 x 2048 (46 MB) 10.5 us, 32000 x 2048 (131 MB) 22.5 us: 3.2 us per
// launch plus the bytes at 6.1 TB/s.
hipError_t launch_gemv(const GemvArgs& g, hipStream_t s) {
  if (g.K % 8 || g.K > kGemvMaxK || g.K <= 0 || g.N <= 0) return hipErrorInvalidValue;
  if (g.glu) return launch<1, true, kGlu>(g, g.N, s);
  if (g.res) return launch<1, false, kResidual>(g, g.N, s);
  if (g.N >= 16384) return launch<2, true, kPlain>(g, g.N, s);
  return launch<1, true, kPlain>(g, g.N, s);
}

// A token's row of the global cache and the first cross-decoder layer's queries. At 4 + 4 layers 43 launches of a step
// over a bf16 cache become 41 (one of the two stored the row), 4 us of 303; an 8-bit cache's row is still coded by a launch of
// its own (42).
hipError_t launch_gemv_pair(const GemvPair& g, hipStream_t s) {
  if (g.K % 8 || g.K > kGemvMaxK || g.K <= 0 || g.N <= 0 || g.N % 256 || g.n_plain != g.N || g.N2 <= 0 || g.res || g.glu) return hipErrorInvalidValue;
  return launch<1, true, kPlain>(g, g.N + g.N2, s);
}

hipError_t launch_norm_rows(const void* x, const void* add, void* y, const void* gain, void* xn, int64_t rows, int dim, float eps, hipStream_t s) {
  hipLaunchKernelGGL(norm_rows_kernel, dim3((unsigned)rows), dim3(256), 0, s, (const u32x4*)x, (const u32x4*)add, (u32x4*)y, (const u32x4*)gain,
                     (u32x4*)xn, dim / 8, eps);
  return hipGetLastError();
}

hipError_t launch_glu_rows(const void* gu, void* h, int64_t rows, int ffn, hipStream_t s) {
  const int64_t total = rows * (ffn / 8);
  int64_t blocks = (total + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(glu_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (const u32x4*)gu, (u32x4*)h, ffn / 8, total);
  return hipGetLastError();
}

}  // namespace yoco
