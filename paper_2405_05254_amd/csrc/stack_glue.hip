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

// ---- y = W x for one row x. W is [N][K] (a row per output), so a wavefront owns ROWS outputs and its lanes run along
// K with 128-bit loads. GLU: output n takes rows n and N + n (the two halves of W): swish(first) * second.
// Args: GemvArgs, or GemvPair for two matrices, the second's workgroups behind the first's (N is a multiple of a workgroup's
// outputs).
enum Epilogue { kPlain, kResidual, kGlu };

// The rows of W that a wavefront takes; `g` becomes the matrix that its workgroup belongs to.
template <int ROWS, Epilogue EPI, typename Args>
struct OwnRows {
  static constexpr bool kPair = std::is_same<Args, GemvPair>::value;
  static constexpr int NR = EPI == kGlu ? 2 * ROWS : ROWS;
  const bf16_t* w[NR];
  int row0;
  bool second;
  __device__ __forceinline__ explicit OwnRows(Args& g) {
    row0 = (blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * ROWS;
    second = false;
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
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      int row = row0 + (EPI == kGlu ? r >> 1 : r);
      row = row < g.N ? row : g.N - 1;                                       // surplus rows repeat the last one, nothing is stored
      if (EPI == kGlu && (r & 1)) row += g.N;
      w[r] = (const bf16_t*)g.W + (int64_t)row * g.K;
    }
  }
  // Stores the outputs; acc: the rows' products, summed over the wavefront here. res: of this lane's output, where one is added.
  __device__ __forceinline__ void store(const Args& g, float (&acc)[NR], float res) const {
    const int lane = threadIdx.x & 63;
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
        out[n] = f32_to_bf16(round_bf16(acc[r]) + res);
      } else if (n >= g.n_plain) {                                           // ln(gamma) of Eq. 4: logsigmoid(x W_gamma) / tau, fp32
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
  __device__ __forceinline__ float residual(const Args& g) const {
    const int lane = threadIdx.x & 63;
    return EPI == kResidual && lane < ROWS && row0 + lane < g.N ? bf16_to_f32(((const bf16_t*)g.res)[row0 + lane]) : 0.f;
  }
};

__device__ __forceinline__ float square(const u32x4& v, float ss) {
#pragma unroll
  for (int i = 0; i < 4; ++i) ss = fmaf(lo_f(v[i]), lo_f(v[i]), fmaf(hi_f(v[i]), hi_f(v[i]), ss));
  return ss;
}
__device__ __forceinline__ u32x4 normed(const u32x4& v, float rstd, const u32x4& gain) {
  u32x4 y;
#pragma unroll
  for (int i = 0; i < 4; ++i) y[i] = pack_bf16(lo_f(v[i]) * rstd * lo_f(gain[i]), hi_f(v[i]) * rstd * hi_f(gain[i]));
  return y;
}
__device__ __forceinline__ float dot(const u32x4& w, const u32x4& x, float acc) {
#pragma unroll
  for (int i = 0; i < 4; ++i) acc = dot2(w[i], x[i], acc);
  return acc;
}

// 16 bytes of a row in memory that every lane reads from, zeros behind its end; AUX: cache policy of the load.
constexpr int kNontemporal = 2;
template <int AUX>
__device__ __forceinline__ u32x4 row_load(const void* row, unsigned bytes, int at) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)row, 0, bytes, 0x00027000);
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, at, 0, AUX));
}

// Rows of up to CH * 512 elements: every wavefront holds the input row itself, a lane the 8 CH elements that its weights
// meet, and norms it itself. With the row in LDS (below) the workgroup's wavefronts wait for one another twice between the first
// load and the first product, in a launch that is over in a few microseconds. The input is requested before the weights (loads
// return in order), all of them at once: behind a norm the compiler has to be told, or it requests the weights when the norm is
// formed, in two thirds of the registers (a token, 4 + 4 layers of 2048: 274.1 us, 268.2 told; of 1024, two loads a row,
// 165.1 and 165.6, so not there). The sum of the norm is taken in the order of a workgroup's four wavefronts (block_total), so
// that a row has the same norm here as in norm_rows_kernel, bit for bit: as a token and as a row of a prompt.
template <int CH, int ROWS, bool NORM, Epilogue EPI, typename Args>
__global__ void __launch_bounds__(256) gemv_short_kernel(Args g) {
  const OwnRows<ROWS, EPI, Args> own(g);
  constexpr int NR = OwnRows<ROWS, EPI, Args>::NR;
  const int at = (threadIdx.x & 63) * 16;
  const unsigned bytes = (unsigned)g.K * 2u;
  u32x4 x[CH], gain[NORM ? CH : 1], w[NR][CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) x[c] = row_load<0>(g.x, bytes, at + c * 1024);
  if (NORM)
#pragma unroll
    for (int c = 0; c < CH; ++c) gain[c] = row_load<0>(g.gain, bytes, at + c * 1024);
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int c = 0; c < CH; ++c) w[r][c] = row_load<kNontemporal>(own.w[r], bytes, at + c * 1024);
  const float res = own.residual(g);
  if constexpr (NORM && CH > 2) __builtin_amdgcn_sched_barrier(0);
  if constexpr (NORM) {
    float part[CH];                                // of 512 elements, a wavefront's share of block_total
#pragma unroll
    for (int c = 0; c < CH; ++c) part[c] = square(x[c], 0.f);
    const float rstd = rsqrtf(sum_over64(part) / (float)g.K + g.eps);
#pragma unroll
    for (int c = 0; c < CH; ++c) x[c] = normed(x[c], rstd, gain[c]);
  }
  float acc[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    acc[r] = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c) acc[r] = dot(w[r][c], x[c], acc[r]);
  }
  own.store(g, acc, res);
}

constexpr int kStep = 2048;                       // elements of K per trip: 4 loads of 16 bytes per lane and row

// Longer rows: the input row lies in LDS, and the weights come in trips, the next one in flight.
template <int ROWS, bool NORM, Epilogue EPI, typename Args>
__global__ void __launch_bounds__(256) gemv_kernel(Args g) {
  constexpr int NR = OwnRows<ROWS, EPI, Args>::NR;
  extern __shared__ __attribute__((aligned(16))) unsigned char x_lds[];      // the input row (normalised), bf16
  __shared__ float red[4];
  const int tid = threadIdx.x, lane = tid & 63;
  const OwnRows<ROWS, EPI, Args> own(g);
  u32x4 w[NR][4];
  auto load = [&](int k0) {
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int k = k0 + c * 512 + lane * 8;
        w[r][c] = u32x4{0, 0, 0, 0};
        if (k < g.K) w[r][c] = __builtin_nontemporal_load((const u32x4*)(own.w[r] + k));
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

  float rstd = 0.f;
  if (NORM) {
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < kKeep; ++i) ss = square(xv[i], ss);
    for (int p = tid + kKeep * 256; p < pieces; p += 256) ss = square(xp[p], ss);
    rstd = rsqrtf(block_total(ss, red) / (float)g.K + g.eps);
  }
  auto put = [&](int p, const u32x4& v, const u32x4& gn) { ((u32x4*)x_lds)[p] = NORM ? normed(v, rstd, gn) : v; };
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
        for (int r = 0; r < NR; ++r) acc[r] = dot(cur[r][c], x, acc[r]);
      }
    }
  }
  own.store(g, acc, own.residual(g));
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

template <int CH, int ROWS, bool NORM, Epilogue EPI, typename Args>
hipError_t launch_short(const Args& g, dim3 grid, hipStream_t s) {
  hipLaunchKernelGGL((gemv_short_kernel<CH, ROWS, NORM, EPI, Args>), grid, dim3(256), 0, s, g);
  return hipGetLastError();
}
// SHORT_ROWS, ROWS: outputs per wavefront where the input row is held in registers, and where it lies in LDS. Held in registers up
// to 2048 elements behind a norm and up to 6144 without one. us a launch inside token steps of 4 + 4 layers (median of the kernel's own
// time; every weight comes from HBM or from what attention's launch has read ahead), in LDS before and now: W_O 2048 x 2048 4.2 and
// 2.6, W_2 2048 x 5632 6.2 and 5.9, SwiGLU 2 x 5632 x 2048 10.4 and 8.8, 6144 x 2048 behind a norm 6.7 and 6.3, 2048 x 2048 4.3 and 4.0;
// of 1024-wide layers 3.2 and 2.2, 4.4 and 3.3, 5.3 and 3.4, 4.1 and 3.8, 3.4 and 3.0. Over 131072 rows, where nothing is read ahead,
// W_O and W_2 together 11.4 and 11.0, SwiGLU 9.7 and 9.0, 2048 x 2048 behind a norm 4.6 either way. Beyond, without a norm 2048 x 8192 is as good
// either way; behind one rows of 2176 and 2560 would gain in registers too (a token, 3 + 3 layers: 246 us and 233, 275 and 263), 2816
// little and 3072 nothing (306 and 302.5, 339 and 338).
template <int SHORT_ROWS, int ROWS, bool NORM, Epilogue EPI, typename Args>
hipError_t launch(const Args& g, int rows, hipStream_t s) {
  const dim3 grid((unsigned)((rows + 4 * SHORT_ROWS - 1) / (4 * SHORT_ROWS)));
  if (g.K <= 1024) return launch_short<2, SHORT_ROWS, NORM, EPI>(g, grid, s);
  if (g.K <= 2048) return launch_short<4, SHORT_ROWS, NORM, EPI>(g, grid, s);
  if constexpr (!NORM) {
    if (g.K <= 3072) return launch_short<6, SHORT_ROWS, NORM, EPI>(g, grid, s);
    if (g.K <= 6144) return launch_short<12, SHORT_ROWS, NORM, EPI>(g, grid, s);
  }
  hipLaunchKernelGGL((gemv_kernel<ROWS, NORM, EPI, Args>), dim3((unsigned)((rows + 4 * ROWS - 1) / (4 * ROWS))), dim3(256), (unsigned)g.K * 2u, s, g);
  return hipGetLastError();
}

}  // namespace

// One output per wavefront where something is added or gated, else two where the row is short or the classifier's outputs are tens
// of workgroups per CU anyway. us a token, 4 + 4 layers of 2048 and of 1024: 266.7 and 164.7; with two where something is added
// 270.5 and 171.2, where it is gated 272.9 and 173.9, with one everywhere 269.2 and 163.8.
hipError_t launch_gemv(const GemvArgs& g, hipStream_t s) {
  if (g.K % 8 || g.K > kGemvMaxK || g.K <= 0 || g.N <= 0) return hipErrorInvalidValue;
  if (g.glu) return launch<1, 1, true, kGlu>(g, g.N, s);
  if (g.res) return launch<1, 1, false, kResidual>(g, g.N, s);
  if (g.N >= 16384) return launch<2, 2, true, kPlain>(g, g.N, s);
  return launch<2, 1, true, kPlain>(g, g.N, s);
}

// A token's row of the global cache and the first cross-decoder layer's queries. At 4 + 4 layers 43 launches of a step
// over a bf16 cache become 41 (one of the two stored the row), 4 us of 303; an 8-bit cache's row is still coded by a launch of
// its own (42).
hipError_t launch_gemv_pair(const GemvPair& g, hipStream_t s) {
  if (g.K % 8 || g.K > kGemvMaxK || g.K <= 0 || g.N <= 0 || g.N % 256 || g.n_plain != g.N || g.N2 <= 0 || g.res || g.glu) return hipErrorInvalidValue;
  return launch<2, 1, true, kPlain>(g, g.N + g.N2, s);
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
