// Gated retention in its recurrent form (section 3.1, Eq. 5):
//   S_n = gamma_n S_{n-1} + K_n^T V_n,   o_n = scale * Q_n S_n,
// optionally followed by the per-head GroupNorm of Eq. 7 (no learned affine)
// and the multiplication by swish(gate) of the same equation.
// fp32 arithmetic on the vector ALU for any storage dtype and head dims up to
// 128. It is the prefill path of every shape the chunkwise MFMA kernels do not
// cover, and the decode step of the self-decoder (one row per sequence, the
// state read and written once: HBM-bound), which at 128 x 128 has a kernel of
// its own further down; the chunk size plays no part here because the
// recurrent and chunkwise forms are the same function.
//
// gret_recurrent_kernel: one workgroup owns one (sequence, head) and keeps the whole state in
// registers, transposed: thread (rr = tid / 32, kk = tid % 32) holds
// S^T[ev][4 kk .. 4 kk + 3] for the rows ev = rr + 8 r. A row of S^T is
// contiguous along the key dimension, so the 32 lanes of a half wavefront
// read and write 512 contiguous bytes, and o[ev] = q . S^T[ev] is a butterfly
// over those 32 lanes: no LDS and no barrier on the path without GroupNorm.
#include "lanes.h"
#include "yoco_common.h"

namespace yoco {

namespace {

constexpr int kMaxDim = 128;
constexpr int kRowsPerThread = kMaxDim / 8;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <typename T> __device__ __forceinline__ f32x4 load4(const T* p);
template <> __device__ __forceinline__ f32x4 load4<float>(const float* p) { return *(const f32x4*)p; }
template <> __device__ __forceinline__ f32x4 load4<bf16_t>(const bf16_t* p) {
  const u32x2 w = *(const u32x2*)p;
  f32x4 r = {__uint_as_float(w[0] << 16), __uint_as_float(w[0] & 0xffff0000u), __uint_as_float(w[1] << 16),
             __uint_as_float(w[1] & 0xffff0000u)};
  return r;
}

__device__ __forceinline__ float half_wave_sum(float x) {      // over the 32 lanes that share tid / 32
  return over32<LaneSum>(x);
}

// Sum of one value per thread over the workgroup; every thread gets the result.
__device__ __forceinline__ float block_sum(float x, float* red) {
  x = over64<LaneSum>(x);
  __syncthreads();                                  // the previous use of red[] is over
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

template <typename T>
__global__ void __launch_bounds__(256) gret_recurrent_kernel(GretView a) {
  __shared__ float red[4];
  const int h = blockIdx.x, b = blockIdx.y;
  const int kk = threadIdx.x & 31, rr = threadIdx.x >> 5;
  const int ek = kk * 4;
  const bool k_on = ek < a.dk;
  const int n_rows = (a.dv - rr + 7) / 8;                 // rows rr, rr + 8, ... below dv

  f32x4 S[kRowsPerThread];
  const size_t st_off = ((size_t)b * a.H + h) * a.dv * a.dk;
#pragma unroll
  for (int r = 0; r < kRowsPerThread; ++r) {
    S[r] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (a.state_in && k_on && r < n_rows) S[r] = *(const f32x4*)(a.state_in + st_off + (size_t)(rr + 8 * r) * a.dk + ek);
  }

  const T* q = (const T*)a.q + ((size_t)b * a.T * a.H + h) * a.dk;
  const T* k = (const T*)a.k + ((size_t)b * a.T * a.H + h) * a.dk;
  const T* v = (const T*)a.v + ((size_t)b * a.T * a.H + h) * a.dv;
  T* o = (T*)a.o + ((size_t)b * a.T * a.H + h) * a.dv;
  const float* g = a.log_gamma + (size_t)b * a.T * a.H + h;
  const float inv_dv = 1.f / (float)a.dv;

  for (int64_t n = 0; n < a.T; ++n) {
    const float gamma = __expf(g[n * a.H]);
    f32x4 kf = {0.f, 0.f, 0.f, 0.f}, qf = kf;
    if (k_on) {
      kf = load4<T>(k + n * a.H * a.dk + ek);
      qf = load4<T>(q + n * a.H * a.dk + ek);
    }
    float out[kRowsPerThread];
    float sum = 0.f;
    const bool store_state = a.state_out && k_on && n == a.T - 1;
#pragma unroll
    for (int r = 0; r < kRowsPerThread; ++r) {
      out[r] = 0.f;
      if (r < n_rows) {
        const float vv = Elem<T>::load(v + n * a.H * a.dv + rr + 8 * r);
        S[r] = gamma * S[r] + kf * vv;
        // the final state leaves row by row, while later rows of a decode step are still arriving
        if (store_state) *(f32x4*)(a.state_out + st_off + (size_t)(rr + 8 * r) * a.dk + ek) = S[r];
        const float part = qf[0] * S[r][0] + qf[1] * S[r][1] + qf[2] * S[r][2] + qf[3] * S[r][3];
        out[r] = a.scale * half_wave_sum(part);
        sum += out[r];
      }
    }
    if (a.group_norm) {
      // every lane of a half wavefront holds the same out[]: count each row once
      const float mean = block_sum(kk == 0 ? sum : 0.f, red) * inv_dv;
      float sq = 0.f;
#pragma unroll
      for (int r = 0; r < kRowsPerThread; ++r)
        if (r < n_rows) sq += (out[r] - mean) * (out[r] - mean);
      const float var = block_sum(kk == 0 ? sq : 0.f, red) * inv_dv;
      const float rstd = rsqrtf(var + a.eps);
#pragma unroll
      for (int r = 0; r < kRowsPerThread; ++r) out[r] = (out[r] - mean) * rstd;
    }
    if (kk == 0) {
      const T* gate = a.gate ? (const T*)a.gate + ((size_t)b * a.T * a.H + h) * a.dv + n * a.H * a.dv : nullptr;
#pragma unroll
      for (int r = 0; r < kRowsPerThread; ++r)
        if (r < n_rows) {
          float y = out[r];
          if (gate) {                                   // swish gate of Eq. 7: y * g * sigmoid(g)
            const float gv = Elem<T>::load(gate + rr + 8 * r);
            y *= gv / (1.f + __expf(-gv));
          }
          Elem<T>::store(o + n * a.H * a.dv + rr + 8 * r, y);
        }
    }
  }

}

// ---- the decode step (T = 1) at dk = dv = 128, state updated in place. Bound by HBM (a state read and written once) and,
// below some hundred units, by latency; so a (sequence, head) gets 16 wavefronts, a thread only four rows
// ev = rr + 32 r of four elements, and the whole state is requested behind the small operands, the gate behind it (ahead
// of it: 158 us at 16 x 24), before anything is computed. A row is stored as soon as it is updated. The four row sums of
// a thread are reduced together (at the first two exchanges a lane keeps half of its rows), after which the eight lanes
// kk / 8 of a half wavefront hold row rr + 32 (kk / 8). Measured against 4 wavefronts of 16 rows a thread, 13 layers:
// 1 x 24 heads 94 -> 59 us, 8 x 24 113 -> 86, 16 x 24 174 -> 155 (4.2 TB/s of 50 MB a layer), 32 x 24 272 -> 248;
// 8 wavefronts of 8 rows 67, 95, 168, 260. With the sums over lanes in registers instead of shuffles (lanes.h) 53, 80 and 150 at 1, 8
// and 16 x 24; with one wavefront finishing the outputs instead of sixteen 47, 74 and 143, 32 x 24 243 -> 240 (torch's in-place
// product of the same states 24.5, 67, 149.5 and 265). States that 60 layers push out of the memory behind the L2s, us a layer: 8 x 24
// 8.02 -> 7.59. Without GroupNorm the barrier and the one wavefront are all there is to it: 5.61 -> 5.52 a layer at 8 x 24 with the
// gate, 1 x 24 3.39 -> 3.44, 8 x 24 5.54 -> 5.47 and 16 x 24 10.68 -> 10.76 without. NT: nontemporal accesses, see launch_step.
constexpr int kStepRows = 4, kStepGroups = 128 / kStepRows;

template <typename T, bool NT>
__global__ void __launch_bounds__(32 * kStepGroups) gret_decode_kernel(GretView a) {
  constexpr int kDim = 128, kR = kStepRows, kSame = 32 / kR;
  __shared__ float outs[kDim];
  const int h = blockIdx.x, b = blockIdx.y;
  const int kk = threadIdx.x & 31, rr = threadIdx.x >> 5;
  const int ek = kk * 4;
  const size_t bh = (size_t)b * a.H + h;
  const T* v = (const T*)a.v + bh * kDim;
  f32x4* st = (f32x4*)(a.state_out + bh * kDim * kDim + (size_t)rr * kDim + ek);
  constexpr int kStride = kStepGroups * kDim / 4;             // from a thread's row to its next one

  const float gamma = __expf(a.log_gamma[bh]);
  const f32x4 kf = load4<T>((const T*)a.k + bh * kDim + ek), qf = load4<T>((const T*)a.q + bh * kDim + ek);
  float vv[kR];
#pragma unroll
  for (int r = 0; r < kR; ++r) vv[r] = Elem<T>::load(v + rr + kStepGroups * r);
  const int ev = rr + kStepGroups * (kk / kSame);             // the row whose output this lane ends up with
  const bool first = kk % kSame == 0;                         // of the lanes that hold the same row
  f32x4 S[kR];
#pragma unroll
  for (int r = 0; r < kR; ++r) S[r] = NT ? __builtin_nontemporal_load(st + r * kStride) : st[r * kStride];
  // Of the rows 2 lane and 2 lane + 1, which the first wavefront finishes; raw and in every wavefront, from V where there is no
  // gate: behind a branch, or converted there, it is waited for at once, and with it everything requested before it.
  struct __attribute__((aligned(2 * sizeof(T)))) Pair { T x[2]; };
  const int lane = threadIdx.x & 63;
  const Pair gate = ((const Pair*)((const T*)(a.gate ? a.gate : a.v) + bh * kDim))[lane];

  float part[kR];
#pragma unroll
  for (int r = 0; r < kR; ++r) {
    S[r] = gamma * S[r] + kf * vv[r];
    if (NT) __builtin_nontemporal_store(S[r], st + r * kStride);
    else st[r * kStride] = S[r];
    part[r] = qf[0] * S[r][0] + qf[1] * S[r][1] + qf[2] * S[r][2] + qf[3] * S[r][3];
  }
  // reduce-scatter over the 32 lanes of the half wavefront: bits 4 and 3 of kk choose a half of the rows each
  static_assert(kR == 4, "two exchanges");
#pragma unroll
  for (int i = 0; i < 2; ++i) {                               // with lane ^ 16: rows i and i + 2, whose odd and even rows of lanes change places
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(part[i]), __float_as_uint(part[i + 2]), false, false);
    part[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  const bool upper = (kk & 8) != 0;
  part[0] = (upper ? part[1] : part[0]) + dpp_mov<0x128>(upper ? part[0] : part[1]);   // row_ror:8, lane ^ 8
  part[0] = over8<LaneSum>(part[0]);
  // One wavefront finishes the 128 outputs: two sums over the workgroup in all sixteen are more instructions than the state takes.
  if (first) outs[ev] = a.scale * part[0];
  __syncthreads();
  if (threadIdx.x >= 64) return;
  float y[2] = {outs[2 * lane], outs[2 * lane + 1]};
  if (a.group_norm) {
    const float mean = over64<LaneSum>(y[0] + y[1]) * (1.f / kDim);
    y[0] -= mean;
    y[1] -= mean;
    const float rstd = rsqrtf(over64<LaneSum>(fmaf(y[0], y[0], y[1] * y[1])) * (1.f / kDim) + a.eps);
    y[0] *= rstd;
    y[1] *= rstd;
  }
  Pair out;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float g = Elem<T>::load(&gate.x[i]);
    if (a.gate) y[i] *= g / (1.f + __expf(-g));               // swish gate of Eq. 7: y * g * sigmoid(g)
    Elem<T>::store(&out.x[i], y[i]);
  }
  ((Pair*)((T*)a.o + bh * kDim))[lane] = out;
}

template <typename T>
void launch_step(const GretView& a, hipStream_t s) {
  // A layer's states are met again at the next token. Up to 16 MB of them, those of 16 layers fit the 256 MB behind the
  // L2s and are left there; more than that is kept from displacing itself. How many layers there are a call does not know,
  // so the line is drawn for 16, where the two sides cross between 16.5 and 18 MB (16 layers: 8 x 24 heads 106 us against
  // 120 nontemporal, 10 x 24 133 against 134, 11 x 24, 16.5 MB, 158 against 172, 12 x 24 182 against 176, 16 x 24 214
  // against 189). Programs of fewer layers would gain past it: of 13, 12 x 24 heads 120 against 142, 14 x 24 154 against 148.
  if ((size_t)a.B * a.H * 128 * 128 * sizeof(float) <= ((size_t)16 << 20))
    hipLaunchKernelGGL((gret_decode_kernel<T, false>), dim3(a.H, a.B), dim3(32 * kStepGroups), 0, s, a);
  else
    hipLaunchKernelGGL((gret_decode_kernel<T, true>), dim3(a.H, a.B), dim3(32 * kStepGroups), 0, s, a);
}

__global__ void __launch_bounds__(256) fill_zero_kernel(float* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0.f;
}

}  // namespace

// A fill kernel, not a memset: a caller may be capturing the stream into a graph.
hipError_t launch_fill_zero(float* p, size_t n, hipStream_t s) {
  size_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

bool gret_recurrent_supported(const GretView& a) {
  return a.dk <= kMaxDim && a.dv <= kMaxDim && a.dk % 4 == 0 && a.B <= 65535;
}

hipError_t launch_gret_recurrent(const GretView& a, int dtype, hipStream_t s) {
  dim3 grid(a.H, a.B), block(256);
  if (a.T == 1 && a.dk == 128 && a.dv == 128 && a.state_in && a.state_in == a.state_out) {   // the decode step
    if (dtype == YOCO_F32) launch_step<float>(a, s);
    else launch_step<bf16_t>(a, s);
    return hipGetLastError();
  }
  if (dtype == YOCO_F32)
    hipLaunchKernelGGL(gret_recurrent_kernel<float>, grid, block, 0, s, a);
  else
    hipLaunchKernelGGL(gret_recurrent_kernel<bf16_t>, grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace yoco
