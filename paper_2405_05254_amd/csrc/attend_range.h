// One wavefront's attention over a range of keys on the vector ALU: the whole of the generic kernels, and how the fp32
// matrix-core kernel redoes a row that came out infinite or NaN.
#pragma once
#include "lanes.h"
#include "yoco_common.h"

namespace yoco {

// LDS traffic of one wave is ordered by the hardware; this keeps the compiler
// from moving a lane's read above another lane's write.
__device__ __forceinline__ void lds_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ float wave_max(float x) { return over64<LaneMax>(x); }
__device__ __forceinline__ float wave_sum(float x) { return over64<LaneSum>(x); }

// Online softmax state of one wave over keys [j_lo, j_hi] of one KV head.
// q_s: this wave's query in LDS (fp32, d entries). p_s: 64 floats of LDS.
// On return (m, l) are the running max / sum and acc[t] holds dimension
// lane + 64 t of the unnormalised output.
template <typename T>
__device__ __forceinline__ void attend_range(const T* __restrict__ kbase, const T* __restrict__ vbase,
                                             int64_t stride_n, int64_t j_lo, int64_t j_hi, int d, float scale,
                                             const float* q_s, float* p_s, float& m, float& l, float acc[4]) {
  const int lane = threadIdx.x & 63;
  for (int64_t c0 = j_lo; c0 <= j_hi; c0 += 64) {
    const int64_t j = c0 + lane;
    const bool valid = j <= j_hi;
    float s = -INFINITY;
    if (valid) {
      const T* kr = kbase + j * stride_n;
      float dot = 0.f;
      for (int e = 0; e < d; ++e) dot = fmaf(q_s[e], Elem<T>::load(kr + e), dot);
      s = dot * scale;
    }
    const float m_new = fmaxf(m, wave_max(s));       // finite: key c0 is valid
    const float alpha = __expf(m - m_new);            // m = -inf on the first chunk -> 0
    const float p = valid ? __expf(s - m_new) : 0.f;
    l = l * alpha + wave_sum(p);
    m = m_new;
    p_s[lane] = p;
    lds_wave_sync();
    const int n = (int)((j_hi - c0 + 1 < 64) ? (j_hi - c0 + 1) : 64);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int e = lane + 64 * t;
      if (e < d) {
        float a = acc[t] * alpha;
        const T* vr = vbase + c0 * stride_n + e;
        for (int jj = 0; jj < n; ++jj) a = fmaf(p_s[jj], Elem<T>::load(vr + jj * stride_n), a);
        acc[t] = a;
      }
    }
    lds_wave_sync();
  }
}

}  // namespace yoco
