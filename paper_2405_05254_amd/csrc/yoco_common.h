// Shared declarations of libyoco's translation units (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "yoco.h"

namespace yoco {

typedef unsigned short bf16_t;  // raw bfloat16 bits

__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// Round to nearest even; NaN stays NaN (quiet).
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x40);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  static __device__ __forceinline__ float load(const float* p) { return *p; }
  static __device__ __forceinline__ void store(float* p, float x) { *p = x; }
};
template <> struct Elem<bf16_t> {
  static __device__ __forceinline__ float load(const bf16_t* p) { return bf16_to_f32(*p); }
  static __device__ __forceinline__ void store(bf16_t* p, float x) { *p = f32_to_bf16(x); }
};

// Addressing of one attention problem family. Strides are in elements.
struct AttnView {
  const void* q;   // [.., Tq, Hq, d]
  const void* k;
  const void* v;
  void* o;         // [.., Tq, Hq, d]
  int64_t q_stride_b, q_stride_t;          // o uses the same strides
  int64_t kv_stride_b, kv_stride_h, kv_stride_n;
  int64_t Tq;       // query rows per sequence
  int64_t q_pos0;   // absolute position of query row 0
  int64_t window;   // keys visible per row (>= 1); INT64_MAX/2 = unbounded
  int Hq, Hkv, d, B;
  float scale;
};

// One gated-retention problem (section 3.1). q, k: [B,T,H,dk]; v, o: [B,T,H,dv];
// log_gamma: [B,T,H] fp32, the natural log of the decays; states: [B,H,dv,dk]
// fp32 (the transpose of S = K^T V), either may be null; gate: like v, may be null.
struct GretView {
  const void* q;
  const void* k;
  const void* v;
  void* o;
  const float* log_gamma;
  const void* gate;          // [B,T,H,dv] or null: the output is multiplied by swish(gate) (Eq. 7)
  const float* state_in;
  float* state_out;
  int64_t T;
  int B, H, dk, dv;
  float scale, eps;
  int group_norm;
};

int compute_units();      // CUs of the device that is current at the first call (a partition has a part of the chip's 256)

// Launchers (each returns the hipError_t of its launch).
hipError_t launch_attn_generic(const AttnView& a, int dtype, hipStream_t s);
// fp32 arithmetic on the matrix cores, head_dim 64 or 128 (attn_f32.hip).
bool attn_f32_supported(const AttnView& a);
hipError_t launch_attn_f32(const AttnView& a, int dtype, hipStream_t s);
hipError_t launch_decode_generic(const yoco_kv_cache& c, const void* q, const int64_t* lens, int64_t fixed_len, int Hq,
                                 float scale, float* ws, int splits, hipStream_t s);
hipError_t launch_decode_merge(const float* ws, void* o, int B, int Hq, int d, int splits, int dtype,
                               hipStream_t s);
hipError_t launch_kv_write(const yoco_kv_cache& c, const void* k, const void* v, const float* row_scale, int b, int64_t pos0, int64_t r0,
                           int64_t n, int src_dtype, hipStream_t s);
hipError_t launch_kv_append(const yoco_kv_cache& c, const void* k, const void* v, const int64_t* pos, int64_t bias, int ring,
                            int src_dtype, hipStream_t s);   // slot = pos[b] + bias; pos null: bias, of every sequence

bool gret_recurrent_supported(const GretView& a);
hipError_t launch_gret_recurrent(const GretView& a, int dtype, hipStream_t s);
hipError_t launch_fill_zero(float* p, size_t n, hipStream_t s);
// Chunkwise form on the matrix cores (bf16, dk = dv = 128).
bool gret_chunk_supported(int B, int64_t T, int H, int dk, int dv, int chunk, int dtype);
size_t gret_chunk_workspace(int B, int64_t T, int H, int chunk);
hipError_t launch_gret_chunk(const GretView& a, int chunk, void* workspace, hipStream_t s);

// bf16, d = 128 fast paths. `supported` functions are host-side predicates.
bool swa_mfma_supported(const AttnView& a, int dtype);
// workspace (or null): where it holds the partial results, the key tiles of few query tiles are shared out over several
// workgroups; swa_mfma_workspace says how much such a call makes use of (0: none).
size_t swa_mfma_workspace(const AttnView& a);
hipError_t launch_swa_mfma(const AttnView& a, void* workspace, size_t workspace_bytes, hipStream_t s);
bool decode_bf16_supported(const yoco_kv_cache& c, int Hq);
// Weights that a decode launch reads ahead for the next launches (decode_tail.h), beside its own work: of up to two matrices, piece
// i (a multiple of 16 bytes; with halves == 2 also the one to_second bytes on) is what workgroup i of the launch that uses it reads.
struct ReadAhead {
  struct { const void* from; int64_t to_second; int bytes, pieces, halves; } part[2];
  int workgroups;               // 0: none
};
// Where one decode launch also merges its splits (decode_tail.h): a wavefront reads all splits of its G / 4 heads, one head
// after another, so up to 16 splits of 4 heads per KV head, or 8 of 8 (in the launch against a merge launch, us: 3 splits of 4 heads, 8 bits, 7.3 and 9.4; 4 x 3 19.3 and 20.2; 8 x 2 15.3 and 16.0; 16 x 3 6.7
// and 7.2; 32 x 3 7.7 and 6.9; 32 x 4 7.9 and 6.8; 16 x 8 9.9 and 7.5), and a launch less on the host, 2.4 us.
constexpr int kMeetSplits = 16;
// Sequences from which on a batch of ragged lengths is shared out finer: each sequence's last split is rounded up, so that the
// splits that are too many for the CUs are about half as many as the sequences.
constexpr int kManySequences = 4;
inline bool decode_meets_in_launch(int G, int splits) { return splits <= 1 || (G <= 8 && (G + 3) / 4 * splits <= kMeetSplits); }
// Both decode launches leave the merged output in o when `tag` is not 0, else partial results for launch_decode_merge.
// k_new / v_new ([B,Hkv,128] bf16, or null): also store and attend to the new token's row at slot lens[b] - 1.
hipError_t launch_decode_bf16(const yoco_kv_cache& c, const void* q, const int64_t* lens, int64_t fixed_len, int Hq, float scale,
                              float* ws, int splits, float inv_ragged, float inv_even, int even, int split, int places, unsigned long long tag, void* o, const void* k_new, const void* v_new, int ring,
                              const ReadAhead& ahead, hipStream_t s);

// 8-bit global cache (cache_i8.hip), head_dim 128: a plane per (sequence, KV head) is a run of 64-row blocks, each
// 8192 code bytes followed by the rows' 64 fp32 scales in row order. Byte offsets of (block row rho, dim e) inside a block:
constexpr int kI8BlockRows = 64;
constexpr int kI8ScaleOffset = 64 * 128;                 // bytes from the start of a block to its scales
constexpr int kI8BlockBytes = kI8ScaleOffset + 64 * 4;   // 8448 = 33 * 256
__host__ __device__ inline int64_t i8_plane_bytes(int64_t N_cap) { return ((N_cap + 63) / 64) * kI8BlockBytes; }
__host__ __device__ inline int i8_k_offset(int rho, int e) {      // K plane: signed code bytes
  return (((((rho >> 2) & 3) * 2 + (e >> 6)) * 64) + ((e >> 4) & 3) * 16 + 4 * (rho >> 4) + (rho & 3)) * 16 + (e & 15);
}
__host__ __device__ inline int i8_v_offset(int rho, int e) {      // V plane: bytes code + 128, transposed
  return (((e >> 4) * 64) + (rho >> 4) * 16 + (e & 15)) * 16 + (rho & 15);
}
// Rows of workgroups that `wanted` more of them take in a grid of c.Hkv x c.B, a multiple of the 8 XCDs in all.
inline unsigned more_rows(const yoco_kv_cache& c, int wanted) {
  const int64_t row = (int64_t)c.Hkv * c.B;
  const int64_t unit = row % 8 == 0 ? 1 : row % 4 == 0 ? 2 : row % 2 == 0 ? 4 : 8;
  return (unsigned)((wanted + row * unit - 1) / (row * unit) * unit);
}
// The other last parameter of the decode kernels: where the lengths make it worth it, the first `split` pairs of sequence and KV head, as many
// as there are more of them than CUs, are cut into `splits` parts each, and the others are whole. The grid has rows for that behind the
// batch's own. A CU's second pair is the same head of the sequence `apart` or, where a CU's two are of other heads, `apart_most` further on.
struct SplitFirst {
  int split, apart, apart_most;
};
inline SplitFirst split_first(const yoco_kv_cache& c, int split) {
  const int cus = c.B * c.Hkv - split;
  return {split, cus / c.Hkv, (cus + c.Hkv - 1) / c.Hkv};
}
inline dim3 decode_grid(const yoco_kv_cache& c, int splits, int split, const ReadAhead& ahead) {
  if (split) return dim3(c.Hkv, c.B + (unsigned)((split * (splits - 1) + c.Hkv - 1) / c.Hkv));
  return dim3(c.Hkv, c.B, splits + more_rows(c, ahead.workgroups));
}
bool cache_i8_supported(int d);
bool decode_i8_supported(const yoco_kv_cache& c, int Hq);
// pos == null: rows [n,Hkv,128] of sequence b to slots pos0 ..; pos != null: one row per sequence to slot pos[b].
// row_scale (or null): float32 [n], every source row is multiplied by its entry (in float32) before it is coded.
hipError_t launch_kv_code_i8(const yoco_kv_cache& c, const void* k, const void* v, const float* row_scale, int b, int64_t pos0, int64_t n,
                             const int64_t* pos, int src_dtype, hipStream_t s);
hipError_t launch_decode_i8(const yoco_kv_cache& c, const void* q, const int64_t* lens, int64_t fixed_len, int Hq, float scale,
                            float* ws, int splits, float inv_ragged, float inv_even, int even, int split, int places, unsigned long long tag, void* o, const ReadAhead& ahead, hipStream_t s);   // q, o bf16

// What stands between the attention calls of a whole bf16 stack (stack_glue.hip). One token: out = W x with W [N][K], the
// input normalised first when gain != null; res: added behind the product; glu: W is [2 N][K] and output n is
// swish(row n) * (row N + n); outputs from n_plain on are log-decays of gated retention, fp32 into log_gamma.
struct GemvArgs {
  const void* x;
  const void* gain;
  const void* W;
  const void* res;
  void* out;
  float* log_gamma;
  int N, K, n_plain, glu;
  float eps, inv_tau;
};
// Two matrices over the same input in one launch: the second is W2 [N2][K] behind a norm of its own (gain2), into out2; the
// first one's outputs are a cache row's K heads and V heads of 128, head i at k_row (v_row) + i * head_stride, or go to out
// where k_row is null. No res, no glu, no log-decays.
struct GemvPair : GemvArgs {
  const void* gain2;
  const void* W2;
  void* out2;
  int N2;
  void *k_row, *v_row;
  int64_t head_stride;
};
constexpr int kGemvMaxK = 16384;      // the input row is held in LDS
hipError_t launch_gemv(const GemvArgs& g, hipStream_t s);
hipError_t launch_gemv_pair(const GemvPair& g, hipStream_t s);
// xn = RMSNorm(x + add) * gain row by row (x + add is stored in y; add == null: no addition, y unused)
hipError_t launch_norm_rows(const void* x, const void* add, void* y, const void* gain, void* xn, int64_t rows, int dim, float eps, hipStream_t s);
hipError_t launch_glu_rows(const void* gu, void* h, int64_t rows, int ffn, hipStream_t s);

// Measured-ceiling microbenchmarks (ceilings.hip).
hipError_t launch_mfma_ceiling(const void* seed, void* sink, int iters, int workgroups, hipStream_t s);
hipError_t launch_attn_loop_ceiling(const void* seed, void* sink, int iters, int workgroups, int mode, hipStream_t s);
hipError_t launch_stream_read(const void* buf, size_t bytes, void* sink, int workgroups, hipStream_t s);

// Partial result of one split, per (b, h, split): o[0..d), then the running max m (log2 units in the fused decodes, whose
// tag follows the sum; natural in the generic kernels) and the sum l, padded so every row starts 16-byte aligned.
__host__ __device__ inline size_t partial_stride(int d) { return (size_t)d + 4; }

}  // namespace yoco
