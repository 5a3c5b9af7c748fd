// Chunkwise gated retention on the matrix cores (section 3.1, Eq. 6; the
// equivalence with Eq. 4 and Eq. 5 is appendix B). bf16, dk = dv = 128.
//
// With G_j the sum of log2(gamma) from the first row of j's chunk up to and
// including j, a chunk of rows that finds the state S before it computes
//   O = scale * ((Q K^T * D) V + (Q S) * 2^(G_j)),   D(j,k) = 2^(G_j - G_k), k <= j
//   S <- 2^(G_last) S + K^T (V * 2^(G_last - G_j))
// The sequence is cut into segments, one or two workgroups' worth per CU over all heads, and a segment into chunks of 64
// rows. The caller's chunk size plays no part, but that it sizes the workspace and with it the most segments there can
// be: another cut is another order of fp32 sums. Launches:
//   1  what a segment adds to the state, for all segments but the last (reads K and V)
//   2  the scan across segments, element-wise and in place: the state before each segment. Up to three earlier segments
//      are folded by launch 3 itself.
//   3  outputs: a workgroup walks its segment with the state in its MFMA accumulators, and hands over the final state.
// Nothing but one state per segment touches memory in between: Q, gate and O move once, K and V twice. Read and written
// at T = 32768 x 24 heads without the gate, by the counters of HBM: 0.45, 0.06 and 0.85 GB in launches 1 to 3, 1.36 in
// all of 0.81 algorithmic (a gate adds 0.2 to both; a form that wrote and read one state per 256-row chunk moved 2.1 GB
// with it). Launch 3 does that at 4 TB/s in 214 us, below the 7.07 of a plain stream: its loads and its ten products per
// chunk where four are asked for do not overlap fully.
//
// Partition: wavefront w owns dims 32 w .. 32 w + 31 of V, of the outputs and of the state, S[128 ek][32 ev] with ev
// along the lanes. A state accumulator is then, rounded to bf16, the A operand of O^T = S^T Q^T as it stands (the rows of
// S are assigned to dims ek so that a lane's eight registers are eight consecutive ones), and the V^T operand of
// O^T += V^T P^T is the B operand of S += K^T V: no operand of either product of the state passes through LDS.
// The scores of a chunk are formed once, a 32 x 32 block per wavefront, and shared through LDS in operand order.
//
// Precision: every operand that is not bf16 by nature (scores times decay, V times decay, the state) is split into a
// bf16 high and low part, 16 significant bits, two products each; accumulation is fp32.
#include "mfma_util.h"
#include "yoco_common.h"

namespace yoco {

namespace {

constexpr int kD = 128;
constexpr int kC = 64;                        // rows per chunk
constexpr int kTileBytes = kC * kD * 2;       // 16 KiB
constexpr int kState = kD * kD;               // elements of one state
constexpr int kMaxChunk = 1024;               // of the caller's chunk size
constexpr int kFold = 3;                      // earlier segments an output workgroup adds up itself
constexpr float kLog2e = 1.4426950408889634f;

typedef float f32x4 __attribute__((ext_vector_type(4)));

struct SegArgs {
  GretView a;
  int n_chunks, per_seg, nseg;   // chunks per sequence and per segment, segments per sequence
  float* state;                  // [B][H][nseg - 1][dv][dk]: what segment s adds; after the scan, the state before segment s + 1
  float* decay;                  // [B][H][nseg - 1]: log2 decay over segment s
  float* init;                   // [B][H][dv][dk]: launch 1's copy of state_in, which launch 3 may overwrite (state_out); null without one
};

__device__ __forceinline__ float lo_f(unsigned x) { return __uint_as_float(x << 16); }
__device__ __forceinline__ float hi_f(unsigned x) { return __uint_as_float(x & 0xffff0000u); }
// (x0, x1) = hi + lo in packed bf16. The remainders are differences, not dot products of hi with (-1, 0) and (0, -1), which are an instruction
// fewer each: those add to the register that holds x, so that a state's x has to be copied first, and what reads them waits.
// Differences of x as it is: where x is a product (weigh, scores times decay) the compiler would make them fused multiply-adds of the unrounded
// product, whose low parts are others.
__device__ __forceinline__ void split_bf16(float x0, float x1, unsigned& hi, unsigned& lo) {
#pragma clang fp contract(off)
  hi = pack_bf16(x0, x1);
  lo = pack_bf16(x0 - lo_f(hi), x1 - hi_f(hi));
}
__device__ __forceinline__ f32x16 mfma(const u32x4& a, const u32x4& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Byte offsets of 16-byte piece c16 of row `row` in a [64][128] bf16 tile: for row-wise operand reads (pieces XOR
// row & 15), and for transposing reads (32-byte pieces XOR row & 7).
__device__ __forceinline__ int row_off(int row, int c16) { return row * 256 + ((c16 ^ (row & 15)) << 4); }
__device__ __forceinline__ int tr_off(int row, int c16) { return row * 256 + (((((c16 >> 1) ^ (row & 7)) << 1) | (c16 & 1)) << 4); }

// Operand of 32 dims x 16 rows from a tile: lane l gets one dim of block blk and, with hf = l / 32, the rows
// 16 t + 4 hf + 0..3, then 16 t + 8 + 4 hf + 0..3. `base` says which dim: in order, or with bits 2 and 3 of the dim exchanged.
__device__ __forceinline__ int tr_base(int lane, bool exchanged) {
  const int s16 = lane & 15, db = (lane >> 4) & 1, z = (lane >> 5) * 4 + (s16 >> 2), p = s16 & 3;
  return z * 256 + ((db ^ z) << 5) + ((exchanged ? ((p & 1) << 1) | (p >> 1) : p) << 3);
}
__device__ __forceinline__ u32x4 tr_frag(const char* tile, int base, int blk, int t) {
  lds_char* p = (lds_char*)tile + (base ^ (blk << 6)) + t * 16 * 256;
  const u32x2 a = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p));
  const u32x2 b = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 8 * 256)));
  return {a[0], a[1], b[0], b[1]};
}

// The V operand of 16 rows (step t) times their weights in LDS, as high and low part.
__device__ __forceinline__ void weigh(const u32x4& vf, const float* w, int t, int hf, u32x4& vh, u32x4& vl) {
  const f32x4 w0 = *(const f32x4*)(w + t * 16 + hf * 4), w1 = *(const f32x4*)(w + t * 16 + 8 + hf * 4);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x4& ww = i < 2 ? w0 : w1;
    unsigned h, l;
    split_bf16(lo_f(vf[i]) * ww[(i & 1) * 2], hi_f(vf[i]) * ww[(i & 1) * 2 + 1], h, l);
    vh[i] = h;
    vl[i] = l;
  }
}
// S += K^T (V * w) for the 16 rows of step t.
__device__ __forceinline__ void add_rows(f32x16 (&S)[4], const char* k_t, int kbase, const u32x4& vh, const u32x4& vl, int t) {
  u32x4 kf[4];
#pragma unroll
  for (int eb = 0; eb < 4; ++eb) kf[eb] = tr_frag(k_t, kbase, eb, t);
#pragma unroll
  for (int eb = 0; eb < 4; ++eb) S[eb] = mfma(kf[eb], vh, S[eb]);
#pragma unroll
  for (int eb = 0; eb < 4; ++eb) S[eb] = mfma(kf[eb], vl, S[eb]);
}

// Workgroup -> (head, segment, sequence). Heads vary fastest, so that workgroups that run together read neighbouring
// 256-byte pieces of the same rows; and the workgroups, dealt to the 8 XCDs round robin, are renumbered so that each XCD
// has a run of them, all heads among it: with one head in eight per XCD, its rows (24 heads apart) fall into 2 of the 16
// channels of its L2, and both passes stop at 4.2 TB/s.
struct Unit {
  int h, sg, b;
};
__device__ __forceinline__ Unit unit_of(int H, int segs) {
  const int total = gridDim.x, bid = blockIdx.x, per = total >> 3, rem = total & 7, xcd = bid & 7;
  const int n = xcd * per + (xcd < rem ? xcd : rem) + (bid >> 3);
  return {n % H, n / H % segs, n / (H * segs)};
}

// Inclusive sum of one value per lane over the wavefront: within rows of 16 lanes, then a row's total into the next one,
// then the lower half's total into the upper half.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ float wave_scan(float x) {
  x = dpp_add<0x111, 0xf>(x);    // row_shr:1
  x = dpp_add<0x112, 0xf>(x);    // row_shr:2
  x = dpp_add<0x114, 0xf>(x);    // row_shr:4
  x = dpp_add<0x118, 0xf>(x);    // row_shr:8
  x = dpp_add<0x142, 0xa>(x);    // row_bcast:15 into rows 1 and 3
  x = dpp_add<0x143, 0xc>(x);    // row_bcast:31 into rows 2 and 3
  return x;
}
__device__ __forceinline__ float lane63(float x) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63)); }

// A state in memory ([ev][ek], fp32) against a wavefront's accumulators: lane (hf, lq) holds ev = 32 wave + lq and, in
// registers 8 u .. 8 u + 7 of block eb, ek = 32 eb + 16 u + 8 hf + 0..7.
template <typename F>
__device__ __forceinline__ void each_piece(int wave, int lane, F f) {
  const int off = (wave * 32 + (lane & 31)) * kD + (lane >> 5) * 8;
#pragma unroll
  for (int eb = 0; eb < 4; ++eb)
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int p = 0; p < 2; ++p) f(eb, u * 8 + p * 4, off + eb * 32 + u * 16 + p * 4);
}
__device__ __forceinline__ void store_state(float* dst, const f32x16 (&S)[4], int wave, int lane) {
  each_piece(wave, lane, [&](int eb, int r, int off) {
    *(f32x4*)(dst + off) = f32x4{S[eb][r], S[eb][r + 1], S[eb][r + 2], S[eb][r + 3]};
  });
}

// ---- launch 1. The segment's chunks are walked from the last to the first, every row weighted by its decay to the end of
// the segment, so the accumulators need no rescaling, and the rows read last are the ones launch 3 starts with.
__global__ void __launch_bounds__(256, 2) gret_segment_kernel(SegArgs g) {
  __shared__ __attribute__((aligned(1024))) char k_t[2][kTileBytes], v_t[2][kTileBytes];
  __shared__ __attribute__((aligned(16))) float w_t[2][kC];
  const GretView& a = g.a;
  const Unit un = unit_of(a.H, g.nseg - 1);
  const int h = un.h, sg = un.sg, b = un.b;
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c_lo = sg * g.per_seg, c_hi = c_lo + g.per_seg;           // never the last segment: all its rows exist
  const int64_t row_bytes = (int64_t)a.H * kD * 2, head0 = ((int64_t)b * a.T * a.H + h) * kD * 2;
  const int c16 = tid & 15, srow = tid >> 4;
  const char* kg = (const char*)a.k + head0;
  const char* vg = (const char*)a.v + head0;
  const float* lg = a.log_gamma + (int64_t)b * a.T * a.H + h;
  const int kbase = tr_base(lane, true), vbase = tr_base(lane, false);
  const int st_off = tr_off(srow, c16);                               // row srow + 16 i is 4096 i further
  uint32_t off[4];                                                    // a thread's pieces from the start of a chunk
#pragma unroll
  for (int i = 0; i < 4; ++i) off[i] = (uint32_t)(srow + 16 * i) * (uint32_t)row_bytes + (uint32_t)(c16 * 16);

  f32x16 S[4];
#pragma unroll
  for (int eb = 0; eb < 4; ++eb)
#pragma unroll
    for (int r = 0; r < 16; ++r) S[eb][r] = 0.f;
  struct Rows { u32x4 k[4], v[4]; float lg; } even, odd;               // two chunks in flight
  float after = 0.f;                                                   // log2 decay of the later chunks (wavefront 0 keeps it)
  auto load = [&](Rows& x, int c) {
    const int64_t r0 = (int64_t)c * kC;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x.k[i] = __builtin_nontemporal_load((const u32x4*)(kg + r0 * row_bytes + off[i]));
      x.v[i] = __builtin_nontemporal_load((const u32x4*)(vg + r0 * row_bytes + off[i]));
    }
    x.lg = wave == 0 ? lg[(r0 + lane) * a.H] : 0.f;
  };
  auto chunk = [&](Rows& x, int c, char* k_d, char* v_d, float* w_d) {
    if (wave == 0) {
      const float G = wave_scan(x.lg * kLog2e), last = lane63(G);
      w_d[lane] = __builtin_amdgcn_exp2f(last - G + after);
      after += last;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      *(u32x4*)(k_d + st_off + i * 4096) = x.k[i];
      *(u32x4*)(v_d + st_off + i * 4096) = x.v[i];
    }
    load(x, c - 2 > c_lo ? c - 2 : c_lo);                              // in flight during the products of two chunks
    __syncthreads();
    u32x4 vh[4], vl[4];
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int t = 0; t < 4; ++t) weigh(tr_frag(v_d, vbase, wave, t), w_d, t, hf, vh[t], vl[t]);
#pragma unroll
    for (int t = 0; t < 4; ++t) add_rows(S, k_d, kbase, vh[t], vl[t], t);
    __builtin_amdgcn_s_setprio(0);
  };
  load(even, c_hi - 1);
  load(odd, c_hi - 2 > c_lo ? c_hi - 2 : c_lo);
  for (int c = c_hi - 1; c >= c_lo; c -= 2) {
    chunk(even, c, k_t[0], v_t[0], w_t[0]);
    if (c - 1 < c_lo) break;
    chunk(odd, c - 1, k_t[1], v_t[1], w_t[1]);
  }
  const int64_t slot = ((int64_t)b * a.H + h) * (g.nseg - 1) + sg;
  store_state(g.state + slot * kState, S, wave, lane);
  if (tid == 0) g.decay[slot] = after;
  if (g.init && sg == 0) {
    const int64_t at = ((int64_t)b * a.H + h) * kState;
    for (int e = tid * 4; e < kState; e += 1024) *(f32x4*)(g.init + at + e) = *(const f32x4*)(a.state_in + at + e);
  }
}

// ---- launch 2: scan over the segments, in place; thread owns 4 consecutive elements of the state. A group of segments is
// loaded together (independent addresses) before the dependent updates run.
__global__ void __launch_bounds__(256) gret_state_scan_kernel(SegArgs g) {
  constexpr int kAhead = 8;
  const int64_t bh = (int64_t)blockIdx.z * g.a.H + blockIdx.y;
  const int e = (blockIdx.x * 256 + threadIdx.x) * 4, n = g.nseg - 1;
  f32x4 R = {0.f, 0.f, 0.f, 0.f};
  if (g.a.state_in) R = *(const f32x4*)(g.a.state_in + bh * kState + e);
  float* st = g.state + bh * n * kState + e;
  for (int s0 = 0; s0 < n; s0 += kAhead) {
    f32x4 U[kAhead];
    float alpha[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const int s = s0 + i < n ? s0 + i : n - 1;
      U[i] = *(const f32x4*)(st + (int64_t)s * kState);
      alpha[i] = __builtin_amdgcn_exp2f(g.decay[bh * n + s]);
    }
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
      if (s0 + i < n) {
        R = U[i] + alpha[i] * R;
        *(f32x4*)(st + (int64_t)(s0 + i) * kState) = R;
      }
  }
}

// ---- launch 3: outputs.
template <bool NORM, bool GATE>
__global__ void __launch_bounds__(256, 2) gret_output_kernel(SegArgs g) {
  __shared__ __attribute__((aligned(1024))) char q_t[kTileBytes], k_t[kTileBytes], v_t[kTileBytes];
  __shared__ __attribute__((aligned(1024))) char p_t[2][kTileBytes / 2];     // scores, high and low parts: [step][hf][query] 16 bytes
  __shared__ __attribute__((aligned(16))) float g_t[kC], w_t[kC];            // G of the chunk's rows, their weights in the state
  __shared__ float red_m[4][kC], red_s[4][kC];                               // GroupNorm: a wavefront's means and sums of squares
  const GretView& a = g.a;
  const Unit un = unit_of(a.H, g.nseg);
  const int h = un.h, sg = un.sg, b = un.b;
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, lq = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t bh = (int64_t)b * a.H + h;
  const int c_lo = sg * g.per_seg, c_hi = c_lo + g.per_seg < g.n_chunks ? c_lo + g.per_seg : g.n_chunks;
  const int64_t row_bytes = (int64_t)a.H * kD * 2, head0 = ((int64_t)b * a.T * a.H + h) * kD * 2;
  const int c16 = tid & 15, srow = tid >> 4;
  const char* qg = (const char*)a.q + head0;
  const char* kg = (const char*)a.k + head0;
  const char* vg = (const char*)a.v + head0;
  const char* gg = (const char*)a.gate + head0;
  char* og = (char*)a.o + head0;
  const float* lg = a.log_gamma + (int64_t)b * a.T * a.H + h;
  const int kbase = tr_base(lane, true), vbase = tr_base(lane, false);
  const int q_off = row_off(srow, c16), kv_off = tr_off(srow, c16);          // row srow + 16 i is 4096 i further

  u32x4 qr[4], kr[4], vr[4], gr[4];
  float lgr = 0.f;
  // a thread's pieces from the start of a chunk; in the chunk that T ends in, rows past the end repeat the last one
  const uint32_t off0 = (uint32_t)srow * (uint32_t)row_bytes + (uint32_t)(c16 * 16);
  const int rows_end = (int)(a.T - (int64_t)(g.n_chunks - 1) * kC);
  auto piece = [&](int i, bool end) {
    const uint32_t o = off0 + (uint32_t)(16 * i) * (uint32_t)row_bytes;
    return end && srow + 16 * i >= rows_end ? (uint32_t)(rows_end - 1) * (uint32_t)row_bytes + (uint32_t)(c16 * 16) : o;
  };
  auto load_qk = [&](int c) {
    const int64_t at = (int64_t)c * kC * row_bytes;
    const bool end = c == g.n_chunks - 1;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t o = piece(i, end);
      qr[i] = *(const u32x4*)(qg + at + o);
      kr[i] = *(const u32x4*)(kg + at + o);
    }
  };
  auto load_v = [&](int c) {
    const int64_t r0 = (int64_t)c * kC;
    const bool end = c == g.n_chunks - 1;
#pragma unroll
    for (int i = 0; i < 4; ++i) vr[i] = *(const u32x4*)(vg + r0 * row_bytes + piece(i, end));
    if (wave == 0) {                                          // not touched here: that would wait for everything in flight
      unsigned row = lane;
      asm volatile("" : "+v"(row));                           // keep what depends on it out of long-lived registers
      row = end && (int)row >= rows_end ? (unsigned)(rows_end - 1) : row;
      lgr = *(const float*)((const char*)(lg + r0 * a.H) + row * (unsigned)a.H * 4u);
    }
  };
  load_qk(c_lo);
  load_v(c_lo);

  // the state before the segment
  f32x16 S[4];
#pragma unroll
  for (int eb = 0; eb < 4; ++eb)
#pragma unroll
    for (int r = 0; r < 16; ++r) S[eb][r] = 0.f;
  auto add_state = [&](const float* src, float alpha) {                      // S = alpha S + src
    each_piece(wave, lane, [&](int eb, int r, int off) {
      const f32x4 x = *(const f32x4*)(src + off);
#pragma unroll
      for (int e = 0; e < 4; ++e) S[eb][r + e] = fmaf(alpha, S[eb][r + e], x[e]);
    });
  };
  const float* before = g.state + bh * (g.nseg - 1) * kState;
  if (g.nseg - 1 > kFold && sg > 0) {
    add_state(before + (int64_t)(sg - 1) * kState, 0.f);
  } else {
    if (a.state_in) add_state((g.nseg > 1 ? g.init : a.state_in) + bh * kState, 0.f);
    for (int s = 0; s < sg; ++s) add_state(before + (int64_t)s * kState, __builtin_amdgcn_exp2f(g.decay[bh * (g.nseg - 1) + s]));
  }

  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int c = c_lo; c < c_hi; ++c) {
    const bool end = c == g.n_chunks - 1;
    if (wave == 0) {
      int row = lane;
      asm volatile("" : "+v"(row));
      const float G = wave_scan(!end || row < rows_end ? lgr * kLog2e : 0.f), last = lane63(G);
      g_t[row] = G;
      w_t[row] = !end || row < rows_end ? __builtin_amdgcn_exp2f(last - G) : 0.f;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      *(u32x4*)(q_t + q_off + i * 4096) = qr[i];
      *(u32x4*)(k_t + kv_off + i * 4096) = kr[i];
      *(u32x4*)(v_t + kv_off + i * 4096) = vr[i];
    }
    __syncthreads();

    // ---- weights scale * s * 2^(G_q - G_k): wavefronts 0..2 take the blocks (keys, queries) (0, 0), (0, 1), (1, 1);
    // wavefront 3 goes through the motions on (1, 0), which nobody reads, so that all of this is one basic block.
    // ---- O^T = S^T Q^T, every query column times scale * 2^(G_q)
    // The operands of the scores are all requested first and the state's first parts split while they arrive; then the
    // products of the state, each step's operands a step ahead; the scores' weights last.
    // Operand addresses are one base each, XORed with the step; hidden from the compiler, which would otherwise keep all
    // sixty of them in registers across the chunks.
    int qa = row_off(lq, hf), ka = tr_off((wave >> 1) * 32 + lq, hf), kta = kbase, va = vbase, pa = (hf * kC + lq) * 16;
    asm volatile("" : "+v"(qa), "+v"(ka), "+v"(kta), "+v"(va), "+v"(pa));
    auto q_frag = [&](int qb, int ks) { return *(const u32x4*)(q_t + (qa ^ (ks << 5)) + qb * 8192); };
    auto split_state = [&](int ks, u32x4& sh, u32x4& sl) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = (ks & 1) * 8 + i * 2;
        unsigned hi, lo;
        split_bf16(S[ks >> 1][r], S[ks >> 1][r + 1], hi, lo);
        sh[i] = hi;
        sl[i] = lo;
      }
    };
    const int kb = wave >> 1, sqb = wave < 3 ? (wave + 1) >> 1 : 0;
    u32x4 kf[4], qf[4], sh[2], sl[2];
    auto request_scores = [&](int ks) {
      kf[ks & 3] = *(const u32x4*)(k_t + (ka ^ (ks << 5)));
      qf[ks & 3] = q_frag(sqb, ks);
    };
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) request_scores(ks);
    split_state(0, sh[0], sl[0]);
    f32x16 s;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      s = mfma(kf[ks & 3], qf[ks & 3], ks ? s : zero);
      if (ks < 4) request_scores(ks + 4);
    }
    if (GATE) {
#pragma unroll
      for (int i = 0; i < 4; ++i) gr[i] = *(const u32x4*)(gg + (int64_t)c * kC * row_bytes + piece(i, end));
    }
    u32x4 q0[2], q1[2];
    // Raised priority while a wavefront feeds the matrix pipe: the SIMD's other one fills in with its vector work (337 ->
    // 329 us at T = 32768 x 24 heads with gate and state; nothing more from requesting the gate or V earlier).
    __builtin_amdgcn_s_setprio(1);
    q0[0] = q_frag(0, 0);
    q1[0] = q_frag(1, 0);
    f32x16 o[2];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const int x = ks & 1, y = x ^ 1;
      if (ks < 7) {
        q0[y] = q_frag(0, ks + 1);
        q1[y] = q_frag(1, ks + 1);
        split_state(ks + 1, sh[y], sl[y]);
      }
      o[0] = mfma(sh[x], q0[x], ks ? o[0] : zero);
      o[1] = mfma(sh[x], q1[x], ks ? o[1] : zero);
      o[0] = mfma(sl[x], q0[x], o[0]);
      o[1] = mfma(sl[x], q1[x], o[1]);
    }
    __builtin_amdgcn_s_setprio(0);
    {
      const float gq = g_t[sqb * 32 + lq];
#pragma unroll
      for (int u = 0; u < 2; ++u) {                                          // registers 8 u .. 8 u + 7: step 2 kb + u of the second product
        u32x4 ph, pl;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const f32x4 gk = *(const f32x4*)(g_t + kb * 32 + u * 16 + i * 8 + hf * 4);
          float p[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int key = u * 16 + i * 8 + hf * 4 + e;
            p[e] = s[u * 8 + i * 4 + e] * (a.scale * __builtin_amdgcn_exp2f(gq - gk[e]));
            p[e] = key <= lq + 32 * (sqb - kb) ? p[e] : 0.f;
          }
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            unsigned hi, lo;
            split_bf16(p[2 * e], p[2 * e + 1], hi, lo);
            ph[2 * i + e] = hi;
            pl[2 * i + e] = lo;
          }
        }
        const int off = pa + ((2 * kb + u) * 2 * kC + sqb * 32) * 16;
        *(u32x4*)(p_t[0] + off) = ph;
        *(u32x4*)(p_t[1] + off) = pl;
      }
    }
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      const float f = a.scale * __builtin_amdgcn_exp2f(g_t[qb * 32 + lq]);
#pragma unroll
      for (int r = 0; r < 16; ++r) o[qb][r] *= f;
    }
    __syncthreads();                                                         // the scores are there; nobody reads Q any more
    if (GATE) {
#pragma unroll
      for (int i = 0; i < 4; ++i) *(u32x4*)(q_t + q_off + i * 4096) = gr[i];
    }
    if (c + 1 < c_hi) load_qk(c + 1);                                        // in flight during the rest of the chunk

    // ---- the chunk joins the state, and O^T += V^T P^T, 16 rows a step. K's operand of a step is requested behind the
    // state products of the step before, P's at the head of the step; either has eight or four products to arrive in.
    u32x4 vf[2], kt[4], pf[2][2], vh[2], vl[2];
    __builtin_amdgcn_s_setprio(1);
    vf[0] = tr_frag(v_t, va, wave, 0);
#pragma unroll
    for (int eb = 0; eb < 4; ++eb) kt[eb] = tr_frag(k_t, kta, eb, 0);
    const float d = __builtin_amdgcn_exp2f(g_t[kC - 1]);
#pragma unroll
    for (int eb = 0; eb < 4; ++eb)
#pragma unroll
      for (int r = 0; r < 16; ++r) S[eb][r] *= d;
    weigh(vf[0], w_t, 0, hf, vh[0], vl[0]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int x = t & 1, y = x ^ 1;
#pragma unroll
      for (int part = 0; part < 2; ++part)
#pragma unroll
        for (int qb = t < 2 ? 0 : 1; qb < 2; ++qb)                           // keys 32.. come after queries ..31
          pf[part][qb] = *(const u32x4*)(p_t[part] + pa + (t * 2 * kC + qb * 32) * 16);
      if (t < 3) vf[y] = tr_frag(v_t, va, wave, t + 1);
#pragma unroll
      for (int part = 0; part < 2; ++part)
#pragma unroll
        for (int eb = 0; eb < 4; ++eb) S[eb] = mfma(kt[eb], part ? vl[x] : vh[x], S[eb]);
      __builtin_amdgcn_sched_barrier(0);
      if (t < 3) {
#pragma unroll
        for (int eb = 0; eb < 4; ++eb) kt[eb] = tr_frag(k_t, kta, eb, t + 1);
      }
#pragma unroll
      for (int part = 0; part < 2; ++part)
#pragma unroll
        for (int qb = t < 2 ? 0 : 1; qb < 2; ++qb) o[qb] = mfma(vf[x], pf[part][qb], o[qb]);
      if (t < 3) weigh(vf[y], w_t, t + 1, hf, vh[y], vl[y]);
      __builtin_amdgcn_sched_barrier(0);
    }

    __builtin_amdgcn_s_setprio(0);
    if (c + 1 < c_hi) load_v(c + 1);                                         // here, because the products leave no registers for it

    // ---- GroupNorm over a query's 128 values: each wavefront's mean and sum of squares about it, combined over the four
    float shift[2], rstd[2];
    if (NORM) {
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
        float sum = 0.f, sq = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) sum += o[qb][r];
        sum += other_half(sum);
        const float m = sum * (1.f / 32.f);
#pragma unroll
        for (int r = 0; r < 16; ++r) sq = fmaf(o[qb][r] - m, o[qb][r] - m, sq);
        sq += other_half(sq);
        if (hf == 0) {
          red_m[wave][qb * 32 + lq] = m;
          red_s[wave][qb * 32 + lq] = sq;
        }
      }
    }
    __syncthreads();                                                         // the norm's parts and the gate are there
    if (NORM) {
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
        float m[4], sq = 0.f, dev = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          m[w] = red_m[w][qb * 32 + lq];
          sq += red_s[w][qb * 32 + lq];
        }
        const float mean = ((m[0] + m[1]) + (m[2] + m[3])) * 0.25f;
#pragma unroll
        for (int w = 0; w < 4; ++w) dev = fmaf(m[w] - mean, m[w] - mean, dev);
        rstd[qb] = rsqrtf(fmaf(32.f, dev, sq) * (1.f / kD) + a.eps);
        shift[qb] = -mean * rstd[qb];
      }
    }
    int ya = row_off(lq, 0) + hf * 8;
    asm volatile("" : "+v"(ya));
    // swish gate of Eq. 7 (y * g * sigmoid(g)), and the tile of outputs in place of the gate's
#pragma unroll
    for (int qb = 0; qb < 2; ++qb)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        u32x2* cell = (u32x2*)(q_t + (ya ^ ((wave * 4 + rq) << 4)) + qb * 8192);
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = NORM ? fmaf(o[qb][rq * 4 + e], rstd[qb], shift[qb]) : o[qb][rq * 4 + e];
        if (GATE) {
          const u32x2 gw = *cell;
          const float gv[4] = {lo_f(gw[0]), hi_f(gw[0]), lo_f(gw[1]), hi_f(gw[1])};
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] *= gv[e] * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-kLog2e * gv[e]));
        }
        *cell = {pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
      }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {                                            // a thread reads the pieces it overwrites with the next chunk's Q
      if (!end || srow + 16 * i < rows_end) *(u32x4*)(og + (int64_t)c * kC * row_bytes + piece(i, false)) = *(const u32x4*)(q_t + q_off + i * 4096);
    }
  }
  if (a.state_out && sg == g.nseg - 1) store_state(a.state_out + bh * kState, S, wave, lane);
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

bool gret_chunk_supported(int B, int64_t T, int H, int dk, int dv, int chunk, int dtype) {
  if (dtype != YOCO_BF16 || dk != kD || dv != kD) return false;
  if (chunk % 128 || chunk > kMaxChunk) return false;
  if (T <= 0 || (T + 127) / 128 > 65535) return false;
  return B <= 65535;
}

// What callers are told to allocate: cumulative decays and one state per chunk of the caller's size, two states per run of
// chunks. The segments' states are fewer; see segments_of.
int gret_segment_chunks(int B, int H, int nc) {
  int64_t s = (int64_t)nc * B * H / 768;
  if (s < 1) s = 1;
  if (s > 16) s = 16;
  return (int)s;
}

size_t gret_chunk_workspace(int B, int64_t T, int H, int chunk) {
  const size_t nc = (size_t)((T + chunk - 1) / chunk), bh = (size_t)B * H;
  const size_t seg = (size_t)gret_segment_chunks(B, H, (int)nc), nseg = (nc + seg - 1) / seg;
  return align256(bh * nc * chunk * sizeof(float)) + align256(bh * nc * kState * sizeof(float)) +
         2 * align256(bh * nseg * kState * sizeof(float)) + align256(bh * nc * sizeof(float)) + align256(bh * nseg * sizeof(float));
}

// What `nseg` segments of `per` chunks take, in us, from what was measured: a launch of outputs 4.2 and one of segments 3.5; a chunk in both
// 4.7 where the chip is nearly empty, 6.3 with a workgroup on every CU, 7.9 where the first CUs have two and 11.8 where all have, which is
// what HBM and the vector units give; the scan, or each earlier segment that is folded; and the way out and back of a workgroup's state.
float estimate_us(int64_t bh, int nseg, int per) {
  constexpr float kOutputs = 4.2f, kSegments = 3.5f, kScan = 4.6f, kFolded = 1.5f, kStateUs = 0.02f;
  const float wgs = (float)(bh * nseg), cus = (float)compute_units();
  if (nseg == 1) return kOutputs + 4.7f * (float)per;
  const float chunk = wgs <= cus ? 4.7f + 1.6f * wgs / cus : 7.9f + 3.9f * (wgs - cus) / cus;
  const bool scanned = nseg - 1 > kFold;
  return kOutputs + kSegments + (scanned ? kScan + kStateUs * wgs : kFolded * (float)(nseg - 1)) + kStateUs * wgs + chunk * (float)per;
}
// Chunks per segment: all segments resident at once, at most two workgroups per CU, and no more segments than the workspace
// holds states for. Where that leaves a segment eight chunks there are as many (32768 rows x 24 heads, 10 segments 355 us, 21
// segments 337; 4 x 5000 x 24, 4 and 5, 218 and 212). Of shorter ones a CU's second workgroup costs more in states than it
// hides (us, two a CU and as here: 4000 rows x 16 heads 55.9 and 47.2, 2 x 3000 x 16 64.9 and 57.9, 4 x 1000 x 16 56.7 and 44.1,
// 4 x 300 x 24, which one launch does then, 43.8 and 29.1), and the count is the one that the estimate finds, if it promises a
// sixtieth (700 x 16 29.7 in 6 segments, 31.0 in 4). With a CU for each workgroup anyway only the one launch is an alternative (4 x 250 x 24
// 27.5 and 24.1; but 2 x 321 x 16 25.2 in 6 segments, 26.3 in 3).
int gret_chunks_per_segment(int B, int64_t T, int H, int chunk) {
  const int64_t bh = (int64_t)B * H, n_chunks = (T + kC - 1) / kC;
  const int64_t nc = (T + chunk - 1) / chunk, old = gret_segment_chunks(B, H, (int)nc);
  const int64_t room = nc + 2 * ((nc + old - 1) / old);                      // states per head in the workspace: nseg - 1 and a copy of state_in
  int64_t most = 2 * compute_units() / bh;
  if (most > room) most = room;
  if (most > n_chunks) most = n_chunks;
  if (most < 1) most = 1;
  auto per_seg = [&](int64_t nseg) { return (int)((n_chunks + nseg - 1) / nseg); };
  auto us_of = [&](int per) { return estimate_us(bh, (int)((n_chunks + per - 1) / per), per); };
  int best = per_seg(most);
  if (best >= 8) return best;
  float us = 0.985f * us_of(best);
  const bool second = bh * ((n_chunks + best - 1) / best) > compute_units();
  for (int64_t nseg = second ? most - 1 : 1; nseg >= 1; --nseg) {
    const float t = us_of(per_seg(nseg));
    if (t < us) {
      us = t;
      best = per_seg(nseg);
    }
  }
  return best;
}

hipError_t launch_gret_chunk(const GretView& a, int chunk, void* workspace, hipStream_t s) {
  SegArgs g;
  g.a = a;
  g.n_chunks = (int)((a.T + kC - 1) / kC);
  g.per_seg = gret_chunks_per_segment(a.B, a.T, a.H, chunk);
  g.nseg = (g.n_chunks + g.per_seg - 1) / g.per_seg;
  const size_t bh = (size_t)a.B * a.H;
  const size_t nc = (size_t)((a.T + chunk - 1) / chunk);
  g.decay = (float*)workspace;                                               // nseg - 1 <= 3 nc of chunk * nc floats
  g.state = (float*)((char*)workspace + align256(bh * nc * chunk * sizeof(float)));
  g.init = a.state_in && g.nseg > 1 ? g.state + bh * (g.nseg - 1) * kState : nullptr;
  if (g.nseg > 1) {
    hipLaunchKernelGGL(gret_segment_kernel, dim3((unsigned)(bh * (g.nseg - 1))), dim3(256), 0, s, g);
    if (g.nseg - 1 > kFold) hipLaunchKernelGGL(gret_state_scan_kernel, dim3(kState / 1024, a.H, a.B), dim3(256), 0, s, g);
  }
  const dim3 grid((unsigned)(bh * g.nseg)), block(256);
  if (a.group_norm && a.gate) hipLaunchKernelGGL((gret_output_kernel<true, true>), grid, block, 0, s, g);
  else if (a.group_norm) hipLaunchKernelGGL((gret_output_kernel<true, false>), grid, block, 0, s, g);
  else if (a.gate) hipLaunchKernelGGL((gret_output_kernel<false, true>), grid, block, 0, s, g);
  else hipLaunchKernelGGL((gret_output_kernel<false, false>), grid, block, 0, s, g);
  return hipGetLastError();
}

}  // namespace yoco
