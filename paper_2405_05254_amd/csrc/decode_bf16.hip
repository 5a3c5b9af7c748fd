// Split-KV decode of the cross-decoder's attention (Eq. 3 with one query row
// per sequence), bf16 cache, head_dim 128. HBM-bound: every byte of the shared
// K^/V^ planes is read exactly once per call and all G query heads of a KV head
// are served from that one read.
//
// Workgroup = 4 wavefronts on one (sequence, KV head, split). Each wavefront
// takes every fourth 32-row step (16 KiB of K and V) of the split,
// with the next step's loads in flight while the current one is reduced. States are
// merged once at the end (lanes by shuffles, wavefronts through LDS, splits as decode_tail.h says).
//
// Two kernels share that frame. decode_bf16_mfma_kernel (further down) puts both
// products on the matrix cores and serves 1..16 heads per KV head at the rate of a
// plain streaming read. decode_bf16_kernel works on the vector ALU: 128-bit loads
// that cover whole 256-byte rows (16 lanes per row), each group of 16 lanes keeping
// its own online-softmax state (m, l, o[8 dims]) per query head; it serves the
// one-token sliding-window step, which also stores the new row.
#include <type_traits>

#include "decode_tail.h"
#include "yoco_common.h"

namespace yoco {

namespace {

constexpr int kD = 128;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegBig = -1.0e30f;   // "no row seen yet": finite, so m - m never makes NaN

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float dot2_bf16(unsigned a, unsigned b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c, false);
}
__device__ __forceinline__ float bf_lo(unsigned x) { return __uint_as_float(x << 16); }
__device__ __forceinline__ float bf_hi(unsigned x) { return __uint_as_float(x & 0xffff0000u); }

template <int G>
struct State {
  float m[G], l[G], o[G][8];
};

// One step: R rows per lane group (rows u*4 + r of the 4R-row step).
// nvalid = rows of this step that exist (4R in the steady state).
template <int G, int R, bool TAIL>
__device__ __forceinline__ void step(State<G>& st, const u32x4 (&kq)[G], const u32x4 (&kr)[R], const u32x4 (&vr)[R],
                                     float scale_log2, int r, int nvalid) {
  float s[R][G];
#pragma unroll
  for (int u = 0; u < R; ++u) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float a = dot2_bf16(kq[h][0], kr[u][0], 0.f);
      a = dot2_bf16(kq[h][1], kr[u][1], a);
      a = dot2_bf16(kq[h][2], kr[u][2], a);
      a = dot2_bf16(kq[h][3], kr[u][3], a);
      a = over16<LaneSum>(a) * scale_log2;
      if (TAIL && (u * 4 + r >= nvalid)) a = -INFINITY;
      s[u][h] = a;
    }
  }
#pragma unroll
  for (int h = 0; h < G; ++h) {
    float mx = s[0][h];
#pragma unroll
    for (int u = 1; u < R; ++u) mx = fmaxf(mx, s[u][h]);
    const float m_new = fmaxf(st.m[h], mx);
    const float alpha = __builtin_amdgcn_exp2f(st.m[h] - m_new);
    float p[R], psum = 0.f;
#pragma unroll
    for (int u = 0; u < R; ++u) {
      p[u] = __builtin_amdgcn_exp2f(s[u][h] - m_new);
      psum += p[u];
    }
    st.l[h] = st.l[h] * alpha + psum;
    st.m[h] = m_new;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float a0 = st.o[h][2 * i] * alpha, a1 = st.o[h][2 * i + 1] * alpha;
#pragma unroll
      for (int u = 0; u < R; ++u) {
        a0 = fmaf(p[u], bf_lo(vr[u][i]), a0);
        a1 = fmaf(p[u], bf_hi(vr[u][i]), a1);
      }
      st.o[h][2 * i] = a0;
      st.o[h][2 * i + 1] = a1;
    }
  }
}

// The call also stores the new token's K/V row (k_new, v_new: [B,Hkv,128]) at slot lens[b] - 1 (modulo
// the capacity for a rolling cache) and attends to it. The row is taken from registers wherever the stream
// meets its slot, so nothing is read back that this launch writes.
template <int G, int R, typename... Last>
__global__ void __launch_bounds__(256) decode_bf16_kernel(yoco_kv_cache c, const bf16_t* __restrict__ q,
                                                          const int64_t* __restrict__ lens, int64_t fixed_len, int Hq, float scale_log2,
                                                          SplitOut out, const bf16_t* __restrict__ k_new, const bf16_t* __restrict__ v_new,
                                                          int ring, Last... last) {
  if (has_read_ahead(out.splits, last...)) return;
  constexpr int kRowsPerStep = 4 * R;
  __shared__ float red_o[4][G][kD];
  __shared__ float red_ml[4][G][2];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane >> 4, seg = lane & 15;

  const SplitRows part = split_rows<128>(out, c, lens, fixed_len, last...);
  const int b = part.b, g = part.g, sp = part.sp;
  if (sp > 0 && sp >= part.splits && out.tag) return;     // a merge launch reads every split, those without rows too
  const int64_t j_lo = part.lo, j_hi = part.hi;
  const int64_t w_lo = j_lo + wave * kRowsPerStep;        // the wavefronts take turns at the split's steps
  constexpr int kTurn = 4 * kRowsPerStep;

  u32x4 kq[G];
#pragma unroll
  for (int h = 0; h < G; ++h)
    kq[h] = *(const u32x4*)(q + ((int64_t)b * Hq + g * G + h) * kD + seg * 8);

  State<G> st;
#pragma unroll
  for (int h = 0; h < G; ++h) {
    st.m[h] = kNegBig;
    st.l[h] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) st.o[h][i] = 0.f;
  }

  const int64_t plane = ((int64_t)b * c.Hkv + g) * c.N_cap * (kD / 8);          // in 16-byte units
  const u32x4* kp = (const u32x4*)c.k + plane + seg;
  const u32x4* vp = (const u32x4*)c.v + plane + seg;

  int64_t slot = -1;                                   // where the new row goes, -1 = nowhere
  u32x4 knew = {0, 0, 0, 0}, vnew = knew;
  {
    const int64_t pos = (lens ? lens[b] : fixed_len) - 1;
    if (pos >= 0 && (ring || pos < c.N_cap)) slot = pos >= c.N_cap ? pos % c.N_cap : pos;
    knew = *(const u32x4*)(k_new + ((int64_t)b * c.Hkv + g) * kD + seg * 8);
    vnew = *(const u32x4*)(v_new + ((int64_t)b * c.Hkv + g) * kD + seg * 8);
    if (slot >= j_lo && slot < j_hi && wave == 0 && lane < 32) {      // the split that owns the slot stores the row
      u32x4* dst = (u32x4*)(lane < 16 ? c.k : c.v) + plane + slot * (kD / 8) + seg;
      *dst = lane < 16 ? knew : vnew;
    }
  }

  if (w_lo < j_hi) {
    const int64_t last = j_hi - 1;
    u32x4 kn[R], vn[R];
    auto load = [&](int64_t row0) {
#pragma unroll
      for (int u = 0; u < R; ++u) {
        int64_t row = row0 + u * 4 + r;
        row = row < last ? row : last;                 // clamped rows are masked in the tail step
        kn[u] = __builtin_nontemporal_load(kp + row * (kD / 8));
        vn[u] = __builtin_nontemporal_load(vp + row * (kD / 8));
        if (row == slot) {                             // the new row comes from the registers, not from memory
          kn[u] = knew;
          vn[u] = vnew;
        }
      }
    };
    load(w_lo);
    int64_t row0 = w_lo;
    for (; row0 + kTurn < j_hi; row0 += kTurn) {               // steps followed by another step
      u32x4 kc[R], vc[R];
#pragma unroll
      for (int u = 0; u < R; ++u) { kc[u] = kn[u]; vc[u] = vn[u]; }
      load(row0 + kTurn);
      step<G, R, false>(st, kq, kc, vc, scale_log2, r, kRowsPerStep);
    }
    step<G, R, true>(st, kq, kn, vn, scale_log2, r, (int)(j_hi - row0));   // last step, 1 row or more
  }

  // merge the 4 lane groups of the wave
#pragma unroll
  for (int h = 0; h < G; ++h) {
    float M = st.m[h];
    M = over_rows<LaneMax>(M);
    const float f = __builtin_amdgcn_exp2f(st.m[h] - M);
    float l = st.l[h] * f;
    l = over_rows<LaneSum>(l);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float x = st.o[h][i] * f;
      st.o[h][i] = over_rows<LaneSum>(x);
    }
    if (lane < 16) {
#pragma unroll
      for (int i = 0; i < 8; ++i) red_o[wave][h][seg * 8 + i] = st.o[h][i];
      if (lane == 0) { red_ml[wave][h][0] = M; red_ml[wave][h][1] = l; }
    }
  }
  __syncthreads();
  finish_split<G>(out, red_o, red_ml, G, (size_t)b * Hq + g * G, sp, part.splits);
}

// ---- 1..16 query heads per KV head: both products on the matrix cores, so the stream stays HBM-bound whatever
// the group size (the heads are the 16 columns of the MFMA; unused columns carry zeros).
// Wavefront step = 32 rows. Scores: S[key, head] = K[key, :] . Q[head, :] as two 16-key tiles of four
// 16x16x32 products, K fragments loaded from the row-major plane as they are (lane = (key, 8-dim group)).
// Output: O^T[dim, head] += V^T[dim, key] P^T[key, head]; the V fragment (8 keys of one dim per lane) comes
// from the wavefront's own LDS staging rows through the transposing 64-bit read, which hands lane n of a
// 16-lane block the column n of the 4 x 16 tile whose row pieces the block's lanes address. Lane (head, qg)
// then owns dims 16 tt + 4 qg + i of its head in o[tt][i], next to that head's scores, so the online-softmax
// rescale is one factor per lane. P is fed as bf16 high part + bf16 remainder (two products), which keeps
// the weights at fp32-like precision; the row sum l is taken in fp32.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr int kMRows = 32;        // rows per wavefront step
constexpr int kVStride = 288;     // bytes per staged V row: 256 + 32, the 4 rows of a transposing read fall in distinct banks
constexpr int kGMax = 16;
constexpr int64_t kResidentBytes = (int64_t)256 << 20;

// A row piece of the stream, nontemporal or not (launch_decode_bf16 says which caches are read how).
template <bool NT>
__device__ __forceinline__ u32x4 stream(const u32x4* p) { return NT ? __builtin_nontemporal_load(p) : *p; }

struct MState {
  float m, l;
  f32x4 o[8];
};

__device__ __forceinline__ bf16x8_t v_fragment(const unsigned char* lds_row_a, const unsigned char* lds_row_b) {
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)lds_row_a);
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)lds_row_b);
  const s16x8 ab = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(bf16x8_t, ab);
}

template <bool TAIL>
__device__ __forceinline__ void mfma_scores(float (&s)[8], const bf16x8_t (&qf)[4], const u32x4 (&kr)[8], float scale_log2,
                                            int qg, int nvalid) {
#pragma unroll
  for (int tau = 0; tau < 2; ++tau) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kr[tau * 4 + t]), qf[t], acc, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float a = acc[i] * scale_log2;
      if (TAIL && (tau * 16 + qg * 4 + i >= nvalid)) a = -INFINITY;
      s[tau * 4 + i] = a;
    }
  }
}

__device__ __forceinline__ void mfma_softmax_pv(MState& st, const float (&s)[8], const unsigned char* vst, int lane) {
  float smax = s[0];
#pragma unroll
  for (int i = 1; i < 8; ++i) smax = fmaxf(smax, s[i]);
  smax = over_rows<LaneMax>(smax);              // the four lanes of a head hold 8 rows each
  const float m_new = fmaxf(st.m, smax);
  float p[8], psum = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    p[i] = __builtin_amdgcn_exp2f(s[i] - m_new);
    psum += p[i];
  }
  const float alpha = __builtin_amdgcn_exp2f(st.m - m_new);
  st.l = st.l * alpha + psum;
  if (__builtin_amdgcn_ballot_w64(m_new != st.m)) {     // rare once the stream has met its large scores
#pragma unroll
    for (int tt = 0; tt < 8; ++tt) st.o[tt] *= alpha;
  }
  st.m = m_new;
  // weights as two bf16 operands: the upper 16 bits, and the upper 16 bits of what those leave
  u32x4 ph, pl;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const unsigned a = __float_as_uint(p[2 * i]), b = __float_as_uint(p[2 * i + 1]);
    const float ra = p[2 * i] - __uint_as_float(a & 0xffff0000u), rb = p[2 * i + 1] - __uint_as_float(b & 0xffff0000u);
    ph[i] = (a >> 16) | (b & 0xffff0000u);
    pl[i] = (__float_as_uint(ra) >> 16) | (__float_as_uint(rb) & 0xffff0000u);
  }
  const bf16x8_t bh = __builtin_bit_cast(bf16x8_t, ph), bl = __builtin_bit_cast(bf16x8_t, pl);
  // the block of 16 lanes with index kg reads rows 4 kg .. 4 kg + 3 of either 16-row tile: lane s of the block
  // addresses row 4 kg + s / 4, dims 16 tt + 4 (s % 4) .. + 3
  const int sl = lane & 15, kg = lane >> 4;
  const unsigned char* ra = vst + (4 * kg + (sl >> 2)) * kVStride + (sl & 3) * 8;
  const unsigned char* rb = ra + 16 * kVStride;
#pragma unroll
  for (int tt = 0; tt < 8; ++tt) {
    const bf16x8_t vf = v_fragment(ra + tt * 32, rb + tt * 32);
    st.o[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, bh, st.o[tt], 0, 0, 0);
    st.o[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, bl, st.o[tt], 0, 0, 0);
  }
}

template <bool APPEND, int GMAX, typename... Last>
__global__ void __launch_bounds__(256, 2) decode_bf16_mfma_kernel(yoco_kv_cache c, const bf16_t* __restrict__ q,
                                                               const int64_t* __restrict__ lens, int64_t fixed_len, int Hq,
                                                               float scale_log2, SplitOut out, const bf16_t* __restrict__ k_new,
                                                               const bf16_t* __restrict__ v_new, int ring, Last... last) {
  if (has_read_ahead(out.splits, last...)) return;
  // V staging of the four wavefronts (4 x 32 rows x 288 B), and the merge buffers beside it: a wavefront that is done writes
  // its state without waiting for the others (13 layers over 16 ragged sequences of up to 1000 rows 145.6 -> 142.5 us)
  constexpr int kStageBytes = kMRows * kVStride;
  __shared__ __attribute__((aligned(16))) unsigned char smem[4 * kStageBytes];
  __shared__ __attribute__((aligned(16))) float red_o[4][GMAX][kD];
  __shared__ float red_ml[4][GMAX][2];
  const int G = Hq / c.Hkv;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int n = lane & 15, qg = lane >> 4;
  unsigned char* vst = smem + wave * kStageBytes;

  // lane (head n, dim group qg) holds dims 32 t + 8 qg .. + 7 of its head's query for t = 0..3; requested for the sequence
  // that it mostly is before the lengths are there
  u32x4 qraw[4] = {};
  auto load_q = [&](int b, int g) {
    if (n < G) {
#pragma unroll
      for (int t = 0; t < 4; ++t) qraw[t] = *(const u32x4*)(q + ((int64_t)b * Hq + g * G + n) * kD + t * 32 + qg * 8);
    }
  };
  if constexpr (!kSplitsFirst<Last...>) load_q(blockIdx.y, blockIdx.x);
  const SplitRows part = split_rows<128>(out, c, lens, fixed_len, last...);
  const int b = part.b, g = part.g, sp = part.sp;
  if (sp > 0 && sp >= part.splits && out.tag) return;     // a merge launch reads every split, those without rows too
  const int64_t j_lo = part.lo, j_hi = part.hi;
  const int64_t w_lo = j_lo + wave * kMRows;              // the wavefronts take turns at the split's 32-row steps

  if (kSplitsFirst<Last...> || __builtin_expect(b != (int)blockIdx.y, 0)) load_q(b, g);
  bf16x8_t qf[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) qf[t] = __builtin_bit_cast(bf16x8_t, qraw[t]);

  MState st;
  st.m = kNegBig;
  st.l = 0.f;
#pragma unroll
  for (int tt = 0; tt < 8; ++tt) st.o[tt] = (f32x4){0.f, 0.f, 0.f, 0.f};

  const int64_t plane = ((int64_t)b * c.Hkv + g) * c.N_cap * (kD / 8);          // in 16-byte units
  const u32x4* kp = (const u32x4*)c.k + plane + qg;                             // K: lane = (row n of a tile, dims 8 qg ..)
  const u32x4* vp = (const u32x4*)c.v + plane + n;                              // V: lane = (row qg of four, 16-byte piece n)

  // APPEND: the new token's row goes to slot lens[b] - 1 (modulo the capacity for a rolling cache) and is attended
  // to from registers wherever the stream meets its slot, so nothing is read back that this launch writes.
  int64_t slot = -1;
  u32x4 knew[4] = {}, vnew = {0, 0, 0, 0};
  if (APPEND) {
    const int64_t pos = (lens ? lens[b] : fixed_len) - 1;
    if (pos >= 0 && (ring || pos < c.N_cap)) slot = pos >= c.N_cap ? pos % c.N_cap : pos;
    const bf16_t* kn = k_new + ((int64_t)b * c.Hkv + g) * kD;
#pragma unroll
    for (int t = 0; t < 4; ++t) knew[t] = *(const u32x4*)(kn + t * 32 + qg * 8);
    vnew = *(const u32x4*)(v_new + ((int64_t)b * c.Hkv + g) * kD + n * 8);
    if (slot >= j_lo && slot < j_hi && wave == 0 && lane < 32) {      // the split that owns the slot stores the row
      const u32x4 x = *(const u32x4*)((lane < 16 ? kn : v_new + ((int64_t)b * c.Hkv + g) * kD) + n * 8);
      *((u32x4*)(lane < 16 ? c.k : c.v) + plane + slot * (kD / 8) + n) = x;
    }
  }

  if (w_lo < j_hi) {
    const int64_t last = j_hi - 1;
    const int n_steps = (int)((j_hi - w_lo + 4 * kMRows - 1) / (4 * kMRows));
    auto walk = [&](auto nt) {
      constexpr bool NT = decltype(nt)::value;
      u32x4 kr[8], vr[8];
      auto load_k = [&](int i) {
#pragma unroll
        for (int tau = 0; tau < 2; ++tau) {
          int64_t row = w_lo + i * (4 * kMRows) + tau * 16 + n;
          row = row < last ? row : last;               // clamped rows are masked
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            kr[tau * 4 + t] = stream<NT>(kp + row * (kD / 8) + t * 4);
            if (APPEND && row == slot) kr[tau * 4 + t] = knew[t];
          }
        }
      };
      auto load_v = [&](int i) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          int64_t row = w_lo + i * (4 * kMRows) + u * 4 + qg;
          row = row < last ? row : last;               // a written row: finite values under weight 0
          vr[u] = stream<NT>(vp + row * (kD / 8));
          if (APPEND && row == slot) vr[u] = vnew;
        }
      };
      auto stage_v = [&]() {
#pragma unroll
        for (int u = 0; u < 8; ++u) *(u32x4*)(vst + (u * 4 + qg) * kVStride + n * 16) = vr[u];
      };
      float s[8];
      load_k(0);
      load_v(0);
      int i = 0;
      for (; i + 1 < n_steps; ++i) {                   // steps followed by another step
        stage_v();
        load_v(i + 1);
        mfma_scores<false>(s, qf, kr, scale_log2, qg, kMRows);
        load_k(i + 1);
        mfma_softmax_pv(st, s, vst, lane);
      }
      mfma_scores<true>(s, qf, kr, scale_log2, qg, (int)(j_hi - w_lo) - i * (4 * kMRows));   // last step, 1 row or more
      stage_v();
      mfma_softmax_pv(st, s, vst, lane);
    };
    // A cache is read again by the next layer: what fits the 256 MB behind the L2s is read so that it stays there, more
    // than that streams past it (8 x 8 x 1700 rows: 14.3 us instead of 14.9; 16 x 8 x 32768: 300 us instead of 368).
    // A rolling cache belongs to one layer and streams. Where lengths differ residence gives more, up to a fifth (32 x 8 x
    // 60..480 rows: 10.3 us streamed, 8.4); where they are equal it costs up to a tenth from 40 to 95 MB, a little more
    // than the L2s hold (32 x 8 x 380 rows: 9.9 us streamed, 10.9). An unsplit launch does not know which.
    if (APPEND || part.total * (float)c.Hkv > (float)(kResidentBytes / (2 * kD * 2))) walk(std::true_type());
    else walk(std::false_type());
  }

  // One state per head and wavefront: the four lanes of a head sum their row sums; then the merge over wavefronts.
  const float l = over_rows<LaneSum>(st.l);
  if (n < G) {
#pragma unroll
    for (int tt = 0; tt < 8; ++tt)
#pragma unroll
      for (int i = 0; i < 4; ++i) red_o[wave][n][tt * 16 + qg * 4 + i] = st.o[tt][i];
    if (qg == 0) { red_ml[wave][n][0] = st.m; red_ml[wave][n][1] = l; }
  }
  __syncthreads();
  finish_split<GMAX>(out, red_o, red_ml, G, (size_t)b * Hq + g * G, sp, part.splits);
}

}  // namespace

bool decode_bf16_supported(const yoco_kv_cache& c, int Hq) {
  if (c.dtype != YOCO_BF16 || c.d != kD) return false;
  const int G = Hq / c.Hkv;
  return G >= 1 && G <= 16 && c.Hkv <= 65535;
}

// Every call without an append, and append calls with 3..16 heads per KV head, take the matrix-core kernel (HBM-bound
// at every group size). The one-token sliding-window step (append, window of about a thousand rows) of 1 or 2 heads per
// KV head keeps the vector-ALU kernel, whose shorter prologue and merge win there (16 x 24 heads x 1024 rows: 36.1 us
// against 40.9; at 3 heads per KV head, 2 x 8 x 2048 rows, 11.6 against 10.2 the other way round).
hipError_t launch_decode_bf16(const yoco_kv_cache& c, const void* q, const int64_t* lens, int64_t fixed_len, int Hq, float scale,
                              float* ws, int splits, float inv_ragged, float inv_even, int even, int split, int places, unsigned long long tag, void* o, const void* k_new, const void* v_new, int ring,
                              const ReadAhead& ahead, hipStream_t s) {
  const SplitOut out = {ws, (bf16_t*)o, splits, inv_ragged, inv_even, even, places, tag};
  const dim3 grid = decode_grid(c, splits, split, ahead), block(256);
  const float sl2 = scale * kLog2e;
  const bf16_t* qp = (const bf16_t*)q;
  const bf16_t* kn = (const bf16_t*)k_new;
  const bf16_t* vn = (const bf16_t*)v_new;
  const int G = Hq / c.Hkv;
  if (G < 1 || G > kGMax || splits > kMaxDecodeSplits || (tag && !decode_meets_in_launch(G, splits))) return hipErrorInvalidValue;
  auto launch = [&](auto... more) {
    auto go = [&](auto* kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, s, c, qp, lens, fixed_len, Hq, sl2, out, kn, vn, ring, more...); };
    if (!kn) {
      if (G <= 4) go(&decode_bf16_mfma_kernel<false, 4, decltype(more)...>);
      else go(&decode_bf16_mfma_kernel<false, kGMax, decltype(more)...>);
    } else if (G == 1) go(&decode_bf16_kernel<1, 8, decltype(more)...>);
    else if (G == 2) go(&decode_bf16_kernel<2, 8, decltype(more)...>);
    else if (G <= 4) go(&decode_bf16_mfma_kernel<true, 4, decltype(more)...>);
    else go(&decode_bf16_mfma_kernel<true, kGMax, decltype(more)...>);
  };
  if (split) launch(split_first(c, split));
  else if (ahead.workgroups) launch(ahead);
  else launch();
  return hipGetLastError();
}

}  // namespace yoco
