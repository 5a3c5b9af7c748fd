// Flash-style attention prefill on bf16 MFMA for gfx950, head_dim 128.
// Serves yoco_swa_prefill (Eq. 8: causal window of C keys) and
// yoco_cross_attn_prefill (Eq. 3: causal over the global cache, GQA) through
// one kernel: a query at absolute position p sees keys j with p - C < j <= p.
//
// Workgroup = 4 wavefronts, 128 query columns; wavefront w owns columns
// 32w .. 32w+31. Columns are the rows of one head or, where n query heads share
// a KV head and it pays (heads_for), of all n, a row's heads side by side. Keys are walked in tiles of 64, only tiles that intersect
// some row's window are visited, and a wavefront skips the tiles that none of
// its own rows can see; the mask is applied only on the tiles that need it.
//
// Orientation: S^T = K Q^T and O^T = V^T P^T with v_mfma_f32_32x32x16_bf16, so
// a query is a lane column (lane % 32) and keys / head dims run along the
// accumulator registers: the softmax max and sum are in-lane plus one swap
// with lane ^ 32, and the P^T accumulator registers are, as they stand, the B
// operand of the second product (the V^T operand is read from LDS with the
// transposing ds_read_b64_tr_b16 in the matching key order).
//
// Precision: S^T uses bf16 products (exact in fp32). P is rounded to fp16, not
// bf16, and V is converted bf16 -> fp16 (exact for |v| in [2^-14, 65504]) when
// it is staged, so the second product runs on the fp16 MFMA at the same rate:
// with bf16 P the rounding of P alone costs as much error as the rounding of
// the bf16 output, and the two together exceed a 2e-3 mean relative error.
// |v| >= 65520 is outside this kernel's domain (it overflows fp16).
//
// Tiles are double buffered in LDS and the next tile is in flight (global ->
// registers) while the current one is computed. LDS rows are 256 B; K is XOR-swizzled
// in 16-byte chunks and V in 32-byte chunks so both operand read patterns are
// bank-conflict free.
#include <type_traits>

#include "mfma_util.h"
#include "yoco_common.h"

namespace yoco {

namespace {

constexpr int kD = 128;          // head dimension
constexpr int kBN = 64;          // keys per tile
constexpr int kNQ = 32;          // query rows per wavefront
constexpr int kWaves = 4;
constexpr int kThreads = kWaves * 64;
constexpr int kStageRows = 1024 / kThreads;   // 16-byte chunks of a K (or V) tile per thread
constexpr int kStageStep = kThreads / 16;     // rows between a thread's chunks
constexpr int kBM = kNQ * kWaves;
constexpr int kTileBytes = kBN * kD * 2;     // 16 KiB
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegBig = -1.0e30f;
constexpr float kLazyLog2 = 8.0f;            // rescale only when the max grows by more than 2^8

// Columns of a query tile: the rows of one query head, or, PACKED, of the n query heads that share a KV head, one head after another
// within a row. n * row <= column < 2^31, so that row = mulhi(column, mul) >> shift is exact (mul d = 2^(32 + shift) + e, 0 < e <= 2^(shift + 1)).
struct Heads {
  int n;
  unsigned mul;
  int shift;
};
template <bool PACKED>
__host__ __device__ __forceinline__ int64_t row_of(const Heads& hs, int64_t col) {
  if (!PACKED) return col;
#ifdef __HIP_DEVICE_COMPILE__
  return (int64_t)(__umulhi((unsigned)col, hs.mul) >> hs.shift);
#else
  return (unsigned)col / (unsigned)hs.n;
#endif
}

// The kernels' last parameter where heads share tiles (PACKED), and no parameter where they do not: as one that is never used it cost a head
// each 0.05 us a launch (18 rows x 64:8 heads 4.67 and 4.75, 43 x 24:8 5.57 and 5.63).
__device__ __forceinline__ Heads heads_of() { return {1, 0, 0}; }
__device__ __forceinline__ const Heads& heads_of(const Heads& shared) { return shared; }

struct Args {
  AttnView a;
  int n_qtiles;       // query tiles per sequence and head, or KV head where its query heads are packed
  int total;          // workgroups
  int64_t n_keys;     // keys that exist (rows beyond are never read)
  int pieces;         // a query tile's key tiles are shared out over so many workgroups
  int heavy_heads;    // query heads of an XCD, whose heavier query tiles go first over all of them; 0: one KV head after another
  float* part;        // pieces > 1: their partial results (kPieceFloats each), merged by a launch of its own
};

// Partial result of one piece: the accumulators of its 4 wavefronts as the lanes hold them, [wave][16][lane][4], then per
// wavefront and query the maximum (raw scores) and the sum of the weights, [wave][32][2].
constexpr int kPieceMl = kBM * kD;
constexpr int kPieceFloats = kPieceMl + kBM * 2;

// The key tiles that some row of query tile qt sees, and of n tiles the ones of piece p of `pieces` (none if hi < lo).
struct Tiles {
  int lo, hi;
};
template <bool PACKED>
__host__ __device__ __forceinline__ Tiles tiles_of(const AttnView& a, const Heads& hs, int qt) {
  const int64_t c0 = (int64_t)qt * kBM, cols = PACKED ? a.Tq * hs.n : a.Tq;
  const int64_t c1 = (c0 + kBM < cols ? c0 + kBM : cols) - 1;
  const int64_t p0 = a.q_pos0 + row_of<PACKED>(hs, c0), p1 = a.q_pos0 + row_of<PACKED>(hs, c1);
  const int64_t lo_key = p0 - a.window + 1 > 0 ? p0 - a.window + 1 : 0;
  return {(int)(lo_key / kBN), (int)(p1 / kBN)};
}
__host__ __device__ __forceinline__ Tiles piece_of(Tiles t, int p, int pieces) {
  const int n = t.hi - t.lo + 1;
  return {t.lo + (int)((int64_t)n * p / pieces), t.lo + (int)((int64_t)n * (p + 1) / pieces) - 1};
}

template <bool SPLIT, typename... Shared>
__global__ void __launch_bounds__(kThreads, 2) swa_mfma_kernel(Args g, Shared... shared) {
  constexpr bool PACKED = sizeof...(Shared) > 0;
  // Two tile buffers as distinct arrays, so that the compiler can tell the
  // stores of the next tile from the operand reads of the current one.
  __shared__ __attribute__((aligned(1024))) char k_a[kTileBytes], k_b[kTileBytes];
  __shared__ __attribute__((aligned(1024))) char v_a[kTileBytes], v_b[kTileBytes];
  const AttnView& a = g.a;
  const Heads heads = heads_of(shared...);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wavefront-uniform: scalar branches below
  const int hf = lane >> 5, lq = lane & 31;

  // ---- workgroup -> (sequence, head, query tile). Workgroups are dealt to
  // the 8 XCDs round robin; give each XCD a contiguous run of tiles so that
  // neighbouring query tiles (which share K/V tiles) meet in one L2. Within a
  // KV head the G query heads of a tile are adjacent; later (heavier under a
  // causal mask) query tiles go first.
  const int bid = blockIdx.x;
  const int per = g.total >> 3, rem = g.total & 7, xcd = bid & 7;
  const int logical = xcd * per + (xcd < rem ? xcd : rem) + (bid >> 3);
  const int G = PACKED ? 1 : a.Hq / a.Hkv;
  int hh = logical % G;
  int qt = g.n_qtiles - 1 - (logical / G) % g.n_qtiles;
  int outer = logical / (G * g.n_qtiles);
  const int piece = SPLIT ? outer % g.pieces : 0;       // the same piece of all query tiles together: they share key tiles
  if (SPLIT) outer /= g.pieces;
  if (!SPLIT && g.heavy_heads) {                        // heavier tiles first over all heads of the XCD
    const int n = (bid >> 3) % g.heavy_heads;
    qt = g.n_qtiles - 1 - (bid >> 3) / g.heavy_heads;
    hh = n % G;
    outer = (xcd * g.heavy_heads + n) / G;
  }
  const int kvh = outer % a.Hkv;
  const int b = outer / a.Hkv;
  const int h = kvh * G + hh;                           // PACKED: the KV head

  const int64_t i0 = (int64_t)qt * kBM;                 // first column of the workgroup
  const int64_t cols = PACKED ? a.Tq * heads.n : a.Tq;
  const int64_t win = a.window;
  // key tiles that intersect the window of some row of the workgroup
  Tiles tiles = tiles_of<PACKED>(a, heads, qt);
  if (SPLIT) {
    tiles = piece_of(tiles, piece, g.pieces);
    if (tiles.hi < tiles.lo) return;                    // fewer tiles than pieces: the merge knows
  }
  const int jt_lo = tiles.lo, jt_hi = tiles.hi;

  const bf16_t* kg = (const bf16_t*)a.k + b * a.kv_stride_b + kvh * a.kv_stride_h;
  const bf16_t* vg = (const bf16_t*)a.v + b * a.kv_stride_b + kvh * a.kv_stride_h;

  // ---- tile walk. The n_t tiles of this workgroup are visited in the cyclic
  // order "tile index mod n_t" (any order is valid for an online softmax):
  // neighbouring query tiles, which share all but two of their key tiles and
  // run at the same time on the same XCD, then touch the same key tile at the
  // same step, so a tile comes from HBM once and from L2 for its other readers.
  const int n_t = jt_hi - jt_lo + 1;
  const int rot = n_t - jt_lo % n_t;                      // step s visits tile jt_lo + (s + rot) % n_t
  auto tile_of = [&](int s) { return jt_lo + (s + rot) % n_t; };

  // ---- tile staging: global -> registers -> LDS for both K and V. (LDS-direct
  // loads were measured slower here: a wavefront's later LDS reads queue behind
  // its pending global_load_lds, which exposes one memory latency per tile.)
  // V is converted to fp16 on the way. The rows of step s+1 are published
  // during the first product of step s, and the loads of step s+2 follow them.
  const int c16 = tid & 15, srow = tid >> 4;             // thread -> 16-byte chunk c16 of rows srow + 16 i
  const uint32_t row_bytes = (uint32_t)a.kv_stride_n * 2u;
  // LDS byte offsets of row srow (row srow + 16 i is 4096 i further: the
  // swizzles depend on row & 15 / row & 7 only, which 16 i does not change)
  const int kst_off = srow * 256 + ((c16 ^ (srow & 15)) << 4);
  const int vst_off = srow * 256 + (((((c16 >> 1) ^ (srow & 7)) << 1) | (c16 & 1)) << 4);
  u32x4 kst[kStageRows], vst[kStageRows];
  auto load_row = [&](int jt, int i) {
    const int64_t tile_row0 = (int64_t)jt * kBN;
    const int lim = (int)(g.n_keys - 1 - tile_row0 < kBN - 1 ? g.n_keys - 1 - tile_row0 : kBN - 1);   // last row that exists
    const int lrow = srow + kStageStep * i;
    const int grow = lrow < lim ? lrow : lim;             // rows past the end repeat the last one (masked later)
    const uint32_t off = (uint32_t)grow * row_bytes + (uint32_t)(c16 << 4);
    kst[i] = *(const u32x4*)((const char*)(kg + tile_row0 * a.kv_stride_n) + off);
    vst[i] = *(const u32x4*)((const char*)(vg + tile_row0 * a.kv_stride_n) + off);
  };
  auto load_tile = [&](int jt) {
#pragma unroll
    for (int i = 0; i < kStageRows; ++i) load_row(jt, i);
  };
  auto store_row = [&](char* k_dst, char* v_dst, int i) {
    u32x4 vh = {bf16x2_to_f16x2(vst[i][0]), bf16x2_to_f16x2(vst[i][1]), bf16x2_to_f16x2(vst[i][2]),
                bf16x2_to_f16x2(vst[i][3])};
    *(u32x4*)(k_dst + kst_off + i * (kStageStep * 256)) = kst[i];
    *(u32x4*)(v_dst + vst_off + i * (kStageStep * 256)) = vh;
  };

  // ---- Q^T fragments (B operand): lane holds query lq, dims ks*16 + hf*8 .. +8
  const int64_t iw = i0 + wave * kNQ;                   // first column of the wavefront
  const bool any_row = iw < cols;
  struct Place {
    int64_t row, at;                                    // elements from the sequence's first query
  };
  auto place_of = [&](int lane_q) -> Place {            // columns past the end repeat the last one
    const int64_t col = iw + lane_q < cols ? iw + lane_q : cols - 1, row = row_of<PACKED>(heads, col);
    return {row, row * a.q_stride_t + (PACKED ? h * heads.n + (col - row * heads.n) : h) * kD};
  };
  const Place own = place_of(lq);
  const bf16_t* qg = (const bf16_t*)a.q + b * a.q_stride_b + own.at;
  bf16x8 qf[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) qf[ks] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qg + ks * 16 + hf * 8));

  // ---- per-lane LDS byte offsets of the operand fragments (within a tile)
  // K (A operand of S^T): row mb*32 + lq, chunk (ks*2 + hf) ^ (row & 15). The
  // chunk field is bits 4..7 of the offset, so k-step ks is koff0 ^ (ks << 5).
  const int koff0 = lq * 256 + ((hf ^ (lq & 15)) << 4);
  // V^T (A operand of O^T) via transposing reads: lane s = lane % 16 of a block
  // of 16 supplies row z = hf*4 + s/4 (+ t*16 + half*8), dims (mb*2 + db)*16 + 4*(s%4),
  // 32-byte chunk (mb*2 + db) ^ z: dim block mb is voff0 ^ (mb << 6).
  const int s16 = lane & 15, db = (lane >> 4) & 1, z = hf * 4 + (s16 >> 2);
  const int voff0 = z * 256 + ((db ^ z) << 5) + ((s16 & 3) << 3);

  const float c = a.scale * kLog2e;                     // scores are kept raw; exponents use s * c
  const float lazy_raw = kLazyLog2 / c;
  float m_used = kNegBig, l_lane = 0.f;
  f32x16 acc_o[4];
#pragma unroll
  for (int mb = 0; mb < 4; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_o[mb][r] = 0.f;

  // the wavefront's first and last position, relative to tile jt_lo; one without rows lies before all keys, so that it stages tiles
  // and multiplies nothing
  const int64_t origin = (int64_t)jt_lo * kBN - a.q_pos0;
  const int pw_lo = any_row ? (int)(row_of<PACKED>(heads, iw) - origin) : -(1 << 29);
  const int pw_hi = !PACKED ? pw_lo + kNQ - 1 : any_row ? (int)(row_of<true>(heads, iw + kNQ < cols ? iw + kNQ - 1 : cols - 1) - origin) : -(1 << 29);
  const int pq_rel0 = PACKED ? (int)(own.row - origin) : pw_lo + lq;      // this lane's query, same origin
  const int win32 = win > (1 << 30) ? (1 << 30) : (int)win;

  // ---- prologue: tile of step 0 into buffer a, tile of step 1 in flight
  load_tile(tile_of(0));
#pragma unroll
  for (int i = 0; i < kStageRows; ++i) store_row(k_a, v_a, i);
  if (n_t > 1) load_tile(tile_of(1));
  __syncthreads();
  // Q is complete here; saying so keeps the loop free of waits on it (the
  // tile prefetch loads issued inside the loop must stay in flight).
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) asm volatile("" : "+v"(qf[ks]));

  // ---- one step = one key tile (64 keys) for this wavefront:
  //   [S^T = K Q^T  with  publishing the staged rows of the next step's tile
  //    and issuing the loads of the tile after it]
  //   mask (edge tiles only), running max, lazy rescale
  //   [weights and O^T += V^T P^T]
  // The first and third part each mix MFMA with vector work in one basic block,
  // so the two wavefronts that share a SIMD (one per resident workgroup) can
  // overlap their pipes in most phase combinations.
  auto step = [&](int st, char* k_cur, char* v_cur, char* k_nxt, char* v_nxt) {
    const int jt = tile_of(st);
    const int j0r = (jt - jt_lo) * kBN;                 // tile's first key, relative origin
    // does some row of this wavefront see some key of the tile? / every row every key?
    const bool need = (j0r <= pw_hi) && (j0r + kBN - 1 > pw_lo - win32);
    const bool full = (j0r + kBN - 1 <= pw_lo) && (j0r > pw_hi - win32);
    // the same for the two 32-key halves: on edge tiles a wavefront multiplies only the halves it needs
    const bool need0 = need && (j0r + 31 > pw_lo - win32);
    const bool need1 = need && (j0r + 32 <= pw_hi);
    const bool both = need0 && need1;
    const bool stage = st + 1 < n_t, prefetch = st + 2 < n_t;
    lds_char* kb = (lds_char*)k_cur;
    lds_char* vb = (lds_char*)v_cur;
    int kbase = koff0, vbase = voff0;
    asm volatile("" : "+v"(kbase), "+v"(vbase));        // keep the 12 derived offsets out of long-lived registers
    auto kfrag = [&](int ks, int mb) {
      return __builtin_bit_cast(bf16x8, *(const __attribute__((address_space(3))) u32x4*)(kb + (kbase ^ (ks << 5)) + mb * 32 * 256));
    };
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 s0 = zero, s1 = zero;                         // keys 0..31 and 32..63 of the tile
    if (both && prefetch) {
      // the common case, one basic block: 16 MFMAs, the 4 staged rows, 8 loads
      const int jt2 = tile_of(st + 2);
      // raised issue priority while this wavefront feeds the matrix pipe: the
      // other wavefront of the SIMD fills in with its vector work (measured -4 %)
      __builtin_amdgcn_s_setprio(2);
      // operand fragments are read two k-steps (4 MFMAs) ahead of their use
      bf16x8 f0[8], f1[8];
      f0[0] = kfrag(0, 0); f1[0] = kfrag(0, 1);
      f0[1] = kfrag(1, 0); f1[1] = kfrag(1, 1);
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        if (ks + 2 < 8) { f0[ks + 2] = kfrag(ks + 2, 0); f1[ks + 2] = kfrag(ks + 2, 1); }
        s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f0[ks], qf[ks], ks == 0 ? zero : s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f1[ks], qf[ks], ks == 0 ? zero : s1, 0, 0, 0);
        // a staged row is published and its registers reloaded at once: the
        // loads go out a pair at a time between the products, not as a burst
        if ((ks & 1) && (ks >> 1) % (4 / kStageRows) == 0) {
          store_row(k_nxt, v_nxt, (ks >> 1) / (4 / kStageRows));
          load_row(jt2, (ks >> 1) / (4 / kStageRows));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_setprio(0);
    } else {
      if (need0) {
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfrag(ks, 0), qf[ks], ks == 0 ? zero : s0, 0, 0, 0);
      }
      if (need1) {
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfrag(ks, 1), qf[ks], ks == 0 ? zero : s1, 0, 0, 0);
      }
      if (stage) {
#pragma unroll
        for (int i = 0; i < kStageRows; ++i) store_row(k_nxt, v_nxt, i);
      }
      if (prefetch) load_tile(tile_of(st + 2));
    }
    if (need) {
      if (!full) {                                       // keys outside (p - C, p] of this lane's query
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = j0r + (r >> 2) * 8 + hf * 4 + (r & 3);
          s0[r] = (need0 && (unsigned)(pq_rel0 - key) < (unsigned)win32) ? s0[r] : -INFINITY;
          s1[r] = (need1 && (unsigned)(pq_rel0 - key - 32) < (unsigned)win32) ? s1[r] : -INFINITY;
        }
      }
      // ---- online softmax (a query is the lane pair l, l ^ 32); the
      // accumulators are rescaled only when the max grows by more than 2^kLazyLog2
      float mx = fmaxf(s0[0], s1[0]);
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, fmaxf(s0[r], s1[r]));
      mx = fmaxf(mx, other_half(mx));
      const bool grow = mx > m_used + lazy_raw;
      if (__builtin_amdgcn_ballot_w64(grow) != 0) {
        const float m_new = grow ? mx : m_used;
        const float alpha = __builtin_amdgcn_exp2f((m_used - m_new) * c);
        m_used = m_new;
        l_lane *= alpha;
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc_o[mb][r] *= alpha;
      }
      const float mc = m_used * c;
      unsigned pk0[8], pk1[8];
      const unsigned ones = 0x3c003c00u;                // (1.0, 1.0) in fp16
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        pk0[r >> 1] = pack_f16(__builtin_amdgcn_exp2f(fmaf(s0[r], c, -mc)), __builtin_amdgcn_exp2f(fmaf(s0[r + 1], c, -mc)));
        pk1[r >> 1] = pack_f16(__builtin_amdgcn_exp2f(fmaf(s1[r], c, -mc)), __builtin_amdgcn_exp2f(fmaf(s1[r + 1], c, -mc)));
        // the row sum uses the rounded weights, the ones the second product sees
        l_lane = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, pk0[r >> 1]), __builtin_bit_cast(f16x2, ones), l_lane, false);
        l_lane = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, pk1[r >> 1]), __builtin_bit_cast(f16x2, ones), l_lane, false);
      }
      // ---- O^T += V^T P^T ; k-step t covers keys t*16 .. t*16+15 of the tile
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (!both && !((t >> 1) ? need1 : need0)) continue;   // a skipped half has zero weights
        const unsigned* pk = (t >> 1) ? pk1 : pk0;
        const int pb = (t & 1) * 4;
        u32x4 pu = {pk[pb], pk[pb + 1], pk[pb + 2], pk[pb + 3]};
        const f16x8 pf = __builtin_bit_cast(f16x8, pu);
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) {
          const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(vb + (vbase ^ (mb << 6)) + (t * 16) * 256));
          const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(vb + (vbase ^ (mb << 6)) + (t * 16 + 8) * 256));
          u32x2 a0 = __builtin_bit_cast(u32x2, v0), a1 = __builtin_bit_cast(u32x2, v1);
          u32x4 vu = {a0[0], a0[1], a1[0], a1[1]};
          acc_o[mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, vu), pf, acc_o[mb], 0, 0, 0);
        }
      }
      __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();
  };
  for (int st = 0; st < n_t; st += 2) {
    step(st, k_a, v_a, k_b, v_b);
    if (st + 1 >= n_t) break;
    step(st + 1, k_b, v_b, k_a, v_a);
  }

  if (!any_row) return;
  const float l_tot = l_lane + other_half(l_lane);
  if (SPLIT) {                                           // unnormalised, in the order that the lanes hold it: 1 KiB a store
    float* const part = g.part + ((((int64_t)b * (PACKED ? a.Hkv : a.Hq) + h) * g.n_qtiles + qt) * g.pieces + piece) * kPieceFloats;
    f32x4* const po = (f32x4*)part + wave * 1024 + lane;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq)
        __builtin_nontemporal_store(f32x4{acc_o[mb][rq * 4], acc_o[mb][rq * 4 + 1], acc_o[mb][rq * 4 + 2], acc_o[mb][rq * 4 + 3]}, po + (mb * 4 + rq) * 64);
    if (hf == 0) *(f32x2*)(part + kPieceMl + (wave * kNQ + lq) * 2) = f32x2{m_used, l_tot};
    return;
  }
  // ---- normalise and store O (bf16, rounded once)
  const float inv = 1.f / l_tot;
  if (iw + lq < cols) {
    int again = lq;
    if (PACKED) asm volatile("" : "+v"(again));          // keeps the place out of registers across the walk
    bf16_t* og = (bf16_t*)a.o + b * a.q_stride_b + place_of(again).at;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        u32x2 w = {pack_bf16(acc_o[mb][rq * 4] * inv, acc_o[mb][rq * 4 + 1] * inv),
                   pack_bf16(acc_o[mb][rq * 4 + 2] * inv, acc_o[mb][rq * 4 + 3] * inv)};
        *(u32x2*)(og + mb * 32 + rq * 8 + hf * 4) = w;
      }
  }
}

// ---- the merge of a query tile's pieces: o = sum_p 2^((m_p - M) c) o_p / sum_p 2^((m_p - M) c) l_p, in a fixed order.
// A workgroup takes 8 RQ dims of a query tile, its lanes what the attention kernel's lanes held. Bound by the partials, 66 KB
// for each piece, which mostly come back from the memory behind the L2s; where query tiles are few, by the trips there: a group of
// pieces each, of as many as 64 registers hold. 16 dims a workgroup are twice the workgroups and half the trips, and gain
// up to as many query tiles as an eighth of the CUs (us a call, with 32 dims and with 16: 9 rows x 3:1 heads over 3831 18.8 and 17.4,
// 38 x 24 over 20108 45.4 and 44.3, 128 x 24 over 16000 48.0 and 46.8; but 69 x 64 heads over 1741, 64 tiles, 25.4 and 27.1),
// where there are more than four pieces, one trip of the larger half (195 x 16:4 over 272, four, 14.2 and 14.9). 8 dims gain nothing more.
template <int RQ, typename... Shared>
__global__ void __launch_bounds__(kThreads) swa_merge_kernel(Args g, Shared... shared) {
  constexpr bool PACKED = sizeof...(Shared) > 0;
  const AttnView& a = g.a;
  const Heads shape = heads_of(shared...);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hf = lane >> 5, lq = lane & 31;
  const int qt = blockIdx.x, mb = blockIdx.y / (4 / RQ), rq0 = blockIdx.y % (4 / RQ) * RQ, head = blockIdx.z, heads = PACKED ? a.Hkv : a.Hq, b = head / heads, h = head % heads;
  const int64_t col = (int64_t)qt * kBM + wave * kNQ + lq, cols = PACKED ? a.Tq * shape.n : a.Tq;
  if ((int64_t)qt * kBM + wave * kNQ >= cols) return;      // a wavefront without rows has stored nothing
  const float c = a.scale * kLog2e;
  const Tiles tiles = tiles_of<PACKED>(a, shape, qt);
  const int n = tiles.hi - tiles.lo + 1, pieces = g.pieces;
  const float* const first = g.part + ((int64_t)head * g.n_qtiles + qt) * pieces * kPieceFloats;
  float M = kNegBig, L = 0.f;
  constexpr int kMergeAhead = 16 / RQ;
  f32x4 o[RQ] = {};
  for (int p0 = 0; p0 < pieces; p0 += kMergeAhead) {       // a group's loads go out together
    f32x2 ml[kMergeAhead];
    f32x4 x[kMergeAhead][RQ];
#pragma unroll
    for (int i = 0; i < kMergeAhead; ++i) {
      const int p = p0 + i < pieces ? p0 + i : pieces - 1;
      const float* const part = first + (int64_t)p * kPieceFloats;
      ml[i] = *(const f32x2*)(part + kPieceMl + (wave * kNQ + lq) * 2);
#pragma unroll
      for (int rq = 0; rq < RQ; ++rq) x[i][rq] = ((const f32x4*)part)[wave * 1024 + (mb * 4 + rq0 + rq) * 64 + lane];
    }
    float m_new = M;
    bool live[kMergeAhead];
#pragma unroll
    for (int i = 0; i < kMergeAhead; ++i) {                // a piece without tiles has stored nothing
      const int p = p0 + i;
      live[i] = p < pieces && (int64_t)n * (p + 1) / pieces > (int64_t)n * p / pieces;
      m_new = live[i] ? fmaxf(m_new, ml[i][0]) : m_new;
    }
    const float alpha = __builtin_amdgcn_exp2f((M - m_new) * c);
    M = m_new;
    L *= alpha;
#pragma unroll
    for (int rq = 0; rq < RQ; ++rq) o[rq] *= alpha;
#pragma unroll
    for (int i = 0; i < kMergeAhead; ++i) {
      if (!live[i]) continue;
      const float f = __builtin_amdgcn_exp2f((ml[i][0] - M) * c);
      L = fmaf(f, ml[i][1], L);
#pragma unroll
      for (int rq = 0; rq < RQ; ++rq)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[rq][e] = fmaf(f, x[i][rq][e], o[rq][e]);
    }
  }
  if (col >= cols) return;
  const float inv = 1.f / L;
  const int64_t row = row_of<PACKED>(shape, col), query_head = PACKED ? h * shape.n + (col - row * shape.n) : h;
  bf16_t* const og = (bf16_t*)a.o + b * a.q_stride_b + row * a.q_stride_t + query_head * kD + mb * 32 + hf * 4;
#pragma unroll
  for (int rq = 0; rq < RQ; ++rq)
    *(u32x2*)(og + (rq0 + rq) * 8) = u32x2{pack_bf16(o[rq][0] * inv, o[rq][1] * inv), pack_bf16(o[rq][2] * inv, o[rq][3] * inv)};
}

Tiles tiles_for(const AttnView& a, const Heads& hs, int qt) { return hs.n > 1 ? tiles_of<true>(a, hs, qt) : tiles_of<false>(a, hs, qt); }
constexpr Heads kOneHead = {1, 0, 0};
int qtiles_for(const AttnView& a, const Heads& hs) { return (int)((a.Tq * hs.n + kBM - 1) / kBM); }
int64_t units_for(const AttnView& a, const Heads& hs) { return (int64_t)a.B * (a.Hq / hs.n); }

// How many pieces a call's query tiles are cut into. A workgroup's walk over the keys is serial, so a call with few
// query tiles leaves the chip idle (64 rows x 16 heads over 24000 rows: 16 workgroups of 376 tiles each, 508 us; in 32 pieces
// 46), and one whose workgroups are no multiple of the places (two a CU) waits for the CUs that hold two (2000 rows x 24
// heads over 16000: 384 workgroups 457 us, in 4 pieces three full rounds, 423). The estimate is in us, from what was measured: a
// 64-key tile takes 1.34 where a CU has one workgroup, 1.6 where some have two and 2.15 where all have; 5 for a launch and
// the two ends of a walk; a merge 5, 0.016 for each piece's way out and back and 0.35 for every trip after the first (1000 rows x 1 head
// 15.7 us without it, in sixteen pieces, 14.0 with, in eight) as far as workgroups have a CU each: two on a CU take less than the
// estimate has it, and beyond that no trip is counted (29 x 16:8 heads over 18145 in 32 pieces 31.0, in 16 35.1, 130 x 32:8 over 4554 in 7
// 35.3, in 4 38.1, 255 x 24:8 over 4932 in 10 35.5, in 5 38.0). 30 shapes of 16 to 4096 rows are within a
// tenth of their best count by it. A cut has to promise a twentieth, because it costs memory.
constexpr int kMaxPieces = 32;
// How many pieces the merge of so many query tiles reads in a trip.
int merge_ahead(int64_t items, int64_t pieces) { return pieces > 4 && 8 * items <= compute_units() ? 8 : 4; }
constexpr int64_t kMaxPieceWgs = 1536;         // bounds the partials at 102 MB
float estimate_us(int64_t items, int n_max, float n_mean, int pieces) {
  const int64_t cus = compute_units(), places = 2 * cus;
  constexpr float kEnds = 5.f, kAlone = 1.34f, kSome = 1.6f, kAll = 2.15f, kMerge = 5.f, kPiece = 0.016f, kTrip = 0.35f;
  const int64_t wgs = items * pieces, full = wgs / places, rest = wgs % places;
  auto tile = [&](int64_t n) { return n <= cus ? kAlone : kSome + (kAll - kSome) * (float)(n - cus) / (float)(places - cus); };
  const float longest = ceilf((float)n_max / (float)pieces), mean = n_mean / (float)pieces;
  float t = (float)full * (mean * kAll + kEnds) + (rest ? mean * tile(rest) + kEnds : 0.f);
  const float least = longest * tile(wgs < places ? wgs : places) + kEnds;
  if (t < least) t = least;
  const int64_t alone = wgs <= cus ? pieces : cus / items;       // pieces at a CU for each workgroup
  return pieces > 1 ? t + kMerge + kPiece * (float)wgs + kTrip * (float)(alone > 1 ? (alone - 1) / merge_ahead(items, alone) : 0) : t;
}
struct Cut {
  int pieces;
  float us;
};
Cut cut_for(const AttnView& a, const Heads& hs, int64_t room) {
  const int n_qtiles = qtiles_for(a, hs);
  const int64_t items = n_qtiles * units_for(a, hs);
  int n_max = 0;
  int64_t sum = 0;
  for (int qt = 0; qt < n_qtiles; ++qt) {
    const Tiles t = tiles_for(a, hs, qt);
    sum += t.hi - t.lo + 1;
    if (t.hi - t.lo + 1 > n_max) n_max = t.hi - t.lo + 1;
  }
  const float mean = (float)sum / (float)n_qtiles;
  Cut best = {1, estimate_us(items, n_max, mean, 1)};
  float us = 0.95f * best.us;
  for (int p = 2; p <= kMaxPieces && p <= n_max && items * p <= kMaxPieceWgs && items * p <= room; ++p) {
    const float t = estimate_us(items, n_max, mean, p);
    if (t < us) {
      us = t;
      best = {p, t};
    }
  }
  return best;
}
int pieces_for(const AttnView& a, const Heads& hs, int64_t room) {
  const int64_t items = qtiles_for(a, hs) * units_for(a, hs);
  return 2 * items > kMaxPieceWgs || 2 * items > room ? 1 : cut_for(a, hs, room).pieces;
}

// Whether the query heads of a KV head share its query tiles. A tile of 128 columns is then 128 / n rows: its walk over the keys is that
// much shorter at the diagonal and at the window's end (24:8 heads, window 1024: 96 % of the key tiles, window 512: 91), fewer
// columns lie idle behind the last row, and walks differ less. us, a head each and so: 4 x 1532 rows x 24:8 77.5 and 73.2, 2 x 1598,
// window 512, 38.8 and 33.2, 12 x 204 22.6 and 15.1, 8 x 655 x 32:8 66.5 and 54.3, 32491 rows, window 2048, 928 and 907; over a
// cache 151 rows x 64:8 over 22574 172 and 144, 1323 x 24:8 over 2102 82.2 and 80.5.
// A call that leaves the chip idle lasts as long as its longest walk, 1.34 a key tile and 0.55 for each wavefront that has columns (its
// queries, its outputs and its share of the CU): a head's last rows on one or two wavefronts of many CUs are then better than on four of a
// few (25 rows x 64:8 over themselves 4.9 and 6.7, 290 x 16:4 11.9 and 12.4, 18 x 32:8 over 3383, cut into pieces, 20.4 and 22.7; the
// other way round 69 x 16:4 7.8 and 7.0, 331 x 6:3 13.8 and 12.6). Rows of one tile a head, which are cut into pieces over a cache, are
// asked the same with half of the key tiles, because the wavefronts' part is not cut (64 x 24:8 over 1031 14.1 and 15.9, 60 x 24:8 over 517 12.3 and 13.6).
// From 2500 key tiles on, up to four tiles a head share always. More of them, in one round of the chip, where no walk comes near what
// it was (window 512, 4 x 727 x 16:8, 25.2 and 23.2, window 1024, 3139 x 16:4, 43.2 and 40.9), or where the estimate promises a fourteenth (1321 x 16:4
// over 13261 211 and 190, 1464 x 16:4 over 585 50.9 and 43.1); what promises less is one or the other (2447 x 16:4 over 154 63.3 and 69.1, 2581 x
// 16:4 over 241 76.0 and 80.6, 2354 x 16:4 over 172 62.5 and 60.9). A cut in two on a CU against none there counts for nothing, the
// estimate has that one too high (1965 x 32:8 over 368 73.0 and 81.1, 1615 x 24:8 over 530 61.3 and 62.8).
// With one key tile there is no walk to shorten (16 x 16:8 over themselves 4.7 and 4.8).
// Of 1768 drawn grouped calls of one round the mean is 3 % faster than a head each; 40 are more than 1 % slower, the worst 4.6 (68 x 24:8
// over 1541 18.1 and 19.0), where two processes differ by up to 4.
Heads heads_for(const AttnView& a, int64_t room) {
  const int n = a.Hq / a.Hkv;
  if (n == 1 || a.Tq * n >= (1LL << 31) - kBM) return kOneHead;
  int bits = 1;
  while ((1LL << bits) < n) ++bits;
  const Heads packed = {n, (unsigned)((1ULL << (31 + bits)) / n + 1), bits - 1};
  if (qtiles_for(a, kOneHead) * units_for(a, kOneHead) > 2 * compute_units()) return packed;
  if (a.q_pos0 + a.Tq <= kBN) return kOneHead;
  int64_t sum[2];
  float longest[2], cut[2];                           // the longest walk, whole and with half its key tiles
  for (int i = 0; i < 2; ++i) {
    const Heads& hs = i ? packed : kOneHead;
    sum[i] = 0;
    longest[i] = cut[i] = 0.f;
    for (int qt = 0, n_qtiles = qtiles_for(a, hs); qt < n_qtiles; ++qt) {
      const Tiles t = tiles_for(a, hs, qt);
      const int64_t left = a.Tq * hs.n - (int64_t)qt * kBM;
      const float walk = 1.34f * (float)(t.hi - t.lo + 1), ends = 0.55f * (float)(left < kBM ? (left + kNQ - 1) / kNQ : kWaves);
      if (walk + ends > longest[i]) longest[i] = walk + ends;
      if (0.5f * walk + ends > cut[i]) cut[i] = 0.5f * walk + ends;
      sum[i] += (t.hi - t.lo + 1) * units_for(a, hs);
      if (i == 0 && sum[0] >= 2500 && a.Tq <= 4 * kBM) return packed;
    }
  }
  if (sum[0] >= 2500) {
    if (longest[1] <= 0.97f * longest[0]) return packed;
    const Cut one = cut_for(a, kOneHead, room), shared = cut_for(a, packed, room);
    const bool alike = one.pieces > 1 || shared.pieces == 1 || qtiles_for(a, packed) * units_for(a, packed) <= compute_units();
    return alike && shared.us <= 0.93f * one.us ? packed : kOneHead;
  }
  return longest[1] <= longest[0] + 0.3f && (a.Tq > kBM || cut[1] <= cut[0] + 0.3f) ? packed : kOneHead;
}

// Where walks differ much (their mean is under three quarters of the longest: causal attention over up to twice the window)
// and the launch is a few rounds of the chip's places, the heavier query tiles go first over all heads of an XCD, so that it
// ends in short walks everywhere: 8 x 1000 rows x 16 heads 69.4 -> 56.4 us, 4096 rows x 24 heads
// without a window 145 -> 127. But all of the XCD's KV heads are walked side by side then, and
// the fewer workgroups of one are in flight, the less of its key tiles comes from the L2 (one KV head after another, heavier
// first, us): 59 x 1900 x 24 heads 1551 and 2174, 12 x 700 x 24 77 and 83, 14 x 1100 x 40 277 and 342, 16 x 4096 x 24 without a
// window 2051 and 2343. In a longer launch the end matters less, too: 8 x 3000 x 24, nine rounds, 503 and 524. Query tiles in
// fours gain for longer (12 x 500 x 24 61.3 and 52.7, 6 x 1000 x 40 118 and 109): dealt out head after head, the heavier ones
// of all heads meet on the same CUs.
// Where query heads share their KV head's tiles, more of its workgroups are in flight already, but their walks are as uneven (one KV head after
// another and heavier first, us): one KV head an XCD gains nothing. Two up to 1.3 rounds (2 x 1464 x 24:8 42.0 and 38.8, 2 x 1367 x 32:8 41.8 and
// 41.2; 1.44 rounds, 2 x 736 x 64:8, 29.7 and 32.3), of walks beyond 20 tiles up to 1.5 (2 x 1838 x 24:8, window 2048, 59.9 and 58.3) and where a later round
// is nearly full (2.8 rounds, 3822 rows, 171 and 162; but 2.3, 3134 rows, 126 and 127). From three on up to 240 query heads two rounds (8 x 881 x
// 16:8 51.9 and 42.5, 8 x 637 x 24:8 43.9 and 39.1, 10 x 430 x 24:8 34.8 and 33.0), up to 216 four (9 x 1257 x 16:8, window 2048, 91.3 and 82.6, 7 x 1150 x 24:8 86.0
// and 81.0, 6 x 1805 x 24:8, window 2048, 156 and 154; but 10 x 557 x 24:8, 2.2 rounds, 43.2 and 44.8). More of them up to four rounds with three or four KV
// heads an XCD (3 x 1300 x 32:8 64.8 and 59.0), with five to eight where the last round is at most half full (8 x 655 x 32:8, 2.6 rounds, 54.3
// and 55.6), with more where it is nearly empty (12 x 1018 x 16:8 86.0 and 79.5). A grouped call of a head each has one round at
// most: 2 x 300 x 64:8 16.5 and 14.5, nine and more heads none.
// A head of three query tiles is left alone where it fills one and a half rounds (12 x 300 x 24 29.6 and 33.0) or nearly one
// (6 x 300 x 24 17.2 and 18.6; 8 x 300, one and an eighth, 26.0 and 24.5), and so is a launch whose workgroups have a CU each.
// Elsewhere one KV head follows another (32768 rows x 24 heads 553 us, heavier first 558; 2 x 4000, window 512, 81.8 and 84.2).
int heavy_heads_for(const AttnView& a, const Heads& hs, int n_qtiles) {
  const int64_t kv_heads = (int64_t)a.B * a.Hkv, wgs = n_qtiles * units_for(a, hs), places = 2 * compute_units();
  const int group = a.Hq / a.Hkv;
  if (kv_heads % 8 || n_qtiles > 256 || 2 * wgs <= places) return 0;
  if (n_qtiles <= 3 && (2 * wgs > 3 * places || (16 * wgs > 13 * places && wgs <= places))) return 0;
  const int64_t rest = wgs % places, query_heads = (int64_t)a.B * a.Hq;
  bool few;
  if (hs.n == 1) {
    few = group == 1 ? wgs <= 2 * places || (kv_heads <= 192 && wgs <= 7 * places) || (n_qtiles % 4 == 0 && wgs <= 3 * places)
                     : group <= 3 || (group <= 8 && kv_heads >= 16);
  } else if (wgs <= places) {
    few = true;
  } else if (kv_heads < 24) {
    const bool long_walks = a.window > 20 * kBN && a.q_pos0 + a.Tq > 20 * kBN;
    few = kv_heads >= 16 && (10 * wgs <= 13 * places || (long_walks && (2 * wgs <= 3 * places || (4 * rest >= 3 * places && wgs <= 3 * places))));
  } else {
    few = (query_heads <= 240 && wgs <= 2 * places) ||
          (wgs <= 4 * places && (query_heads <= 216 || kv_heads <= 32 || 8 * rest <= places || (kv_heads <= 64 && 2 * rest <= places)));
  }
  if (!few) return 0;
  int64_t sum = 0, longest = 0;
  for (int qt = 0; qt < n_qtiles; ++qt) {
    const Tiles t = tiles_for(a, hs, qt);
    sum += t.hi - t.lo + 1;
    if (t.hi - t.lo + 1 > longest) longest = t.hi - t.lo + 1;
  }
  return 4 * sum < 3 * longest * n_qtiles ? (int)(units_for(a, hs) / 8) : 0;
}

}  // namespace

bool swa_mfma_supported(const AttnView& a, int dtype) {
  if (dtype != YOCO_BF16 || a.d != kD) return false;
  if (!(a.scale > 0.f) || !(a.scale < 1e30f)) return false;      // the kernel tracks max(s) and multiplies by scale later
  if (a.q_pos0 + a.Tq >= (1LL << 30)) return false;                 // 32-bit relative positions inside the kernel
  const int64_t n_qtiles = (a.Tq + kBM - 1) / kBM;
  const int64_t total = n_qtiles * a.Hq * a.B;
  return total < (1LL << 31);
}

size_t swa_mfma_workspace(const AttnView& a) {
  auto bytes = [&](const Heads& hs) {
    const int pieces = pieces_for(a, hs, kMaxPieceWgs);
    return pieces > 1 ? (size_t)qtiles_for(a, hs) * units_for(a, hs) * pieces * kPieceFloats * sizeof(float) : 0;
  };
  const Heads hs = heads_for(a, kMaxPieceWgs);
  const size_t one = bytes(kOneHead), own = hs.n > 1 ? bytes(hs) : 0;        // never less than for a head each
  return one > own ? one : own;
}

hipError_t launch_swa_mfma(const AttnView& a, void* workspace, size_t workspace_bytes, hipStream_t s) {
  const int64_t room = workspace ? (int64_t)(workspace_bytes / (kPieceFloats * sizeof(float))) : 0;
  const Heads heads = heads_for(a, room);
  Args g;
  g.a = a;
  g.n_qtiles = qtiles_for(a, heads);
  g.n_keys = a.q_pos0 + a.Tq;
  g.part = (float*)workspace;
  g.pieces = pieces_for(a, heads, room);
  const int64_t units = units_for(a, heads);
  g.total = (int)(g.n_qtiles * units * g.pieces);
  g.heavy_heads = g.pieces == 1 ? heavy_heads_for(a, heads, g.n_qtiles) : 0;
  auto launch = [&](auto... shared) {
    if (g.pieces == 1) {
      hipLaunchKernelGGL((swa_mfma_kernel<false, decltype(shared)...>), dim3(g.total), dim3(kThreads), 0, s, g, shared...);
      return;
    }
    hipLaunchKernelGGL((swa_mfma_kernel<true, decltype(shared)...>), dim3(g.total), dim3(kThreads), 0, s, g, shared...);
    if (merge_ahead(g.n_qtiles * units, g.pieces) == 8)
      hipLaunchKernelGGL((swa_merge_kernel<2, decltype(shared)...>), dim3(g.n_qtiles, 8, (unsigned)units), dim3(kThreads), 0, s, g, shared...);
    else
      hipLaunchKernelGGL((swa_merge_kernel<4, decltype(shared)...>), dim3(g.n_qtiles, 4, (unsigned)units), dim3(kThreads), 0, s, g, shared...);
  };
  if (heads.n > 1) launch(heads);
  else launch();
  return hipGetLastError();
}

}  // namespace yoco
