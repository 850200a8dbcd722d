// Causal prefill attention of a prompt under the progressive sliding
// attention window (Sec. 4.2, Eq. psaw: the window narrows during prefill
// as well as decoding).  The query at position i of sequence b (i < n_b)
// attends the keys p <= i with p < C_sink or p >= vis_start(i), the first
// visible position of Eq. psaw with the i + 1 tokens [0, i] in view (computed
// per query from the layer's factor); without PSAW every p <= i (plain
// causal attention, Eq. attn_eq per position).
//
// attn_prefill_bf16<D, W, NS, PAGED>: one workgroup per (block of queries,
// batch, query head), over a contiguous or paged cache.  A wave takes W = 32
// (8 waves) or 16 (12 waves) queries as the columns of its MFMA tiles; with
// NS > 1 key sides (W = 32), NS waves share the same queries and each takes
// its own 32- or 64-key part of every key tile, their online softmax states
// combined at the end.  Key tiles (64 rows; 128 with NS > 1) are loaded once
// per workgroup (whole rows, one tile ahead of their use; the default cache
// policy, since the unit's other query blocks read the same rows) into two
// LDS buffers, K and V both row-major, and a wave computes per 32 keys
//   S^T (32 keys x W queries) = K . Q^T     (v_mfma_f32_32x32x16_bf16, or
//                                            16x16x32 twice)
//   O^T (d x W queries)      += V^T . P^T   (P as bf16 hi + lo parts; the
//                                            V^T operand by transposing LDS reads)
// with an online softmax per query (rescaled lazily).  A block visits only
// the key tiles that meet its queries' visible ranges -- the sink
// [0, C_sink) and the band from the smallest vis_start of its queries to
// its last query -- so tiles that PSAW masks for every query of the block
// are never loaded: that is the prefill work PSAW saves.  Inside the block a
// wave skips the keys masked for all of its queries and takes the
// per-(key, query) mask only where some of its queries see them in part.
//
// What bounds it: power on long prompts, the longest block on short ones.
// 32 queries per wave halve the LDS reads per product of 16 (16 KB per 32
// keys): one prompt of 32 heads x 16384 at d 128 went from 6.4 to 5.8
// million cycles, while the clock under this load fell from 2.10 to 2.05 GHz:
// 2971 -> 2900 us in turn on one card, 1137 TFLOP/s issued with the
// probabilities' low part (a large plain bf16 product of normal data reached
// 1394 there, of zeros 1793).  32 heads x 4096 went from 246 to 204 us, two
// paged prompts of 12k under PSAW (8 key heads) from 2712 to 2495, 64 heads x
// 7777 at d 64 from 1026 to 749, 16 heads x 1122 from 48.5 to 25.6.  Short
// prompts on many units and single rounds of blocks keep the 16.  Two groups
// of waves held half a step apart by barriers (one group's products beside
// the other's softmax) took the same cycles; dot products for the remainders
// p - hi were slower, and raised issue priority for the products changed
// nothing.
#include <type_traits>

#include "prefill_plan.h"
#include "prhs_internal.h"

namespace prhs {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef short v4i16_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr float kLn2 = 0.69314718055994530942f;
constexpr float kLazyLog2 = 8.f;  // log2 of the largest probability between rescales

struct PrefillArgs {
  KvView kv;
  const __bf16* q;        // [B][Hq][T][D]
  int T;
  int qblock;             // queries per workgroup
  int qfirst;             // queries of a unit's first workgroup
  int group;              // units of an XCD worked through side by side
  int psaw;               // nonzero: row i attends [0, sink) U [first visible at i + 1, i]
  double psaw_f;          // Eq. psaw factor of the layer
  int sink;
  float scale_log2;
  float* out;             // [B][Hq][T][D]
  float* lse;             // [B][Hq][T] or null
};

// K tile in LDS: 16-byte chunk c of tile row r at slot c ^ (r mod D/8), so
// the whole-row writes and the MFMA-order reads (16 rows, one chunk each)
// hit distinct banks.
template <int D>
__device__ __forceinline__ int k_slot(int r, int c) {
  constexpr int CH = D / 8;
  return r * CH + (c ^ (r & (CH - 1)));
}

// Whole-row loads of tile rows [ks, ks + KT): each thread takes RPL 16-byte
// chunks of K and of V, at these element offsets.  Rows at or past n (the
// prompt) read row n - 1.  A paged cache resolves every row through the
// block table (a row outside the table's valid pages reads element 0 of the
// cache instead: no access outside it); there the row offsets of each tile
// come from LDS, where its first KT threads store them (one block-table read
// per row) two tiles ahead of the loads.
template <int D, int KT, int NT>
struct TileOffs {
  static constexpr int RPL = (KT * (D / 8) + NT - 1) / NT;  // chunks per thread
  int64_t e[RPL];
};
template <int D, int KT, int NT>
struct TileRegs {
  u32x4_t x[TileOffs<D, KT, NT>::RPL];
};

// This thread's chunks of the tile at rows [ks, ks + KT) of a
// contiguous cache.
template <int D, int KT, int NT>
__device__ __forceinline__ void tile_offsets(TileOffs<D, KT, NT>& off, int64_t unit_row0, int ks, int n) {
  constexpr int CH = D / 8;
#pragma unroll
  for (int j = 0; j < TileOffs<D, KT, NT>::RPL; ++j) {
    const int e = (int)threadIdx.x + j * NT;
    const int r = (e / CH) % KT, c = e % CH;
    off.e[j] = (unit_row0 + min(ks + r, n - 1)) * D + c * 8;
  }
}

// The same from the tile's row offsets in LDS (paged cache).
template <int D, int KT, int NT>
__device__ __forceinline__ void tile_offsets_lds(TileOffs<D, KT, NT>& off, const int64_t* rows) {
  constexpr int CH = D / 8;
#pragma unroll
  for (int j = 0; j < TileOffs<D, KT, NT>::RPL; ++j) {
    const int e = (int)threadIdx.x + j * NT;
    off.e[j] = rows[(e / CH) % KT] + (e % CH) * 8;
  }
}

// Element offset of the row of position min(pos, n - 1) of (b, kv head g) in
// a paged cache (element 0 for a position outside the table's valid pages:
// no access outside the cache).
__device__ __forceinline__ int64_t paged_row(const KvView& kv, int b, int g, int pos, int n) {
  const int64_t row = kv_row_offset(kv, b, g, min(pos, n - 1));
  return row < 0 ? 0 : row;
}

// This thread's chunks of a tile of K or V (`base`).
template <int D, int KT, int NT>
__device__ __forceinline__ void tile_load(TileRegs<D, KT, NT>& R, const void* base,
                                          const TileOffs<D, KT, NT>& off) {
  constexpr int CH = D / 8;
#pragma unroll
  for (int j = 0; j < TileOffs<D, KT, NT>::RPL; ++j) {
    const int e = (int)threadIdx.x + j * NT;
    if ((KT * CH) % NT != 0 && e >= KT * CH) break;
    R.x[j] = *(const u32x4_t*)((const __bf16*)base + off.e[j]);
  }
}

// V tile in LDS: row-major, 16-byte chunk c of tile row r at slot
// v_chunk(r, c) of its row, so that the transposing operand reads below (per
// 32 lanes 4 key rows x 64 bytes with 32 queries a wave, 8 x 32 with 16) hit
// distinct banks.  Rows 16 apart share the permutation.
template <int D, int W>
__device__ __forceinline__ int v_chunk(int r, int c) {
  if (W == 32) return D == 128 ? c ^ ((r & 3) << 2) : c ^ (((r >> 1) & 1) << 2);
  return D == 128 ? c ^ ((r & 7) << 1) : c ^ (((r >> 1) & 3) << 1);
}

template <int D, int KT, int NT, int W, bool V>
__device__ __forceinline__ void tile_store(const TileRegs<D, KT, NT>& R, u32x4_t* dst) {
  constexpr int CH = D / 8;
#pragma unroll
  for (int j = 0; j < TileOffs<D, KT, NT>::RPL; ++j) {
    const int e = (int)threadIdx.x + j * NT;
    if ((KT * CH) % NT != 0 && e >= KT * CH) break;
    const int r = e / CH, c = e % CH;
    dst[V ? r * CH + v_chunk<D, W>(r, c) : k_slot<D>(r, c)] = R.x[j];
  }
}

// Types of a wave of W = 32 or 16 queries: lane (col, grp) = (lane % W,
// lane / W) has its share of query col, the scores of W / 2 of 32 keys and
// its dims of each W-dim block of O^T.
template <int W>
struct Wave;
template <>
struct Wave<32> {
  typedef f32x16_t Scores;
  typedef f32x16_t Out;
};
template <>
struct Wave<16> {
  typedef f32x8_t Scores;
  typedef f32x4_t Out;
};

// Maximum over the 64 / W lanes of a query, by lane swaps: swapping a value
// with itself leaves a lane holding its own value and its partner's.
template <int W>
__device__ __forceinline__ float max_over_groups(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  if (W == 16) {
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
  }
  return v;
}

// Key of a 32-key sub-tile that score r of lane group grp belongs to.
template <int W>
__device__ __forceinline__ int score_key(int r, int grp) {
  return (W == 32 ? 8 : 16) * (r >> 2) + 4 * grp + (r & 3);
}

// K operand of one 32-key sub-tile.  W = 32: product kk takes dims 16 kk +
// 8 grp .. + 7 of key col; W = 16: product (h, kk) dims 32 kk + 8 grp .. + 7
// of key 16 h + col.
template <int D>
struct KFrag {
  u32x4_t x[D / 16];
};
// LDS slot of this lane's piece of product j.
template <int D, int W>
__device__ __forceinline__ int kfrag_slot(int row0, int j, int col, int grp) {
  if (W == 32) return k_slot<D>(row0 + col, 2 * j + grp);
  constexpr int KS = D / 32;
  return k_slot<D>(row0 + 16 * (j / KS) + col, 4 * (j % KS) + grp);
}
template <int D>
__device__ __forceinline__ void load_kfrag(KFrag<D>& K, const unsigned char* sk, const int (&off)[D / 16],
                                           int base) {
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) K.x[kk] = *(const u32x4_t*)(sk + off[kk] + base);
}

// Scores of the sub-tile against one wave's queries: S^T = K . Q^T, lane
// (col, grp) query col at keys score_key(r, grp).
template <int D, int W>
__device__ __forceinline__ typename Wave<W>::Scores tile_scores(const KFrag<D>& K, const bf16x8_t* qf) {
  if constexpr (W == 32) {
    f32x16_t acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, K.x[kk]), qf[kk], acc, 0, 0, 0);
    return acc;
  } else {
    f32x4_t acc[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      acc[h] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < D / 32; ++kk)
        acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, K.x[h * (D / 32) + kk]), qf[kk],
                                                         acc[h], 0, 0, 0);
    }
    return __builtin_shufflevector(acc[0], acc[1], 0, 1, 2, 3, 4, 5, 6, 7);
  }
}

// P^T of one sub-tile as bf16 hi + lo parts, in the K-index order of the
// products: product t takes r = 8t .. 8t + 7 of the lane's scores.
template <int W>
struct Probs {
  uint32_t hi[W / 4], lo[W / 4];
};

// The online softmax of one sub-tile (keys ks32 .. ks32 + 31): the
// per-(key, query) mask unless `full`, the running maximum, O and l rescaled
// where it rises, and the probabilities.
template <int D, int W>
__device__ __forceinline__ void tile_softmax(typename Wave<W>::Scores x, int ks32, int grp, int qi, bool qvalid,
                                             int my_vis, int sink, float scale_log2, bool full,
                                             float& m_run, float& l_run, typename Wave<W>::Out* o, Probs<W>& P) {
  if (!full) {
#pragma unroll
    for (int r = 0; r < W / 2; ++r) {
      const int p = ks32 + score_key<W>(r, grp);
      const bool vis = qvalid && p <= qi && (p < sink || p >= my_vis);
      x[r] = vis ? x[r] : -INFINITY;
    }
  }
  float mt = x[0];
#pragma unroll
  for (int r = 1; r < W / 2; ++r) mt = fmaxf(mt, x[r]);
  mt = max_over_groups<W>(mt);
  // lazy rescaling: the reference m_run (and with it O and l) moves only
  // when some query of the wave sees its maximum rise by more than 2^8, so
  // the probabilities stay below 2^8; O / l does not depend on the reference
  const float m_new = fmaxf(m_run, mt * scale_log2);
  if (__builtin_amdgcn_ballot_w64(m_new > m_run + kLazyLog2)) {
    const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
    m_run = m_new;
    l_run *= alpha;
#pragma unroll
    for (int blk = 0; blk < D / W; ++blk) o[blk] *= alpha;
  }
  // while m_run is -inf every score is -inf too: a finite reference makes
  // every probability 0 without a branch
  const float mref = m_run == -INFINITY ? 0.f : m_run;
  float psum = 0.f;
#pragma unroll
  for (int w = 0; w < W / 4; ++w) {
    const float p0 = __builtin_amdgcn_exp2f(fmaf(x[2 * w], scale_log2, -mref));
    const float p1 = __builtin_amdgcn_exp2f(fmaf(x[2 * w + 1], scale_log2, -mref));
    psum += p0 + p1;
    const uint32_t hp = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{p0, p1}, bf16x2_t));
    const float r0 = p0 - __uint_as_float(hp << 16);
    const float r1 = p1 - __uint_as_float(hp & 0xFFFF0000u);
    P.hi[w] = hp;
    P.lo[w] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{r0, r1}, bf16x2_t));
  }
  l_run += psum;
}

// V^T operand of one product.  W = 32: over keys 16t .. 16t + 15 of the
// sub-tile, block blk (32 dims) needs dim 32 blk + col at keys 16t + 4 grp +
// i and 16t + 8 + 4 grp + i, i = 0 .. 3; W = 16: over its 32 keys, dim 16 blk
// + col at keys 4 grp + i and 16 + 4 grp + i.  Two transposing LDS loads from
// the row-major tile: in each 16-lane group, lane 4e + q points at the 8-byte
// piece q of 16 dims of key row e, and the load hands lane c dim c at the
// four rows.
template <int D, int W>
struct VFrag {
  bf16x8_t x[D / W];
};
// Byte offset of this lane's piece of block blk, first of the two loads.
template <int D, int W>
__device__ __forceinline__ int vfrag_offset(int row0, int blk, int lane) {
  const int e = (lane >> 2) & 3, q = lane & 3, grp = lane / W, g1 = W == 32 ? (lane >> 4) & 1 : 0;
  const int r = row0 + 4 * grp + e;
  return r * (D * 2) + (q & 1) * 8 + 16 * v_chunk<D, W>(r, W / 8 * blk + 2 * g1 + (q >> 1));
}
template <int D, int W>
__device__ __forceinline__ void load_vfrag(VFrag<D, W>& V, const unsigned char* sv, const int (&off)[D / W],
                                           int base) {
#pragma unroll
  for (int blk = 0; blk < D / W; ++blk) {
    const unsigned char* vp = sv + off[blk] + base;
    const v4i16_t a0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) v4i16_t*)vp);
    const v4i16_t a1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) v4i16_t*)(vp + (W == 32 ? 8 : 16) * (D * 2)));
    V.x[blk] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7));
  }
}

// O^T += V^T P^T over the keys of one operand.
template <int D, int W>
__device__ __forceinline__ void tile_products(const VFrag<D, W>& V, const Probs<W>& P, int t, typename Wave<W>::Out* o) {
  const bf16x8_t phi = __builtin_bit_cast(bf16x8_t, make_uint4(P.hi[4 * t], P.hi[4 * t + 1], P.hi[4 * t + 2], P.hi[4 * t + 3]));
  const bf16x8_t plo = __builtin_bit_cast(bf16x8_t, make_uint4(P.lo[4 * t], P.lo[4 * t + 1], P.lo[4 * t + 2], P.lo[4 * t + 3]));
#pragma unroll
  for (int blk = 0; blk < D / W; ++blk) {
    if constexpr (W == 32) {
      o[blk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(V.x[blk], phi, o[blk], 0, 0, 0);
      o[blk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(V.x[blk], plo, o[blk], 0, 0, 0);
    } else {
      o[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(V.x[blk], phi, o[blk], 0, 0, 0);
      o[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(V.x[blk], plo, o[blk], 0, 0, 0);
    }
  }
}

template <int D, int W, int NS, bool PAGED>
__global__ __launch_bounds__(64 * waves_of(W)) __attribute__((amdgpu_waves_per_eu(waves_per_simd(D, W, NS, PAGED), waves_per_simd(D, W, NS, PAGED))))
void attn_prefill_bf16(PrefillArgs a) {
  constexpr int kThreads = 64 * waves_of(W);
  constexpr int QG = waves_of(W) / NS;      // waves that differ in queries
  constexpr int SUB = NS == 4 ? 1 : 2;      // 32-key sub-tiles per wave and tile
  constexpr int KT = 32 * NS * SUB;         // key rows per tile
  constexpr int KS = W == 32 ? D / 16 : D / 32;  // Q operands
  constexpr int DB = D / W;    // output blocks of W dims
  constexpr int CH = D / 8;    // 16-byte chunks per row
  __shared__ u32x4_t s_kv[4][KT * CH];  // K tiles, then V tiles
  u32x4_t (*s_k)[KT * CH] = s_kv, (*s_v)[KT * CH] = s_kv + 2;
  __shared__ float s_ml[NS > 1 ? (NS - 1) * QG : 1][2][64];
  __shared__ int s_vmin;
  __shared__ int64_t s_rows[2][PAGED ? KT : 1];  // paged: row offsets of upcoming tiles
  // blocks of qblock queries (at most W QG), the first of qfirst
  const int nqb = 1 + (max(a.T - a.qfirst, 0) + a.qblock - 1) / a.qblock;
  int bh, qb;
  block_of(a.kv.batch * a.kv.hq, nqb, a.group, (int)blockIdx.x, &bh, &qb);
  const int hq = a.kv.hq, G = hq / a.kv.hkv;
  const int b = bh / hq, h = bh % hq, g = h / G;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane % W, grp = lane / W;
  const int n = min(kv_seq_len(a.kv, b), a.T);  // prompt positions with a query
  const int QB = qb ? a.qblock : a.qfirst;
  const int q0 = qb ? a.qfirst + (qb - 1) * a.qblock : 0;
  // NS waves share their queries, each taking its part (kside) of every key
  // tile.  Waves w and w + 4 share a SIMD: there the sides of one query group,
  // or, in a block of at most half the groups, nothing.
  const bool thin = QB <= W * QG / 2;
  const int qwave = thin ? wave / NS : wave % QG, kside = thin ? wave % NS : wave / QG;
  const int qi = q0 + qwave * W + col;             // this lane's query position
  const size_t qrow = ((size_t)b * hq + h) * a.T;
  const int qlast = min(q0 + QB, n) - 1;      // last query of the block inside the prompt

  if (qlast < q0) {  // the whole block lies past the prompt: empty rows
    for (int e = tid; e < QB * D; e += kThreads) {
      const int i = q0 + e / D;
      if (i < a.T) a.out[(qrow + i) * D + e % D] = 0.f;
    }
    if (a.lse)
      for (int i = q0 + tid; i < min(q0 + QB, a.T); i += kThreads) a.lse[qrow + i] = -INFINITY;
    return;
  }

  // the block's key range: the sink, then the band from the smallest first
  // visible position of its queries to its last query
  const int sink_end = min(a.sink, qlast + 1);
  if (wave == 0) {
    int v = sink_end;
    if (a.psaw) {
      v = 0x7FFFFFFF;
      for (int i = q0 + lane; i <= qlast; i += 64) v = min(v, psaw_first_visible(a.psaw_f, a.sink, i + 1));
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off));
    }
    if (lane == 0) s_vmin = v;
  }
  // this lane's query and its first visible non-sink position
  const bool qvalid = qi <= qlast;
  const int my_vis = (a.psaw && qvalid) ? psaw_first_visible(a.psaw_f, a.sink, qi + 1) : 0;
  // a tile needs no mask for this wave when all of its queries lie in
  // the prompt, the tile ends at or before the first of them, and it lies
  // inside the sink or at or past the largest of their vis_start
  const int qw0 = q0 + W * qwave;
  const bool wave_all = qw0 + W - 1 <= qlast;
  int wvis = my_vis, wvmin = qvalid ? my_vis : 0x7FFFFFFF;
#pragma unroll
  for (int off = 1; off < W; off <<= 1) {
    wvis = max(wvis, __shfl_xor(wvis, off));
    wvmin = min(wvmin, __shfl_xor(wvmin, off));
  }
  // each lane group holds the wave's queries: the results are uniform
  wvis = __builtin_amdgcn_readfirstlane(wvis);
  wvmin = __builtin_amdgcn_readfirstlane(wvmin);
  // and it needs no work at all when it lies past the wave's last query or
  // between the sink and the smallest of their vis_start (every product
  // would be masked; skipping leaves O, m and l exactly as they are)
  const int wlast = qw0 <= qlast ? min(qw0 + W - 1, qlast) : -1;
  bf16x8_t qf[KS];
  {
    const __bf16* qp = a.q + (qrow + (qvalid ? qi : q0)) * D + grp * 8;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) qf[kk] = __builtin_bit_cast(bf16x8_t, *(const uint4*)(qp + 512 / W * kk));
  }
  __syncthreads();
  const int band_lo = min(max(s_vmin, sink_end), qlast + 1);
  const int nsink = (sink_end + KT - 1) / KT;
  const int tb0 = max(nsink, band_lo / KT), tb1 = qlast / KT;
  const int ntiles = nsink + (tb1 >= tb0 ? tb1 - tb0 + 1 : 0);

  const int64_t row0 = ((int64_t)b * a.kv.hkv + g) * a.kv.capacity;
  float m_run = -INFINITY, l_run = 0.f;
  typename Wave<W>::Out o[DB];
#pragma unroll
  for (int i = 0; i < DB; ++i)
#pragma unroll
    for (int r = 0; r < W * W / 64; ++r) o[i][r] = 0.f;

  auto tile_start = [&](int t) { return (t < nsink ? t : tb0 + (t - nsink)) * KT; };
  auto full_tile = [&](int ks) {
    return wave_all && ks + 32 * SUB - 1 <= qw0 && (ks + 32 * SUB <= a.sink || ks >= wvis);
  };
  auto masked_tile = [&](int ks) {
    return ks > wlast || (ks >= a.sink && ks + 32 * SUB - 1 < wvmin);
  };
  TileOffs<D, KT, kThreads> offs;
  TileRegs<D, KT, kThreads> rk, rv;
  auto rows_of = [&](int t) { return paged_row(a.kv, b, g, tile_start(max(min(t, ntiles - 1), 0)) + tid, n); };
  auto offsets = [&](int t) {
    if constexpr (PAGED) tile_offsets_lds<D, KT, kThreads>(offs, s_rows[t & 1]);
    else tile_offsets<D, KT, kThreads>(offs, row0, tile_start(max(min(t, ntiles - 1), 0)), n);
  };
  if (PAGED) {
    if (tid < KT) {
      s_rows[0][tid] = rows_of(0);
      s_rows[1][tid] = rows_of(1);
    }
    __syncthreads();
  }
  offsets(0);
  tile_load<D, KT, kThreads>(rk, a.kv.k, offs);
  tile_load<D, KT, kThreads>(rv, a.kv.v, offs);
  offsets(1);
  // LDS byte offsets of this lane's operand pieces, fixed for the launch:
  // with the buffer a constant of the code below, an operand read costs no
  // address arithmetic
  int koff[D / 16], voff[DB];
#pragma unroll
  for (int j = 0; j < D / 16; ++j) koff[j] = 16 * kfrag_slot<D, W>(32 * SUB * kside, j, col, grp);
#pragma unroll
  for (int blk = 0; blk < DB; ++blk) voff[blk] = vfrag_offset<D, W>(32 * SUB * kside, blk, lane);
  int64_t prow = 0;
  auto step = [&](auto buf, int t) {
    constexpr int BUF = decltype(buf)::value;
    constexpr int kTileBytes = KT * D * 2;
    tile_store<D, KT, kThreads, W, false>(rk, s_k[BUF]);
    tile_store<D, KT, kThreads, W, true>(rv, s_v[BUF]);
    lds_barrier();
    // paged: the table read is issued before the tile loads, so waiting for
    // it later does not wait for them
    if (PAGED && tid < KT) prow = rows_of(t + 2);
    if (PAGED) offsets(t + 1);
    tile_load<D, KT, kThreads>(rk, a.kv.k, offs);  // tile t + 1 (the last one again at the end)
    tile_load<D, KT, kThreads>(rv, a.kv.v, offs);
    if (!PAGED) offsets(t + 2);
    const int ks = tile_start(t) + 32 * SUB * kside;  // this wave's keys of the tile
    if (!masked_tile(ks)) {
      const bool full = full_tile(ks);
#pragma unroll
      for (int i = 0; i < SUB; ++i) {
        KFrag<D> kf;
        Probs<W> P;
        VFrag<D, W> v;
        load_kfrag<D>(kf, (const unsigned char*)s_kv, koff, BUF * kTileBytes + 32 * i * D * 2);
        const auto x = tile_scores<D, W>(kf, qf);
        tile_softmax<D, W>(x, ks + 32 * i, grp, qi, qvalid, my_vis, a.sink, a.scale_log2, full, m_run,
                           l_run, o, P);
#pragma unroll
        for (int w = 0; w < W / 16; ++w) {
          load_vfrag<D, W>(v, (const unsigned char*)s_kv + 2 * kTileBytes, voff,
                           BUF * kTileBytes + (32 * i + 16 * w) * D * 2);
          tile_products<D, W>(v, P, w, o);
        }
      }
    }
    if (PAGED && tid < KT) s_rows[t & 1][tid] = prow;  // tile t + 2, read after the next barrier
  };
  for (int t = 0; t < ntiles; t += 2) {
    step(std::integral_constant<int, 0>{}, t);
    if (t + 1 < ntiles) step(std::integral_constant<int, 1>{}, t + 1);
  }
  if constexpr (NS > 1) {
    // combine the key sides: the others hand (m, l, O) to side 0 through LDS
    lds_barrier();  // the tiles are read
    float* so = (float*)&s_kv[0][0] + lane;
    if (kside) {
      const int j = (kside - 1) * QG + qwave;
#pragma unroll
      for (int blk = 0; blk < DB; ++blk)
#pragma unroll
        for (int r = 0; r < 16; ++r) so[((j * DB + blk) * 16 + r) * 64] = o[blk][r];
      s_ml[j][0][lane] = m_run;
      s_ml[j][1][lane] = l_run;
    }
    lds_barrier();
    if (kside) return;
    float m1[NS - 1], M = m_run;
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) M = fmaxf(M, m1[s] = s_ml[s * QG + qwave][0][lane]);
    const float mr = M == -INFINITY ? 0.f : M;
    const float f0 = __builtin_amdgcn_exp2f(m_run - mr);
    m_run = M;
    l_run *= f0;
#pragma unroll
    for (int blk = 0; blk < DB; ++blk) o[blk] *= f0;
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) {
      const int j = s * QG + qwave;
      const float f = __builtin_amdgcn_exp2f(m1[s] - mr);
      l_run += f * s_ml[j][1][lane];
#pragma unroll
      for (int blk = 0; blk < DB; ++blk)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[blk][r] += f * so[((j * DB + blk) * 16 + r) * 64];
    }
  }

  // lane (col, grp) holds dims W blk + 8 j + 4 grp .. + 3 of query col
  if (W == 16) l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
  if (qi < min(q0 + QB, a.T)) {
    float* op = a.out + (qrow + qi) * D + 4 * grp;
    const float inv = (qvalid && l_run > 0.f) ? 1.f / l_run : 0.f;
#pragma unroll
    for (int blk = 0; blk < DB; ++blk)
#pragma unroll
      for (int j = 0; j < W * W / 256; ++j)
        *(float4*)(op + W * blk + 8 * j) = make_float4(o[blk][4 * j] * inv, o[blk][4 * j + 1] * inv,
                                                       o[blk][4 * j + 2] * inv, o[blk][4 * j + 3] * inv);
    if (a.lse && grp == 0)
      a.lse[qrow + qi] = (qvalid && l_run > 0.f) ? (m_run + log2f(l_run)) * kLn2 : -INFINITY;
  }
}

}  // namespace

hipError_t launch_prefill(const PrefillLaunch& s, hipStream_t stream) {
  if (s.kv.batch == 0 || s.T == 0) return hipSuccess;
  PrefillArgs a;
  a.kv = s.kv;
  a.q = (const __bf16*)s.q;
  a.T = s.T;
  a.psaw = s.psaw;
  a.psaw_f = s.psaw_f;
  a.sink = s.sink;
  a.scale_log2 = s.scale * 1.44269504088896340736f;
  a.out = s.out;
  a.lse = s.lse;
  const long long units = (long long)s.kv.batch * s.kv.hq;
  const int cus = device_cus();
  const PrefillPlan plan = plan_of({s.T, s.kv.d, s.kv.paged, s.psaw, s.psaw_f, s.sink}, units, cus);
  const int nqb = plan.blocks(s.T);
  a.qblock = plan.qblock;
  a.qfirst = plan.qfirst;
  a.group = unit_group((int)(units / kXcds), nqb, cus);
  const dim3 grid((unsigned)(nqb * units));
#define PRHS_PREFILL_GO(DV, W, NS, PG) \
  hipLaunchKernelGGL((attn_prefill_bf16<DV, W, NS, PG>), grid, dim3(64 * waves_of(W)), 0, stream, a)
#define PRHS_PREFILL_LAUNCH(DV, PG)                        \
  do {                                                     \
    if (plan.w == 16) PRHS_PREFILL_GO(DV, 16, 1, PG);      \
    else if (plan.ns == 1) PRHS_PREFILL_GO(DV, 32, 1, PG); \
    else if (plan.ns == 2) PRHS_PREFILL_GO(DV, 32, 2, PG); \
    else PRHS_PREFILL_GO(DV, 32, 4, PG);                   \
  } while (0)
  if (s.kv.d == 128) {
    if (s.kv.paged) PRHS_PREFILL_LAUNCH(128, true);
    else PRHS_PREFILL_LAUNCH(128, false);
  } else {
    if (s.kv.paged) PRHS_PREFILL_LAUNCH(64, true);
    else PRHS_PREFILL_LAUNCH(64, false);
  }
#undef PRHS_PREFILL_LAUNCH
#undef PRHS_PREFILL_GO
  return hipGetLastError();
}

}  // namespace prhs
