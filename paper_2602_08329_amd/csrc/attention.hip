// Decode attention over a per-kv-head index set (token-sparse attention,
// Def. 3.1) or over every cached key (Eq. attn_eq), split-K:
//
// attn_split_*: one workgroup per (unit, split) handles a contiguous chunk of
// the unit's index list: it gathers K/V rows, computes scaled logits and keeps
// an online softmax (running max m, running sum l, unnormalised output o).  A
// unit that fits one split writes its output directly; otherwise each split
// stores (m, l, o) and
// attn_merge: one workgroup per query head of a split unit combines them in
// split order,
//   y = sum_s 2^(m_s - M) o_s / sum_s 2^(m_s - M) l_s,
//   lse = ln 2 * (M + log2 sum_s 2^(m_s - M) l_s).
// The merge is a launch of its own: merging inside the split kernel would need
// device-scope fences, which on this chip write back and invalidate a whole
// L2 slice per workgroup.
//
// Latency: the workgroup first resolves every list entry of its chunk to a
// physical row id (the set entries load together with the unit's lengths,
// then block-table loads for paged caches) and stages the ids in LDS.  Waves
// then walk 32-row tiles with two register buffers: the K/V loads of the next
// tile are in flight while the current tile is multiplied.  Loads are issued
// unconditionally (a missing row reads row 0) and invalid rows are masked
// afterwards, so no load waits on a branch.
//
// bf16 inputs use MFMA for both products of a wave's 32-row tile:
//   S^T (32 keys x 16 heads) = K_tile . Q^T  (v_mfma_f32_16x16x32_bf16, two 16-row halves)
//   O^T (d x 16 heads)      += V_tile^T . P^T, P split into bf16 hi + lo parts so
//                              the probabilities keep ~16 significant bits.
// Every K and V load reads whole rows (d/8 lanes of 16 bytes per row), the
// pattern that sustains full bandwidth per CU; the MFMA operand order of K
// (4 lanes per key) would read 64-byte pieces of 16 rows per load, which
// this chip serves at well under half that rate.  K therefore goes through
// a per-wave LDS tile (XOR-swizzled, conflict-free both ways) into operand
// order; the dimension order inside a row is permuted identically on K and
// Q.  V needs no transpose: a lane's 8 rows x 8 dims block feeds the second
// product directly.  K and V bytes are read once, with the streaming policy.
// fp32 inputs take a vector-ALU path (d/4 lanes per row, up to eight of a unit's
// query heads in one workgroup).
#include <stdlib.h>

#include <algorithm>
#include <mutex>

#include "prhs_internal.h"

namespace prhs {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr float kLn2 = 0.69314718055994530942f;
constexpr int kRowsPerThread = 8;   // staged list entries per thread
constexpr int kMaxSplits = 4096;
constexpr int kMaxWaves = 8;        // waves of an attention workgroup
// Sparse sets of at most this many rows per unit are not split: a launch of
// one workgroup per unit beats a split launch plus its merge launch (fp32
// rows are twice as long: 32 units of 500 rows 20.7 us unsplit, 13.4 split; 4
// units of 150 rows 5.6 and 7.9).  Dense fp32 streams the same; up to
// kNoSplitManyF32 rows where kManyF32 units keep the chip busy (64 units of 16
// heads over 146 rows at d 128 19.4 us in three splits, 11.4 unsplit, 48 of 338
// 25.6 and 17.8); up to kNoSplitMostF32 where kMostF32 do (160 of 16 over 490 at
// d 64 39.6 and 27.5, 200 of 4 over 700 46 and 29.9, 160 of 1 over 1120 23 and
// 18; but 160 of 8 over 1989 89 and 102, 96 of 4 over 879 16.6 and 18.3); and
// fewer where few units have many heads (kNoSplitHeadRowsF32 rows times heads: 12
// units of 16 heads over 219 rows 10.0 us in four splits, 11.6 unsplit; 32 of 8
// over 203 9.0 and 7.4).
constexpr int kNoSplitRows = 512;
constexpr int kNoSplitRowsF32 = 256;
constexpr int kNoSplitManyF32 = 450, kManyF32 = 40;
constexpr int kNoSplitMostF32 = 1200, kMostF32 = 128;
constexpr int kNoSplitHeadRowsF32 = 2048;
// fp32 splits: at least kMinRowsF32 rows (half of that where the splits of all
// heads are fewer than kFewHeadsF32: one unit of 8 heads over 377 rows 8.7 -> 7.6,
// 4 of 16 over 178 9.3 -> 8.5 us), and no more than kMergeSplitsF32 of them per
// unit once the launch has 256 workgroups, since the merge reads every split's
// output of every head (dense, 8 units of 4 heads at d 128: 2000 rows in 125
// splits 18.3 us, in 32 13.6; 8000 rows in 125 26.5, in 32 19.8).
constexpr int kMinRowsF32 = 64;
constexpr long long kFewHeadsF32 = 256;
constexpr long long kMergeSplitsF32 = 32;

struct AttnArgs {
  KvView kv;
  const void* q;
  const int32_t* set_idx;
  const int32_t* set_len;
  const int32_t* tail_start;  // [B] or null: rows also cover [tail_start[b], n_b)
  const int32_t* unit_row;    // [units] or null: pool row of set_idx each unit attends
  const int32_t* unit_tail;   // [units] with unit_row: first position of the unit's tail
  int pool_rows;
  const int32_t* unit_gate;   // [units] or null: the gate's choice per unit
  int units_side;             // 1: only units with unit_gate < 0; 2: only >= 0; else all
  int psaw;                   // nonzero: positions in [psaw_sink, first visible) are skipped
  double psaw_f;              // Eq. psaw factor of the layer (first visible at length n:
  int psaw_sink;              // psaw_first_visible(psaw_f, psaw_sink, n))
  int set_cap;
  float scale_log2;
  int chunk, nsplit;
  float* part_o;    // [B*Hq][nsplit][D]
  float* part_ml;   // [B*Hq][nsplit][2]
  float* out;
  float* lse;
};

// The rows a unit attends, in order: the first `base` come from its index
// set (entries at or beyond t0 are skipped), then the tail positions
// [t0, t0 + L - base).  Dense: rows are the positions [0, n_b).  Without a
// tail t0 = n_b.  L never exceeds set_cap, the bound the split geometry uses.
// The set is row u of set_idx, or with a pool the row unit_row[u] (a row
// outside the pool gives an empty set) and the tail from unit_tail[u].
struct UnitSpan {
  int L, base, t0;
  int mask_lo, mask_hi;  // rows at positions in [mask_lo, mask_hi) are skipped (PSAW)
};

template <bool DENSE>
__device__ __forceinline__ UnitSpan unit_span(const AttnArgs& a, int u, int b, int nb) {
  UnitSpan sp;
  sp.t0 = nb;
  sp.mask_lo = sp.mask_hi = 0;
  if (DENSE) {
    sp.L = sp.base = nb;
    return sp;
  }
  if (a.psaw) {
    sp.mask_lo = a.psaw_sink;
    sp.mask_hi = psaw_first_visible(a.psaw_f, a.psaw_sink, nb);
  }
  int row = u, t0 = nb;
  bool tail = false;
  if (a.unit_row) {
    row = a.unit_row[u];
    t0 = a.unit_tail[u];
    tail = true;
    if (row < 0 || row >= a.pool_rows) {
      sp.L = sp.base = 0;
      return sp;
    }
  } else if (a.tail_start) {
    t0 = a.tail_start[b];
    tail = true;
  }
  int L = a.set_len[row];
  L = L < 0 ? 0 : (L > a.set_cap ? a.set_cap : L);
  sp.base = L;
  if (tail) {
    t0 = t0 < 0 ? 0 : (t0 > nb ? nb : t0);
    sp.t0 = t0;
    L += nb - t0;
    L = L > a.set_cap ? a.set_cap : L;
  }
  sp.L = L;
  return sp;
}

// Units a launch leaves alone (their outputs untouched): with a side filter,
// the ones on the other side of the gate's decision.
__device__ __forceinline__ bool unit_excluded(const AttnArgs& a, int u) {
  if (!a.unit_gate || (a.units_side != 1 && a.units_side != 2)) return false;
  const bool retrieving = a.unit_gate[u] < 0;
  return a.units_side == 1 ? !retrieving : retrieving;
}

// Row id (element offset / d) of position pos of (b, kv head g), or -1 when
// the position lies outside [0, nb) or outside the cache.
template <bool PAGED>
__device__ __forceinline__ int32_t phys_row(const KvView& kv, int b, int g, int pos, int nb) {
  if (pos < 0 || pos >= nb) return -1;
  if (!PAGED) {
    if (pos >= kv.capacity) return -1;
    return (b * kv.hkv + g) * kv.capacity + pos;
  }
  const int page = pos / kv.page_size;
  if (page >= kv.max_pages) return -1;
  const int phys = kv.table[(int64_t)b * kv.max_pages + page];
  if (phys < 0 || phys >= kv.num_pages) return -1;
  return (phys * kv.hkv + g) * kv.page_size + (pos - page * kv.page_size);
}

// Loads the set entries [start, start + chunk) of unit u before the unit's
// length is known, so that these loads share one memory latency with the
// length loads.  Entries at or past the length are loaded and never used; a
// set row holds set_cap entries, so every load stays inside it.
template <bool DENSE>
__device__ __forceinline__ void prefetch_entries(const AttnArgs& a, int u, int start,
                                                 int32_t (&raw)[kRowsPerThread]) {
#pragma unroll
  for (int k = 0; k < kRowsPerThread; ++k) raw[k] = -1;
  if (DENSE) return;
  int row = u;
  bool ok = true;
  if (a.unit_row) {
    row = a.unit_row[u];
    ok = row >= 0 && row < a.pool_rows;
  }
  const int32_t* idx = a.set_idx + (size_t)(ok ? row : 0) * a.set_cap;
  const int lim = min(start + a.chunk, a.set_cap);
#pragma unroll
  for (int k = 0; k < kRowsPerThread; ++k) {
    const int t = start + (int)threadIdx.x + k * (int)blockDim.x;
    if (ok && t < lim) raw[k] = idx[t];
  }
}

// Resolves list entries [start, start + n) of the unit to row ids in s_row,
// from the entries prefetch_entries loaded; for a paged cache all block-table
// loads of a thread are issued before any is used.  n <= blockDim * 8.
template <bool DENSE, bool PAGED>
__device__ __forceinline__ void stage_rows(const AttnArgs& a, const int32_t (&raw)[kRowsPerThread],
                                           int start, int n, const UnitSpan& sp, int nb, int b,
                                           int g, int32_t* s_row) {
  int pos[kRowsPerThread];
#pragma unroll
  for (int k = 0; k < kRowsPerThread; ++k) {
    const int r = threadIdx.x + k * blockDim.x;
    const int t = start + r;
    pos[k] = -1;
    if (r < n) {
      if (DENSE) {
        pos[k] = t;
      } else {
        int p;
        if (t < sp.base) {
          p = raw[k];
          p = p < sp.t0 ? p : -1;
        } else {
          p = sp.t0 + (t - sp.base);
        }
        pos[k] = (p >= sp.mask_lo && p < sp.mask_hi) ? -1 : p;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < kRowsPerThread; ++k) {
    const int r = threadIdx.x + k * blockDim.x;
    if (r < n) s_row[r] = phys_row<PAGED>(a.kv, b, g, pos[k], nb);
  }
  __syncthreads();
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// Maximum over the lanes col, col + 16, col + 32 and col + 48 (the four
// lane groups of one MFMA column), by the cross-half and cross-row lane
// swaps: each swap of a value with itself leaves a lane holding its own
// value and its partner's, one in each result.
__device__ __forceinline__ float max_over_groups(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Maximum over all 64 lanes, in every lane: rotations by 8, 4, 2 and 1
// inside each row of 16 lanes (DPP row_ror), then across the four rows.
__device__ __forceinline__ float wave_max(float v) {
#define PRHS_ROR_MAX(CTRL)                                                                    \
  v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), \
                                                          CTRL, 0xF, 0xF, false)))
  PRHS_ROR_MAX(0x128);  // row_ror:8
  PRHS_ROR_MAX(0x124);  // row_ror:4
  PRHS_ROR_MAX(0x122);  // row_ror:2
  PRHS_ROR_MAX(0x121);  // row_ror:1
#undef PRHS_ROR_MAX
  return max_over_groups(v);
}

// Sum over the same four lanes.
__device__ __forceinline__ float sum_over_groups(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

template <int DB>
struct VRow;
template <>
struct VRow<8> {  // d = 128: 8 bf16 per lane per row
  uint32_t w[4];
};
template <>
struct VRow<4> {  // d = 64: 4 bf16 per lane per row
  uint32_t w[2];
};

template <int DB>
__device__ __forceinline__ VRow<DB> load_vrow(const __bf16* p) {
  VRow<DB> v;
  if constexpr (DB == 8) {
    const u32x4_t x = stream_load16(p);
    v.w[0] = x[0]; v.w[1] = x[1]; v.w[2] = x[2]; v.w[3] = x[3];
  } else {
    const u32x2_t x = stream_load8(p);
    v.w[0] = x[0]; v.w[1] = x[1];
  }
  return v;
}


// Registers of one wave's 32-row tile: K rows as loaded (whole rows, D/8
// lanes of 16 bytes per row, so every load reads whole 128-byte lines), V
// rows (16s + 4 grp + j) and the validity of the V rows, which are also the
// rows of the lane's logits.
template <int D>
struct Tile {
  static constexpr int KS = D / 32;  // products per 16-row half = K loads per half
  static constexpr int DB = D / 16;
  u32x4_t kraw[2][KS];
  VRow<DB> vf[2][4];
  uint32_t ok;
};

// K staging in LDS: a wave's 32 x D tile, row-major in 16-byte chunks, chunk
// c of tile row r at slot c ^ (r mod D/8), so that both the row-wise writes
// and the MFMA-order reads (16 rows, one chunk each) hit distinct banks.
template <int D>
__device__ __forceinline__ int kst_slot(int r, int c) {
  constexpr int CH = D / 8;
  return r * CH + (c ^ (r & (CH - 1)));
}

// LDS bytes per wave: its K staging tile, reused at the end for its G output
// rows of D + 1 floats.
__host__ __device__ constexpr int attn_wave_bytes(int D, int G) {
  return ((32 * D * 2 > G * (D + 1) * 4 ? 32 * D * 2 : G * (D + 1) * 4) + 15) & ~15;
}

template <int D>
__device__ __forceinline__ void load_tile(Tile<D>& T, const int32_t* s_row, int r0, int n,
                                          const __bf16* kb, const __bf16* vb, int lane) {
  constexpr int KS = D / 32;
  constexpr int DB = D / 16;
  constexpr int CH = D / 8, RPI = 64 / CH;  // chunks per row, rows per K load
  const int col = lane & 15, grp = lane >> 4;
  const int kc = lane % CH, kr = lane / CH;
  // all row ids of the tile first (unconditional LDS reads: s_row spans whole
  // tiles), then every load, so that no load waits on a single LDS read
  int rk[2][KS], rv[2][4];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
#pragma unroll
    for (int j = 0; j < KS; ++j) {
      const int r = r0 + 16 * s + j * RPI + kr;
      const int x = s_row[r];
      rk[s][j] = r < n ? x : -1;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = r0 + 16 * s + grp * 4 + j;
      const int x = s_row[r];
      rv[s][j] = r < n ? x : -1;
    }
  }
  T.ok = 0u;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
#pragma unroll
    for (int j = 0; j < KS; ++j)
      T.kraw[s][j] = stream_load16(kb + (int64_t)(rk[s][j] < 0 ? 0 : rk[s][j]) * D + kc * 8);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      T.vf[s][j] = load_vrow<DB>(vb + (int64_t)(rv[s][j] < 0 ? 0 : rv[s][j]) * D + col * DB);
      if (rv[s][j] >= 0) T.ok |= 1u << (s * 4 + j);
    }
  }
}

// Online-softmax state of one wave: lane (col, grp) owns query head col and
// output dims grp * d/4 .. (grp + 1) * d/4 - 1 via the o[] accumulators.
template <int D>
struct WaveState {
  float m, l;
  f32x4_t o[D / 16];
};

template <int D>
__device__ __forceinline__ void consume_tile(Tile<D>& T, WaveState<D>& st, const bf16x8_t* qf,
                                             float scale_log2, u32x4_t* kst, int lane) {
  constexpr int KS = D / 32;
  constexpr int DB = D / 16;
  constexpr int CH = D / 8, RPI = 64 / CH;
  const int col = lane & 15, grp = lane >> 4;
  // K rows to MFMA operand order through the wave's LDS tile: lane (col,
  // grp) takes dims 32kk + 8grp .. +7 of tile row 16s + col for product kk.
  // LDS operations of one wave complete in order; the wave barriers keep
  // the compiler from moving them across each other.
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int j = 0; j < KS; ++j) kst[kst_slot<D>(16 * s + j * RPI + lane / CH, lane % CH)] = T.kraw[s][j];
  __builtin_amdgcn_wave_barrier();
  bf16x8_t kf[2][KS];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
      kf[s][kk] = __builtin_bit_cast(bf16x8_t, kst[kst_slot<D>(16 * s + col, 4 * kk + grp)]);
  __builtin_amdgcn_wave_barrier();
  float x[2][4];
  float mt = -INFINITY;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[s][kk], qf[kk], acc, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool ok = (T.ok >> (s * 4 + e)) & 1u;
      x[s][e] = ok ? acc[e] * scale_log2 : -INFINITY;
      mt = fmaxf(mt, x[s][e]);
    }
  }
  // rows past the set read a stand-in row: zero their V values (a zero
  // probability times a non-finite value would still be NaN), only in the
  // waves that have such rows
  if (__builtin_amdgcn_ballot_w64(T.ok != 0xFFu)) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (!((T.ok >> (s * 4 + e)) & 1u)) {
#pragma unroll
          for (int w = 0; w < DB / 2; ++w) T.vf[s][e].w[w] = 0u;
        }
  }
  mt = max_over_groups(mt);
  // lazy rescaling: the reference st.m (and with it o and l) moves only when
  // some head of the wave sees its maximum rise by more than 2^8, so the
  // probabilities stay below 2^8; o / l does not depend on the reference
  const float m_new = fmaxf(st.m, mt);
  if (__builtin_amdgcn_ballot_w64(m_new > st.m + 8.f)) {
    const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(st.m - m_new);
    st.m = m_new;
    st.l *= alpha;
#pragma unroll
    for (int blk = 0; blk < DB; ++blk) st.o[blk] *= alpha;
  }
  // while st.m is -inf every score is -inf too: a finite reference makes
  // every probability 0 without a branch
  const float mref = st.m == -INFINITY ? 0.f : st.m;
  float psum = 0.f;
  uint32_t hi[4], lo[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const int j0 = 2 * w, j1 = 2 * w + 1;
    const float p0 = __builtin_amdgcn_exp2f(x[j0 >> 2][j0 & 3] - mref);
    const float p1 = __builtin_amdgcn_exp2f(x[j1 >> 2][j1 & 3] - mref);
    psum += p0 + p1;
    const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{p0, p1}, bf16x2_t));
    hi[w] = h;
    lo[w] = __builtin_bit_cast(uint32_t, __builtin_convertvector(
        f32x2_t{p0 - __uint_as_float(h << 16), p1 - __uint_as_float(h & 0xFFFF0000u)}, bf16x2_t));
  }
  st.l += psum;
  const bf16x8_t phi = __builtin_bit_cast(bf16x8_t, make_uint4(hi[0], hi[1], hi[2], hi[3]));
  const bf16x8_t plo = __builtin_bit_cast(bf16x8_t, make_uint4(lo[0], lo[1], lo[2], lo[3]));
#pragma unroll
  for (int blk = 0; blk < DB; ++blk) {
    uint32_t aw[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int j0 = 2 * w, j1 = 2 * w + 1;
      // element blk of rows j0 (low half) and j1 (high half), one byte
      // permute: selector bytes 0-3 index the second source, 4-7 the first
      aw[w] = __builtin_amdgcn_perm(T.vf[j1 >> 2][j1 & 3].w[blk >> 1], T.vf[j0 >> 2][j0 & 3].w[blk >> 1],
                                    (blk & 1) ? 0x07060302u : 0x05040100u);
    }
    const bf16x8_t av = __builtin_bit_cast(bf16x8_t, make_uint4(aw[0], aw[1], aw[2], aw[3]));
    st.o[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, phi, st.o[blk], 0, 0, 0);
    st.o[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, plo, st.o[blk], 0, 0, 0);
  }
}

// Writes out/lse of query head bh from (M, sum, unnormalised numerator).
__device__ __forceinline__ void write_final(const AttnArgs& a, size_t bh, int D, int dim, float M,
                                            float num, float den) {
  a.out[bh * D + dim] = den > 0.f ? num / den : 0.f;
  if (a.lse && dim == 0) a.lse[bh] = den > 0.f ? (M + log2f(den)) * kLn2 : -INFINITY;
}

template <int D, bool DENSE, bool PAGED>
__global__ __launch_bounds__(512) void attn_split_bf16(AttnArgs a) {
  constexpr int KS = D / 32;
  constexpr int DB = D / 16;
  // dynamic LDS: [nwaves][attn_wave_bytes] wave regions (K staging, then the
  // wave's outputs), then the staged row ids [blockDim * kRowsPerThread]
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  __shared__ float sm_m[8][16];
  __shared__ float sm_l[8][16];
  const int split = blockIdx.x, u = blockIdx.y;
  const int hkv = a.kv.hkv, hq = a.kv.hq, G = hq / hkv;
  const int wbytes = attn_wave_bytes(D, G);
  int32_t* s_row = (int32_t*)(dyn + (size_t)(blockDim.x >> 6) * wbytes);
  const int b = u / hkv, g = u % hkv;
  const int start = split * a.chunk;
  const int nwaves = blockDim.x >> 6;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 15, grp = lane >> 4;
  // set entries, query and lengths load together
  int32_t raw[kRowsPerThread];
  prefetch_entries<DENSE>(a, u, start, raw);
  const __bf16* qb = (const __bf16*)a.q;
  bf16x8_t qf[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    const int qh = col < G ? col : 0;
    const uint4* qp = (const uint4*)(qb + ((size_t)b * hq + g * G + qh) * D + grp * 8);
    const uint4 v = qp[4 * kk];
    qf[kk] = __builtin_bit_cast(bf16x8_t, col < G ? v : make_uint4(0, 0, 0, 0));
  }
  const int nb = kv_seq_len(a.kv, b);
  if (!DENSE && unit_excluded(a, u)) return;
  const UnitSpan sp = unit_span<DENSE>(a, u, b, nb);
  const int L = sp.L;
  if (L == 0 && split == 0) {  // empty set: y = 0, lse = -inf
    for (int e = threadIdx.x; e < G * D; e += blockDim.x)
      write_final(a, (size_t)b * hq + g * G + e / D, D, e % D, -INFINITY, 0.f, 0.f);
    return;
  }
  if (start >= L) return;
  const int n = min(L, start + a.chunk) - start;
  stage_rows<DENSE, PAGED>(a, raw, start, n, sp, nb, b, g, s_row);

  const __bf16* kb = (const __bf16*)a.kv.k;
  const __bf16* vb = (const __bf16*)a.kv.v;
  WaveState<D> st;
  st.m = -INFINITY;
  st.l = 0.f;
#pragma unroll
  for (int i = 0; i < DB; ++i) st.o[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // this wave's tiles: wave, wave + nwaves, ...; the steady-state body always
  // has a next tile, so its prefetch is unconditional and the compiler can
  // wait for the current buffer only
  const int ntiles = (n + 31) >> 5;
  const int iters = wave < ntiles ? (ntiles - wave + nwaves - 1) / nwaves : 0;
  if (iters > 0) {
    Tile<D> A, B;
    u32x4_t* kst = (u32x4_t*)(dyn + (size_t)wave * wbytes);
    const int step = 32 * nwaves;
    int r0 = wave * 32;
    load_tile<D>(A, s_row, r0, n, kb, vb, lane);
    int i = 0;
    for (; i + 2 < iters; i += 2) {
      load_tile<D>(B, s_row, r0 + step, n, kb, vb, lane);
      consume_tile<D>(A, st, qf, a.scale_log2, kst, lane);
      load_tile<D>(A, s_row, r0 + 2 * step, n, kb, vb, lane);
      consume_tile<D>(B, st, qf, a.scale_log2, kst, lane);
      r0 += 2 * step;
    }
    if (i + 1 < iters) {
      load_tile<D>(B, s_row, r0 + step, n, kb, vb, lane);
      consume_tile<D>(A, st, qf, a.scale_log2, kst, lane);
      consume_tile<D>(B, st, qf, a.scale_log2, kst, lane);
    } else {
      consume_tile<D>(A, st, qf, a.scale_log2, kst, lane);
    }
  }

  st.l = sum_over_groups(st.l);
  if (grp == 0) {
    sm_m[wave][col] = st.m;
    sm_l[wave][col] = st.l;
  }
  if (col < G) {
    float* wo = (float*)(dyn + (size_t)wave * wbytes) + col * (D + 1);
#pragma unroll
    for (int blk = 0; blk < DB; ++blk)
#pragma unroll
      for (int i = 0; i < 4; ++i) wo[(grp * 4 + i) * DB + blk] = st.o[blk][i];
  }
  __syncthreads();
  const int nsp = (L + a.chunk - 1) / a.chunk;
  for (int e = threadIdx.x; e < G * D; e += blockDim.x) {
    const int h = e / D, dim = e - h * D;
    float M = -INFINITY;
    for (int w = 0; w < nwaves; ++w) M = fmaxf(M, sm_m[w][h]);
    float num = 0.f, den = 0.f;
    if (M != -INFINITY) {
      for (int w = 0; w < nwaves; ++w) {
        const float f = __builtin_amdgcn_exp2f(sm_m[w][h] - M);
        num += f * ((const float*)(dyn + (size_t)w * wbytes))[h * (D + 1) + dim];
        den += f * sm_l[w][h];
      }
    }
    const size_t bh = (size_t)b * hq + g * G + h;
    if (nsp == 1) {
      write_final(a, bh, D, dim, M, num, den);
    } else {
      const size_t pidx = bh * a.nsplit + split;
      a.part_o[pidx * D + dim] = num;
      if (dim == 0) {
        a.part_ml[pidx * 2] = M;
        a.part_ml[pidx * 2 + 1] = den;
      }
    }
  }
}

// Loads of K and of V per wave step of the fp32 kernel (registers bound it).
constexpr int kLoadsF32 = 4;

template <int U>
struct F32Rows {
  float4 k[U], v[U];
  uint32_t ok;
};

template <int D, int U>
__device__ __forceinline__ void load_rows_f32(F32Rows<U>& T, const int32_t* s_row, int t, int n,
                                              const float* kb, const float* vb, int lane) {
  constexpr int LPR = D / 4, RPI = 64 / LPR;
  const int c = lane % LPR, sub = lane / LPR;
  int row[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int r = t + j * RPI + sub;
    const int x = s_row[min(r, n - 1)];
    row[j] = r < n ? x : -1;
  }
  T.ok = 0u;
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int64_t off = (int64_t)(row[j] < 0 ? 0 : row[j]) * D + c * 4;
    T.k[j] = stream_load_f32x4(kb + off);
    T.v[j] = stream_load_f32x4(vb + off);
    if (row[j] >= 0) T.ok |= 1u << j;
  }
}

template <int D, int GP, int U>
__device__ __forceinline__ void consume_rows_f32(F32Rows<U>& T, const float4 (&q)[GP], float scale_log2,
                                                 float (&m)[GP], float (&l)[GP], float4 (&o)[GP]) {
  constexpr int LPR = D / 4;
  // a row outside the set or the cache read a stand-in row
#pragma unroll
  for (int j = 0; j < U; ++j)
    if (!((T.ok >> j) & 1u)) T.v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
  float x[U][GP], mn[GP];
  bool rise = false;
#pragma unroll
  for (int h = 0; h < GP; ++h) {
    float mt = -INFINITY;
#pragma unroll
    for (int j = 0; j < U; ++j) {
      float s = q[h].x * T.k[j].x;
      s = fmaf(q[h].y, T.k[j].y, s);
      s = fmaf(q[h].z, T.k[j].z, s);
      s = fmaf(q[h].w, T.k[j].w, s);
      s = group_sum<LPR>(s);
      x[j][h] = ((T.ok >> j) & 1u) ? s * scale_log2 : -INFINITY;
      mt = fmaxf(mt, x[j][h]);
    }
    // over the wave's row groups: they share one softmax state
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(mt), __float_as_uint(mt), false, false);
    mt = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    if (LPR == 16) {
      const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(mt), __float_as_uint(mt), false, false);
      mt = fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
    }
    mn[h] = fmaxf(m[h], mt);
    rise = rise || mn[h] > m[h] + 8.f;
  }
  // lazy rescaling, as in the bf16 kernel: probabilities stay below 2^8
  if (__builtin_amdgcn_ballot_w64(rise)) {
#pragma unroll
    for (int h = 0; h < GP; ++h) {
      const float alpha = mn[h] == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m[h] - mn[h]);
      m[h] = mn[h];
      l[h] *= alpha;
      o[h].x *= alpha; o[h].y *= alpha; o[h].z *= alpha; o[h].w *= alpha;
    }
  }
#pragma unroll
  for (int h = 0; h < GP; ++h) {
    const float mref = m[h] == -INFINITY ? 0.f : m[h];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const float p = __builtin_amdgcn_exp2f(x[j][h] - mref);
      l[h] += p;
      o[h].x = fmaf(p, T.v[j].x, o[h].x);
      o[h].y = fmaf(p, T.v[j].y, o[h].y);
      o[h].z = fmaf(p, T.v[j].z, o[h].z);
      o[h].w = fmaf(p, T.v[j].w, o[h].w);
    }
  }
}

// Sum over a wave's row groups (lanes of equal dims), in every lane.
template <int LPR>
__device__ __forceinline__ float over_row_groups(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  if (LPR == 16) {
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(b[0]) + __uint_as_float(b[1]);
  }
  return v;
}

// fp32 inputs on the vector ALU: a workgroup per (unit, split) and GP = 1, 2, 4
// or 8 of the unit's query heads together (launch_typed chooses), so a row of K
// and V is read once for GP heads, ceil(heads / GP) times in all.  A row is D / 4
// lanes of 16 bytes, so a wave load takes RPI whole rows; each step takes U loads
// of K and of V, the next step's in flight while one is multiplied.  A lane keeps
// 4 dims of every head's query and output; the dot products are summed over
// a row's lanes by DPP moves.  What bounds it: HBM on many rows, the chain of
// length, row id and row loads (about 7 us a launch) on few.  Against one
// workgroup per query head, which read every row once per head with one load
// in flight (at d 128, sets of 500 rows in 32 units of 4 heads: 27.3 -> 13.4
// us; dense, 128 units of 4 heads over 4000 rows, 524 MB: 289 -> 99 us,
// 5.3 TB/s).
template <int D, int GP, bool DENSE>
__global__ __launch_bounds__(64 * kMaxWaves) void attn_split_f32(AttnArgs a) {
  constexpr int LPR = D / 4, RPI = 64 / LPR;
  constexpr int U = kLoadsF32, ROWS = U * RPI;
  // dynamic LDS: [nwaves][GP][D] wave outputs, then the staged row ids
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  __shared__ float sm_m[kMaxWaves][16];
  __shared__ float sm_l[kMaxWaves][16];
  const int hkv = a.kv.hkv, hq = a.kv.hq;
  const int parts = (hq / hkv + GP - 1) / GP;  // workgroups that share a unit's heads
  const int split = blockIdx.x, u = blockIdx.y / parts;
  const int h0 = (blockIdx.y % parts) * GP, G = min(hq / hkv - h0, GP);  // this one's heads
  const int b = u / hkv, g = u % hkv;
  const size_t qh0 = (size_t)b * hq + g * (hq / hkv) + h0;
  const int nwaves = blockDim.x >> 6;
  float* s_o = (float*)dyn;
  int32_t* s_row = (int32_t*)(s_o + (size_t)nwaves * GP * D);
  const int start = split * a.chunk;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = lane % LPR, sub = lane / LPR;
  int32_t raw[kRowsPerThread];
  prefetch_entries<DENSE>(a, u, start, raw);
  const float* qp = (const float*)a.q + qh0 * D + c * 4;
  float4 q[GP];
#pragma unroll
  for (int h = 0; h < GP; ++h) q[h] = h < G ? load_f32x4(qp + h * D) : make_float4(0.f, 0.f, 0.f, 0.f);
  const int nb = kv_seq_len(a.kv, b);
  if (!DENSE && unit_excluded(a, u)) return;
  const UnitSpan sp = unit_span<DENSE>(a, u, b, nb);
  const int L = sp.L;
  if (L == 0 && split == 0) {  // empty set: y = 0, lse = -inf
    for (int e = threadIdx.x; e < G * D; e += blockDim.x)
      write_final(a, qh0 + e / D, D, e % D, -INFINITY, 0.f, 0.f);
    return;
  }
  if (start >= L) return;
  const int n = min(L, start + a.chunk) - start;
  if (a.kv.paged) stage_rows<DENSE, true>(a, raw, start, n, sp, nb, b, g, s_row);
  else stage_rows<DENSE, false>(a, raw, start, n, sp, nb, b, g, s_row);
  const float* kb = (const float*)a.kv.k;
  const float* vb = (const float*)a.kv.v;
  float m[GP], l[GP];
  float4 o[GP];
#pragma unroll
  for (int h = 0; h < GP; ++h) {
    m[h] = -INFINITY;
    l[h] = 0.f;
    o[h] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  // this wave's steps: wave, wave + nwaves, ...
  const int nsteps = (n + ROWS - 1) / ROWS;
  const int iters = wave < nsteps ? (nsteps - wave + nwaves - 1) / nwaves : 0;
  if (iters > 0) {
    F32Rows<U> A, B;
    const int stride = ROWS * nwaves;
    int t = wave * ROWS;
    load_rows_f32<D, U>(A, s_row, t, n, kb, vb, lane);
    int i = 0;
    for (; i + 2 < iters; i += 2) {
      load_rows_f32<D, U>(B, s_row, t + stride, n, kb, vb, lane);
      consume_rows_f32<D, GP, U>(A, q, a.scale_log2, m, l, o);
      load_rows_f32<D, U>(A, s_row, t + 2 * stride, n, kb, vb, lane);
      consume_rows_f32<D, GP, U>(B, q, a.scale_log2, m, l, o);
      t += 2 * stride;
    }
    if (i + 1 < iters) {
      load_rows_f32<D, U>(B, s_row, t + stride, n, kb, vb, lane);
      consume_rows_f32<D, GP, U>(A, q, a.scale_log2, m, l, o);
      consume_rows_f32<D, GP, U>(B, q, a.scale_log2, m, l, o);
    } else {
      consume_rows_f32<D, GP, U>(A, q, a.scale_log2, m, l, o);
    }
  }
#pragma unroll
  for (int h = 0; h < GP; ++h) {
    l[h] = over_row_groups<LPR>(l[h]);
    o[h].x = over_row_groups<LPR>(o[h].x);
    o[h].y = over_row_groups<LPR>(o[h].y);
    o[h].z = over_row_groups<LPR>(o[h].z);
    o[h].w = over_row_groups<LPR>(o[h].w);
    if (sub == 0) *(float4*)(s_o + ((size_t)wave * GP + h) * D + c * 4) = o[h];
    if (lane == 0) {
      sm_m[wave][h] = m[h];
      sm_l[wave][h] = l[h];
    }
  }
  __syncthreads();
  const int nsp = (L + a.chunk - 1) / a.chunk;
  for (int e = threadIdx.x; e < G * D; e += blockDim.x) {
    const int h = e / D, dim = e - h * D;
    float M = -INFINITY;
    for (int w = 0; w < nwaves; ++w) M = fmaxf(M, sm_m[w][h]);
    float num = 0.f, den = 0.f;
    if (M != -INFINITY) {
      for (int w = 0; w < nwaves; ++w) {
        const float f = __builtin_amdgcn_exp2f(sm_m[w][h] - M);
        num += f * s_o[((size_t)w * GP + h) * D + dim];
        den += f * sm_l[w][h];
      }
    }
    const size_t bh = qh0 + h;
    if (nsp == 1) {
      write_final(a, bh, D, dim, M, num, den);
    } else {
      const size_t pidx = bh * a.nsplit + split;
      a.part_o[pidx * D + dim] = num;
      if (dim == 0) {
        a.part_ml[pidx * 2] = M;
        a.part_ml[pidx * 2 + 1] = den;
      }
    }
  }
}

// Combines the split partials of one query head (grid: batch * num_q_heads,
// 256 threads).  Every thread first loads all it may need (the m, l and
// numerators of its first kMergePerThread split slots, for 256 / d split
// groups) together with the unit's lengths, before the number of splits in
// use is known, so the kernel costs one memory latency; slots past that
// number (stale values of earlier calls) are masked, never used in
// arithmetic.  The max, the weights and the sums follow in registers and
// LDS.  Units that fit one split were written by the split kernel and are
// skipped.
constexpr int kMergePerThread = 16;

template <int D, bool DENSE>
__global__ __launch_bounds__(256) void attn_merge(AttnArgs a) {
  constexpr int SG = 256 / D;
  __shared__ float s_red[SG][D];
  __shared__ float s_den[SG];
  __shared__ float s_max[4];
  const int bh = blockIdx.x;
  const int hkv = a.kv.hkv, hq = a.kv.hq, G = hq / hkv;
  const int b = bh / hq, h = bh % hq, u = b * hkv + h / G;
  const float* ml = a.part_ml + (size_t)bh * a.nsplit * 2;
  const float* po = a.part_o + (size_t)bh * a.nsplit * D;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int sg = tid / D, dim = tid - sg * D;
  // the first batch of slots below nsplit (a launch argument: no load
  // waits for another)
  float m0[kMergePerThread], l0[kMergePerThread], o0[kMergePerThread];
#pragma unroll
  for (int k = 0; k < kMergePerThread; ++k) {
    const int s = sg + k * SG;
    const bool in = s < a.nsplit;
    m0[k] = in ? ml[2 * s] : -INFINITY;
    l0[k] = in ? ml[2 * s + 1] : 0.f;
    o0[k] = in ? po[(size_t)s * D + dim] : 0.f;
  }
  if (!DENSE && unit_excluded(a, u)) return;
  const int L = unit_span<DENSE>(a, u, b, kv_seq_len(a.kv, b)).L;
  const int nsp = (L + a.chunk - 1) / a.chunk;
  if (nsp <= 1) return;
  float mx = -INFINITY, num = 0.f, den = 0.f;
  for (int s0 = sg; s0 < nsp; s0 += SG * kMergePerThread) {
    float m[kMergePerThread], l[kMergePerThread], o[kMergePerThread];
#pragma unroll
    for (int k = 0; k < kMergePerThread; ++k) {
      const int s = s0 + k * SG;
      const bool ok = s < nsp;
      if (s0 == sg) {
        m[k] = ok ? m0[k] : -INFINITY;
        l[k] = ok ? l0[k] : 0.f;
        o[k] = ok ? o0[k] : 0.f;
      } else {
        m[k] = ok ? ml[2 * s] : -INFINITY;
        l[k] = ok ? ml[2 * s + 1] : 0.f;
        o[k] = ok ? po[(size_t)s * D + dim] : 0.f;
      }
    }
    // rescale the running sums to the new maximum of this thread
    float bm = mx;
#pragma unroll
    for (int k = 0; k < kMergePerThread; ++k) bm = fmaxf(bm, m[k]);
    if (bm != -INFINITY) {
      const float r = __builtin_amdgcn_exp2f(mx - bm);
      num *= r;
      den *= r;
#pragma unroll
      for (int k = 0; k < kMergePerThread; ++k) {
        const float f = __builtin_amdgcn_exp2f(m[k] - bm);
        num += f * o[k];
        den += f * l[k];
      }
      mx = bm;
    }
  }
  // block-wide maximum
  const float wm = wave_max(mx);
  if (lane == 0) s_max[wave] = wm;
  __syncthreads();
  const float M = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
  const float f = (mx == -INFINITY || M == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mx - M);
  s_red[sg][dim] = num * f;
  if (dim == 0) s_den[sg] = den * f;
  __syncthreads();
  if (sg == 0) {
    float tot = 0.f, dt = 0.f;
#pragma unroll
    for (int k = 0; k < SG; ++k) {
      tot += s_red[k][dim];
      dt += s_den[k];
    }
    write_final(a, bh, D, dim, M, tot, dt);
  }
}

int env_int(const char* name, int dflt) {
  const char* e = getenv(name);
  const int x = e ? atoi(e) : 0;
  return x > 0 ? x : dflt;
}

// Most workgroups of a launch: one per CU for sets; for a dense bf16 stream of
// few units one per CU where it is short enough that the merge of more splits
// costs more than it gains (1 x 8 units of 4000 rows at d 128 18.1 us with
// 1024, 10.9 with 256; 16 of 8000 23.4 and 18.9, 4 of 38800 34.8 and 22.5),
// two, all resident together, for a longer one (8 units of 32000 rows, 131 MB:
// 256, 512 and 1024 workgroups 33.3, 31.3 and 35.9 us, 80 of 9000 68.5, 65.8
// and 67.1).  PRHS_ATTN_GROUPS and PRHS_ATTN_DENSE_GROUPS override them (tuning
// knobs, read once per process).
constexpr long long kLongDenseBytes = 96LL << 20;
constexpr long long kDenseGroups = 1024;
long long dense_groups_override() {
  static const int v = env_int("PRHS_ATTN_DENSE_GROUPS", 0);
  return v;
}
long long target_groups(int dtype, bool dense, long long bytes) {
  static const int sparse_v = env_int("PRHS_ATTN_GROUPS", 256);
  if (!dense) return sparse_v;
  if (dense_groups_override()) return dense_groups_override();
  return dtype != 1 ? kDenseGroups : (bytes < kLongDenseBytes ? 256 : 512);
}

// Splits of a dense bf16 stream of many units (more than half the CUs): none
// where a workgroup can stage a unit's rows, as that saves the merge launch
// (192 units of 1719 rows at d 128 26.5 us, in two splits 31.4; 224 of 1855
// 37.4 and 42.0; 400 of 490 22.7 and 34.6), except on up to a quarter more units
// than CUs of kLongUnitBytes or more of K and V, where the CUs that take two
// of them keep the rest waiting (300 units of 1606 rows 43.9 us, in four
// splits 39.3; 257 of 1142 35.4 and 32.0; 300 of 990 at d 64, 250 KB, 20.2
// and 22.9).  Split, a launch has about kDenseGroups workgroups, which even out
// ragged lengths (240 ragged units of 2801 rows: 480 workgroups 50.8 us, 1200
// 48.2; 256 of 8385 2048 workgroups 151, 1280 137), but not a few more than fill
// the kDenseSlots places for one a whole number of times (136 units of 11811
// rows: 1088 workgroups 119 us, 952 104; units a few more than the CUs are better
// off with the finer splits, 260 of 5488 in three 130, in four 125).
constexpr long long kLongUnitBytes = 320LL << 10;
constexpr long long kDenseSlots = 512;   // two workgroups a CU
long long many_unit_splits(long long units, long long rows, int d, long long cmax) {
  const long long least = (rows + cmax - 1) / cmax;
  const bool few_over = units > 256 && units <= 320;
  if (least == 1 && !(few_over && rows * d * 4 >= kLongUnitBytes)) return 1;
  const long long k = std::max(least, (kDenseGroups + units - 1) / units);
  const long long over = units * k % kDenseSlots;
  return !few_over && over > 0 && over <= kDenseSlots / 4 && k > least ? k - 1 : k;
}

// Waves per bf16 workgroup: 4, or what PRHS_ATTN_WAVES sets (0: not set).
int wave_override() {
  static const int v = [] {
    const int x = env_int("PRHS_ATTN_WAVES", 0);
    return x <= kMaxWaves ? x : 0;
  }();
  return v;
}
int wave_limit() { return wave_override() ? wave_override() : 4; }

template <int D, int GP, bool DENSE>
void launch_f32(const AttnArgs& a, int units, int waves, hipStream_t stream) {
  constexpr int kWaveBytes = GP * D * (int)sizeof(float) + 64 * kRowsPerThread * (int)sizeof(int32_t);
  static_assert(kMaxWaves * kWaveBytes <= 65536, "dynamic LDS that needs no attribute");
  hipLaunchKernelGGL((attn_split_f32<D, GP, DENSE>), dim3(a.nsplit, units * ((a.kv.hq / a.kv.hkv + GP - 1) / GP)),
                     dim3(64 * waves), waves * kWaveBytes, stream, a);
}

template <int D, bool DENSE, bool PAGED>
hipError_t launch_typed(const AttnArgs& a, int dtype, int units, int waves, hipStream_t stream) {
  if (dtype == 1) {
    const int G = a.kv.hq / a.kv.hkv;
    const size_t dyn = (size_t)waves * attn_wave_bytes(D, G) +
                       (size_t)64 * waves * kRowsPerThread * sizeof(int32_t);
    if (dyn > 65536) {
      const hipError_t e = hipFuncSetAttribute((const void*)attn_split_bf16<D, DENSE, PAGED>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((attn_split_bf16<D, DENSE, PAGED>), dim3(a.nsplit, units), dim3(64 * waves),
                       dyn, stream, a);
  } else {
    // heads per workgroup: all (up to 8), or fewer while the launch has at most
    // a wave for each of the four SIMDs of a CU, where the heads' serial work
    // costs more than reading the rows again from the caches, and a workgroup a
    // head where half the CUs get a wave at most (but unsplit for up to four; 8 units of 8
    // heads over 60 rows at d 64: 8 heads 8.0 us, 4 6.3, 2 5.8, 1 6.1; 48 of 16
    // over 338 rows at d 128: 8 heads a workgroup 21, 4 17.8, 2 24; 112 of 16 over
    // 82 rows 15.3, 20.0 and -; one of 8 over 377 rows in 12 splits 2 heads 8.8, 1
    // 7.5; unsplit 12 of 4 over 133 5.9 and 5.3, but 2 of 8 over 198 8.5 and 9.3)
    const int G = a.kv.hq / a.kv.hkv;
    const long long row_waves = (long long)units * a.nsplit * waves;   // of one workgroup a split
    int gp = G == 1 ? 1 : (G == 2 ? 2 : (G <= 4 ? 4 : 8));
    // waves up to which gp is halved, from 2 and from more
    const int halve[2] = {a.nsplit > 1 || G <= 4 ? device_cus() / 2 : 0, 4 * device_cus()};
    while (gp > 1 && row_waves * ((G + gp - 1) / gp) <= halve[gp > 2]) gp >>= 1;
    if (gp == 1) launch_f32<D, 1, DENSE>(a, units, waves, stream);
    else if (gp == 2) launch_f32<D, 2, DENSE>(a, units, waves, stream);
    else if (gp == 4) launch_f32<D, 4, DENSE>(a, units, waves, stream);
    else launch_f32<D, 8, DENSE>(a, units, waves, stream);
  }
  if (a.nsplit > 1)
    hipLaunchKernelGGL((attn_merge<D, DENSE>), dim3(a.kv.batch * a.kv.hq), dim3(256), 0, stream,
                       a);
  return hipGetLastError();
}

struct AttnLayout {
  size_t part_o, part_ml, total;
};

AttnLayout attn_layout(int batch, int hq, int d, int nsplit) {
  const size_t parts = (size_t)batch * hq * nsplit;
  AttnLayout L;
  size_t off = 0;
  L.part_o = off;  off += (parts * d * 4 + 255) & ~(size_t)255;
  L.part_ml = off; off += parts * 2 * 4;
  L.total = off;
  return L;
}

int waves_for(int dtype, bool dense, long long groups, int chunk) {
  // fp32: a wave per 16 rows where the workgroups are fewer than two per CU
  // (all rows load at once), else per 32 (less to combine: 1248 units of 60
  // rows 14.1 -> 12.9 us, dense 32 units of 4001 rows 38.8 -> 30.7)
  if (dtype != 1) {
    const int rows = groups < 2LL * device_cus() ? 16 : 32;
    return std::min(kMaxWaves, (chunk + rows - 1) / rows);
  }
  // twice the waves for at least two tiles each while every workgroup has a CU
  // to itself: more of the set's rows load at once (8 units of 300 rows 8.8 ->
  // 8.0 us, 16 of 500 11.5 -> 11.0, 72 of 280 at d 64 7.5 -> 7.1; 64 of 200
  // 8.6 -> 9.0, 384 of 640 30.0 -> 32.9).  Such a workgroup leaves no room on its
  // CU for another launch's; the gate's two branches on two streams lose nothing
  // by it (blocks of 4 steps, four waves -> eight, us: 16 x 8 units 398 -> 384, 8 x
  // 32 467 -> 464, 4 x 8 433 -> 431, 2 x 32 521 -> 522)
  int w = chunk / 32;
  const bool twice = !dense && groups <= device_cus() && chunk >= 256 && !wave_override();
  const int lim = wave_limit() * (twice ? 2 : 1);
  return w < 1 ? 1 : std::min({w, lim, kMaxWaves});
}

}  // namespace

// Rows per workgroup: a multiple of the per-wave tile (32 rows for bf16, 16
// rows for fp32), so that the launch has at most target_groups() workgroups,
// at most kMaxSplits splits, and balanced so the splits of a full unit differ
// by at most one tile.  At most, and not about: 160 units of 800 rows run
// 25.0 us as 320 workgroups, where some CUs take two, and 19.4 as 160 (192
// units of 1200 rows 32.6 and 27.3, 80 of 1500 23.3 and 21.2).  Where the
// rows staged per workgroup, 8 per thread, allow no such split, sets take the
// fewest splits they allow and a dense stream twice the workgroups and so on
// (16 units of 65537 rows: 528 workgroups 105 us, 1008 92).  Dense bf16 streams
// of many units: many_unit_splits.
void attn_split_geometry(int dtype, bool dense, int batch, int hq, int hkv, int d, int rows_cap,
                         int* chunk, int* nsplit) {
  const int gran = dtype == 1 ? 32 : 16;
  const long long units = std::max(1LL, (long long)batch * hkv);
  const long long rows = rows_cap > 0 ? rows_cap : 1;
  const long long threads = dtype == 1 ? 64LL * wave_limit() : 256;
  const long long cmax = threads * kRowsPerThread;
  auto rows_of = [&](long long groups) {
    const long long k = std::max(1LL, groups / units);
    return (rows + k - 1) / k;
  };
  long long tg = target_groups(dtype, dense, rows * units * d * 4);
  while (dense && rows_of(tg) > cmax) tg *= 2;
  long long c = rows_of(tg);
  if (dense && dtype == 1 && units > 128 && !dense_groups_override()) {
    const long long k = many_unit_splits(units, rows, d, cmax);
    c = (rows + k - 1) / k;
  }
  const long long cmin = (rows + kMaxSplits - 1) / kMaxSplits;
  if (dtype != 1) {
    c = std::max(c, std::min((rows + kMergeSplitsF32 - 1) / kMergeSplitsF32, rows_of(256)));
    const long long least = std::max<long long>(c, kMinRowsF32);
    const bool few = (rows + least - 1) / least * batch * hq < kFewHeadsF32 &&
                     rows <= kMergeSplitsF32 * kMinRowsF32 / 2;
    c = std::max<long long>(c, few ? kMinRowsF32 / 2 : kMinRowsF32);
  }
  if (c < cmin) c = cmin;
  long long whole = dtype == 1 ? (dense ? 0 : kNoSplitRows) : kNoSplitRowsF32;
  if (dense && dtype != 1)
    whole = units >= kMostF32   ? kNoSplitMostF32
            : units >= kManyF32 ? kNoSplitManyF32
                                : std::min(whole, (long long)kNoSplitHeadRowsF32 * hkv / hq);
  if (rows <= whole && rows <= cmax) c = rows;
  if (c > cmax) c = cmax;
  if (c < gran) c = gran;
  const long long ns = (rows + c - 1) / c;
  c = (rows + ns - 1) / ns;
  c = ((c + gran - 1) / gran) * gran;
  if (c > cmax) c = cmax;
  *chunk = (int)c;
  *nsplit = (int)((rows + c - 1) / c);
}

// Scratch for the split-K partials of prhs_sparse_decode_attn_static, the
// entry point for callers that cannot allocate.  Every device that runs it
// holds its own copy until the process ends; calls on one device share it.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

hipError_t attn_static_scratch(void** ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

size_t attn_call_bytes(int dtype, bool dense, int batch, int hq, int hkv, int d, int rows_cap) {
  int chunk, nsplit;
  attn_split_geometry(dtype, dense, batch, hq, hkv, d, rows_cap, &chunk, &nsplit);
  return attn_layout(batch, hq, d, nsplit).total;
}

// A program keeps one workspace for its largest batch and longest rows, and a
// smaller call can want more of it: its units take more splits each (bf16 sets
// of 2000 rows: 24 sequences of 8 units 192 splits in all, one sequence 256).
// So the size is a bound over every smaller call, from what attn_split_geometry
// may take: at most target_groups() workgroups or the fewest splits that staging
// allows, a dense launch up to a split a unit more, or twice those splits.
size_t attn_workspace_bytes(int dtype, bool dense, int batch, int hq, int hkv, int d,
                            int rows_cap) {
  const long long units = (long long)batch * hkv, rows = rows_cap > 0 ? rows_cap : 1;
  const long long cmax = (dtype == 1 ? 64LL * wave_limit() : 256) * kRowsPerThread;
  const long long least = (rows + cmax - 1) / cmax;
  long long groups;   // splits of all units
  if (!dense) {
    const bool whole = rows <= (dtype == 1 ? kNoSplitRows : kNoSplitRowsF32) && rows <= cmax;
    groups = whole ? units : std::max(target_groups(dtype, false, 0), units * least);
  } else {
    const long long set = dense_groups_override();
    const long long halved = dtype == 1 && !set ? std::min(units, 128LL) : units;
    groups = std::max({set ? set : kDenseGroups + (dtype == 1 ? units : 0), units * least,
                       least > 1 ? 2 * halved * least : 0});
  }
  const int gran = dtype == 1 ? 32 : 16;
  groups = std::min(groups, units * ((rows + gran - 1) / gran));
  // the largest launch of any batch up to this one has at most that many splits
  const long long per = units > 0 ? (groups + units - 1) / units : 0;
  return std::max(attn_layout(batch, hq, d, (int)per).total,
                  attn_call_bytes(dtype, dense, batch, hq, hkv, d, rows_cap));
}

hipError_t launch_attention(const AttnLaunch& s, bool dense, hipStream_t stream) {
  if (s.kv.batch == 0) return hipSuccess;
  AttnArgs a;
  a.kv = s.kv;
  a.q = s.q;
  a.set_idx = s.set_idx;
  a.set_len = s.set_len;
  a.tail_start = dense ? nullptr : s.tail_start;
  a.unit_row = dense ? nullptr : s.unit_row;
  a.unit_tail = dense ? nullptr : s.unit_tail;
  a.pool_rows = s.pool_rows;
  a.unit_gate = dense ? nullptr : s.unit_gate;
  a.units_side = s.units_side;
  a.psaw = dense ? 0 : s.psaw;
  a.psaw_f = s.psaw_f;
  a.psaw_sink = s.psaw_sink;
  a.set_cap = s.set_cap;
  a.scale_log2 = s.scale * 1.44269504088896340736f;
  const int rows_cap = dense ? s.kv.max_seq_len : s.set_cap;
  attn_split_geometry(s.dtype, dense, s.kv.batch, s.kv.hq, s.kv.hkv, s.kv.d, rows_cap, &a.chunk,
                      &a.nsplit);
  const AttnLayout L = attn_layout(s.kv.batch, s.kv.hq, s.kv.d, a.nsplit);
  char* ws = (char*)s.ws;
  a.part_o = (float*)(ws + L.part_o);
  a.part_ml = (float*)(ws + L.part_ml);
  a.out = s.out;
  a.lse = s.lse;
  const int units = s.kv.batch * s.kv.hkv;
  const int waves = waves_for(s.dtype, dense, (long long)units * a.nsplit, a.chunk);
  const bool paged = s.kv.paged != 0;
#define PRHS_ATTN_DISPATCH(DV)                                                          \
  if (dense) {                                                                          \
    return paged ? launch_typed<DV, true, true>(a, s.dtype, units, waves, stream)       \
                 : launch_typed<DV, true, false>(a, s.dtype, units, waves, stream);     \
  }                                                                                     \
  return paged ? launch_typed<DV, false, true>(a, s.dtype, units, waves, stream)        \
               : launch_typed<DV, false, false>(a, s.dtype, units, waves, stream);
  if (s.kv.d == 128) {
    PRHS_ATTN_DISPATCH(128)
  }
  PRHS_ATTN_DISPATCH(64)
#undef PRHS_ATTN_DISPATCH
}

}  // namespace prhs
