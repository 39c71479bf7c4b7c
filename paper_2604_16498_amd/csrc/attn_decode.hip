// bf16 fused attention for one new query per sequence over a KV cache (decode).  HBM-bound:
// every cached K and V row is read exactly once, with 128-bit loads, and nothing else of
// comparable size moves.
//
// Split-KV: a block (kv head, sequence, range) streams one contiguous range of cache rows of ONE kv
// head for all G = Hq/Hkv query heads that share it (grouped-query attention reads the cache
// once per group, not once per query head).  The 4 waves of a block (8 for some short rows) take the 16-row tiles
// of the range in turn and each keeps two tiles of K and V loads in flight
// ahead of the one it is working on.  The number of ranges is chosen on the host by an estimate of their time, at
// most two blocks per compute unit: a large batch needs no split at all (one block per
// (kv head, sequence) walks the whole cache and writes the final output itself: no partials, no
// second kernel), a small batch is cut into ranges that are multiples of 128 rows.
//
// Per tile of 16 rows:
//   scores   S[row, head] = K . q^T on the matrix cores (v_mfma_f32_16x16x32_bf16, heads padded
//            to 16).  K is loaded straight from HBM in the MFMA A layout: lane = (row l%16, 16-byte
//            chunk), the contraction order over dh is permuted so that one wave-wide load reads 64
//            contiguous bytes of each row.  No LDS, no transposition.
//   softmax  in the accumulator layout (lane = head, 4 rows per lane): running maximum per head
//            with LAZY rescaling (the accumulators are only rescaled when some row beats the
//            maximum, which becomes rare after the first tiles), exp2 domain.
//   P . V    each lane owns 8 output columns for every head.  P goes through a 16 x G float
//            patch of LDS (the only cross-lane traffic), is packed with its neighbour row to
//            bf16 pairs, V rows of two steps are interleaved with byte permutes, and the
//            accumulation runs on v_dot2_f32_bf16: two rows per instruction, fp32 accumulate.
// Wave and block partials are merged in a fixed order; with more than one split the block writes
// (m, l, o) per query head to the workspace and a second kernel merges the splits in split order
// -- no atomics, so the result is bitwise reproducible.
#include <math.h>
#include "common.hpp"

namespace forge {
namespace {

constexpr int TILE = 16;                  // cache rows per MFMA tile
constexpr int GRAIN = 128;                // a split is a multiple of this many rows (two tiles per wave of four)
constexpr int MAX_SPLITS = 64;            // what plan_splits was fitted over, and a bound of the workspace

struct DecParams {
  const bf16* q;
  const bf16* k;
  const bf16* v;
  float* part;     // [B, Hkv, splits, G, dh + 2]
  bf16* out;       // [B, Hq * dh]: written directly when splits == 1
  int q_heads, kv_heads, kv_len, splits;   // kv_heads counts blocks: cache heads x passes
  int heads_first;      // grid (kv_heads, batch, splits); otherwise (splits, kv_heads, batch)
  int passes;           // blocks (of G query heads each) that share one cache head
  int rows_per_split;   // multiple of GRAIN
  int64_t kv_bs, kv_hs;
  float scale_log2e;
  const int* kv_pos;   // per-sequence: rows [0, kv_pos[b]] (clamped to kv_len - 1); NULL: kv_len rows
  int batch;
  int by_length;       // > 0: blocks take the sequences by length, in rounds of this many; at most 64 sequences then
};

// lanes l, l ^ 16, l ^ 32, l ^ 48 (on the vector ALU: the LDS permute that a shuffle is costs 50 ns a step)
template <typename Op>
__device__ inline float across_rows(float x, Op op) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return op(__uint_as_float(h[0]), __uint_as_float(h[1]));
}
// the sums of four values over those lanes: row r of 16 lanes gets that of x[r]
__device__ inline float sum_to_rows(const float* x) {
  float t[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[2 * i]), __float_as_uint(x[2 * i + 1]), false, false);
    t[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(t[0]), __float_as_uint(t[1]), false, false);
  return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}

// G: query heads per KV head, 1 ... 8 (the MFMA's 16 head columns hold them zero-padded; the
// P . V accumulators grow with G, so the larger groups run at two blocks per SIMD instead of three)
// FREE: the loads of a tile are left to the scheduler.
template <int DH, int G, int NWAVES, bool FREE = false>
__global__ __launch_bounds__(NWAVES * 64, G > 4 || NWAVES == 8 ? 2 : 3) void attn_decode_kernel(DecParams p) {
  constexpr int NJ = DH / 32;          // MFMAs (and K loads) per tile
  constexpr int LPR = DH / 8;          // lanes per V row
  constexpr int KPS = 64 / LPR;        // rows per wave-wide V load
  constexpr int VSTEPS = TILE / KPS;   // V loads per tile
  constexpr int NPAIR = VSTEPS / 2;    // row pairs per lane per tile
  __shared__ __attribute__((aligned(16))) float pbuf[NWAVES][TILE][G];
  __shared__ __attribute__((aligned(16))) float abuf[NWAVES][G];
  __shared__ float sm[NWAVES][G][DH + 2];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // Lengths are known here only.  All blocks of a round are resident, one per CU, and a CU's next block comes a round later: the
  // sequences from the longest to the shortest, every other round backwards, give each CU about the same number of rows.  The
  // last round runs forwards: where it is broken, its blocks come to the first CUs, which a backward round before it left the
  // shorter ones.
  int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
  if (p.by_length > 0) {
    const int mine = lane < p.batch ? min(max(p.kv_pos[lane], 0), p.kv_len - 1) : -1;    // a lane per sequence
    if (!__all(mine == __builtin_amdgcn_readfirstlane(mine) || mine < 0)) {
      const int l = bx + gridDim.x * (by + gridDim.y * bz), first = l - l % p.by_length;
      const int all = gridDim.x * gridDim.y * gridDim.z;
      const int at = ((all - 1) / p.by_length - l / p.by_length) & 1 ? 2 * first + min(all - first, p.by_length) - 1 - l : l;
      bx = at % gridDim.x;
      by = at / gridDim.x % gridDim.y;
      bz = at / gridDim.x / gridDim.y;
      int place = 0;                                     // sequences before this lane's
      for (int j = 0; j < p.batch; ++j) {
        const int other = __builtin_amdgcn_readlane(mine, j);
        place += other > mine || (other == mine && j < lane);
      }
      int& seq = p.heads_first ? by : bz;
      seq = __ffsll((unsigned long long)__ballot(lane < p.batch && place == seq)) - 1;
    }
  }
  const int g = p.heads_first ? bx : by, b = p.heads_first ? by : bz, split = p.heads_first ? bz : bx;
  const int krow = lane & 15, kg = lane >> 4;          // MFMA layout: row in tile / lane group
  const int head = lane & 15;                          // ... and the accumulator's column
  const int slot = lane / LPR, c = lane % LPR;         // V layout: row in step / 16-byte chunk

  // query heads g G ... g G + G - 1 attend to cache head g / passes
  const int64_t cache_head = (int64_t)b * p.kv_bs + (int64_t)(g / p.passes) * p.kv_hs;
  const bf16* kb = p.k + cache_head;
  const bf16* vb = p.v + cache_head;
  const int split_begin = split * p.rows_per_split;
  // tiles of this wave that begin before the end of the range, rounded up to a pair (the loop
  // takes two per trip; the loads stay unconditional so that their count per trip is fixed)
  // a split that lies wholly past the end of a short sequence writes a neutral partial
  // (maximum -1e30, sum 0), which the combine weighs with exactly 0
  const int kv_len = p.kv_pos != nullptr ? min(max(p.kv_pos[b], 0), p.kv_len - 1) + 1 : p.kv_len;
  const int row_end = min(kv_len, split_begin + p.rows_per_split);
  const int rows_w = row_end - split_begin - wave * TILE;          // <= 0: no tile for this wave
  const int ntile = rows_w > 0 ? (ceil_div(rows_w, NWAVES * TILE) + 1) / 2 * 2 : 0;
  const int last = max(row_end, 1) - 1;   // (not kv_len - 1: tiles past the end of a range would read the next range's rows)

  // q as the MFMA B operand: lane = (head, chunk 4j + kg); heads >= G are zero columns
  bf16x8 qf[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    u32x4 t = {0, 0, 0, 0};
    if (head < G) t = *reinterpret_cast<const u32x4*>(p.q + ((int64_t)b * p.q_heads + g * G + head) * DH + (4 * j + kg) * 8);
    qf[j] = __builtin_bit_cast(bf16x8, t);
  }

  u32x4 kr[2][NJ], vr[2][VSTEPS];
  // tile t of this wave: rows base .. base + 15 (the waves take the tiles of the range in turn)
  auto tile_base = [&](int t) { return split_begin + (t * NWAVES + wave) * TILE; };
  // (scheduled among its neighbours, a tile's loads go to second registers, and the copies back wait for them; with that and
  // the reductions on the vector ALU, us: 8 sequences up to 641 rows of 12 heads of 64 7.6 -> 7.0, 25 of 950 rows of 8 of 128
  // 21.6 -> 20.7, 64 of 2049 98.0 -> 97.0)
  auto load_tile = [&](int t, u32x4 (&kk)[NJ], u32x4 (&vv)[VSTEPS]) {
    if constexpr (!FREE) __builtin_amdgcn_sched_barrier(0);
    const int base = tile_base(t);
#pragma unroll
    for (int j = 0; j < NJ; ++j)   // rows past the end re-read the last row (masked below)
      kk[j] = *reinterpret_cast<const u32x4*>(kb + (int64_t)min(base + krow, last) * DH + (4 * j + kg) * 8);
#pragma unroll
    for (int s = 0; s < VSTEPS; ++s)
      vv[s] = *reinterpret_cast<const u32x4*>(vb + (int64_t)min(base + s * KPS + slot, last) * DH + c * 8);
    if constexpr (!FREE) __builtin_amdgcn_sched_barrier(0);
  };
  load_tile(0, kr[0], vr[0]);
  load_tile(1, kr[1], vr[1]);

  float m_run = -1e30f, l_part = 0.f;      // accumulator layout: this lane's head
  float acc[G][8];                         // V layout: this lane's 8 columns, all heads
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[h][e] = 0.f;
  const float cl = p.scale_log2e;

  for (int t0 = 0; t0 < ntile; t0 += 2) {
#pragma unroll
   for (int u = 0; u < 2; ++u) {
    const int t = t0 + u;
    u32x4 (&kk)[NJ] = kr[u];
    u32x4 (&vv)[VSTEPS] = vr[u];
    const int base = tile_base(t);
    if (base < row_end) {     // wave-uniform: tiles wholly past the end contribute nothing
      // ---- scores ------------------------------------------------------------------------------
      floatx4 sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kk[j]), qf[j], sacc, 0, 0, 0);
      float sc[4];
      float mx = -INFINITY;
#pragma unroll
      for (int v = 0; v < 4; ++v) {     // accumulator register v is row 4 kg + v
        sc[v] = base + 4 * kg + v < row_end ? sacc[v] * cl : -INFINITY;
        mx = fmaxf(mx, sc[v]);
      }
      mx = across_rows(mx, [](float a, float b) { return fmaxf(a, b); });
      // ---- lazy rescale --------------------------------------------------------------------------
      if (__any(mx > m_run)) {
        const float m_new = fmaxf(m_run, mx);
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        m_run = m_new;
        l_part *= alpha;
        if (lane < G) abuf[wave][lane] = alpha;      // lane = head (kg == 0)
        wave_lds_sync();
        float al[G];
#pragma unroll
        for (int h = 0; h < G; ++h) al[h] = abuf[wave][h];
#pragma unroll
        for (int h = 0; h < G; ++h)
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[h][e] *= al[h];
      }
      // ---- probabilities, through LDS to the V layout ---------------------------------------------
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float pr = __builtin_amdgcn_exp2f(sc[v] - m_run);   // exp2(-inf) = 0 past the end
        l_part += pr;
        if (head < G) pbuf[wave][4 * kg + v][head] = pr;
      }
      wave_lds_sync();
      // ---- P . V on dot2: rows (s, s+1) of this lane's slot packed as bf16 pairs ---------------------
#pragma unroll
      for (int pi = 0; pi < NPAIR; ++pi) {
        const int ra = (2 * pi) * KPS + slot, rb = (2 * pi + 1) * KPS + slot;
        bf16x2 pp[G];
#pragma unroll
        for (int h = 0; h < G; ++h) {
          pp[h][0] = (bf16)pbuf[wave][ra][h];
          pp[h][1] = (bf16)pbuf[wave][rb][h];
        }
        const u32x4 va = vv[2 * pi], vb2 = vv[2 * pi + 1];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          // (va.lo, vb.lo) and (va.hi, vb.hi): element 2d and 2d+1 of both rows
          const uint32_t lo = __builtin_amdgcn_perm(vb2[d], va[d], 0x05040100);
          const uint32_t hi = __builtin_amdgcn_perm(vb2[d], va[d], 0x07060302);
          const bf16x2 vlo = __builtin_bit_cast(bf16x2, lo), vhi = __builtin_bit_cast(bf16x2, hi);
#pragma unroll
          for (int h = 0; h < G; ++h) {
            acc[h][2 * d] = __builtin_amdgcn_fdot2_f32_bf16(vlo, pp[h], acc[h][2 * d], false);
            acc[h][2 * d + 1] = __builtin_amdgcn_fdot2_f32_bf16(vhi, pp[h], acc[h][2 * d + 1], false);
          }
        }
      }
    }
    wave_lds_sync();   // this tile's LDS reads are done before the next tile's writes
    // refill the registers just consumed (unconditional: past the end the last row is read
    // again, which keeps the number of loads per trip, and with it the wait counts, fixed)
    load_tile(t + 2, kr[u], vr[u]);
   }
  }

  // ---- merge inside the wave: plain sums (one running maximum per head for the whole wave), each row of 16 lanes gets
  // the columns that its number picks -------------------------------------------------------------------------
  if constexpr (LPR == 8) {
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        acc[h][e] += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(acc[h][e]), 0x128, 0xf, 0xf, true));   // row_ror:8
  }
  l_part = across_rows(l_part, [](float a, float b) { return a + b; });
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float x = sum_to_rows(&acc[h][4 * j]);
      if (LPR == 16 || (lane & 8) == 0) sm[wave][h][c * 8 + 4 * j + kg] = x;
    }
  if (lane < G) { sm[wave][lane][DH] = m_run; sm[wave][lane][DH + 1] = l_part; }
  lds_barrier();
  // ---- merge the waves, fixed order -------------------------------------------------------------------
  float* dst = p.part + ((((int64_t)b * p.kv_heads + g) * p.splits + split) * G) * (DH + 2);
  for (int idx = tid; idx < G * DH; idx += NWAVES * 64) {
    const int h = idx / DH, d = idx % DH;
    float mn = sm[0][h][DH];
#pragma unroll
    for (int w = 1; w < NWAVES; ++w) mn = fmaxf(mn, sm[w][h][DH]);
    float o = 0.f, lt = 0.f;
#pragma unroll
    for (int w = 0; w < NWAVES; ++w) {
      const float a = __builtin_amdgcn_exp2f(sm[w][h][DH] - mn);
      o += sm[w][h][d] * a;
      lt += sm[w][h][DH + 1] * a;
    }
    if (p.splits == 1) {   // the whole cache in one block: this is the result
      p.out[((int64_t)b * p.q_heads + g * G + h) * DH + d] = (bf16)(o / lt);
    } else {
      dst[h * (DH + 2) + d] = o;
      if (d == 0) { dst[h * (DH + 2) + DH] = mn; dst[h * (DH + 2) + DH + 1] = lt; }
    }
  }
}

// one block per (batch, query head): merge the splits in split order and normalise, 8 splits per round trip (their maxima,
// sums and outputs are requested together; weights worked out by one wave first and handed over through LDS were a second trip
// and a barrier: 9 sequences up to 1323 rows of 8 heads of 128, attention and merge, 14.85 | 14.1 us, 5 up to 8192 28.1 | 27.4)
template <int DH>
__global__ __launch_bounds__(DH) void attn_decode_combine(const float* __restrict__ part,
                                                          bf16* __restrict__ out, int q_heads,
                                                          int kv_heads, int splits) {
  const int h = blockIdx.x, b = blockIdx.y, d = threadIdx.x;
  const int G = q_heads / kv_heads;
  const int g = h / G, hh = h % G;
  const float* src = part + ((((int64_t)b * kv_heads + g) * splits) * G + hh) * (DH + 2);
  const int64_t stride = (int64_t)G * (DH + 2);
  float m = -1e30f, l = 0.f, o = 0.f;
  for (int z0 = 0; z0 < splits; z0 += 8) {
    float mz[8], lz[8], oz[8];
#pragma unroll
    for (int z = 0; z < 8; ++z) {
      const float* p = src + min(z0 + z, splits - 1) * stride;
      mz[z] = p[DH];
      lz[z] = p[DH + 1];
      oz[z] = p[d];
    }
    float mn = m;
#pragma unroll
    for (int z = 0; z < 8; ++z) mn = fmaxf(mn, mz[z]);
    const float a = __builtin_amdgcn_exp2f(m - mn);
    l *= a;
    o *= a;
    m = mn;
#pragma unroll
    for (int z = 0; z < 8; ++z) {                         // (selects: a weight of 0 would turn an infinite output into NaN)
      const float w = __builtin_amdgcn_exp2f(mz[z] - mn);
      l += z0 + z < splits ? lz[z] * w : 0.f;
      o += z0 + z < splits ? oz[z] * w : 0.f;
    }
  }
  out[((int64_t)b * q_heads + h) * DH + d] = (bf16)(o / l);
}

// Number of row ranges: the count with the least estimated time.  A block alone on its CU streams 43.5 KB of cache per us
// (rows of 64: 29, with 8 waves 42), slower with others beside it, the chip 6.5 MB (of a ragged batch 0.7 of the longest
// cache: a guess at its lengths, which the host does not know), and the merge of the ranges is a launch of 3.5 us.  Fitted
// by choice, not by time, to 2000 drawn caches timed at every count: 0.4 % off the best in the geometric mean, where about
// two blocks per CU and ranges of 256 rows at least (the rule before last) were 9 % off, one block per CU and a block
// of 45 KB per us whatever its rows (the last rule) 2.8 %, with 7 % of the caches more than 5 % slower than before it.
// us, merge included, those two | this: 33 sequences up to 5183 rows of 4 heads of 64 34.3, 60.1 | 31.4, 20 up to 6187 of
// 8 of 128 63.2, 76.3 | 63.1, 24 up to 1501 of 8 of 128 30.2, 23.8 | 23.8, 7 up to 8352 of 12 of 64 29.3, 38.2 | 28.8.
struct SplitPlan { int splits, rows_per_split; };
constexpr int MIN_CUT_ROWS = 512;         // a shorter cache is never cut, so its calls need no workspace
// the most ranges a batch is ever cut into, whatever the cache length
inline int max_splits(int batch, int kv_heads) {
  return (int)min((int64_t)MAX_SPLITS, ceil_div64(2 * (int64_t)compute_units(), (int64_t)batch * kv_heads));
}
// 8 waves where 4 have not enough bytes in flight: short rows, one block per CU at most, a cache of some length (us, 4 | 8:
// 8 sequences up to 641 rows of 12 heads of 64 9.0 | 7.2, 4 x 348 6.5 | 5.8, but 25 x 743 15.0 | 16.9, 2 x 113 4.2 | 4.4)
inline bool eight_waves(int batch, int kv_heads, int kv_len, int head_dim, int group) {
  return head_dim == 64 && group == 1 && (int64_t)batch * kv_heads <= compute_units() && kv_len >= 256;
}
inline SplitPlan plan_splits(int batch, int kv_heads, int kv_len, int head_dim, int group, bool ragged) {
  SplitPlan best = {1, ceil_div(kv_len, GRAIN) * GRAIN};
  if (kv_len < MIN_CUT_ROWS) return best;
  const int64_t pairs = (int64_t)batch * kv_heads, cus = compute_units();
  const double row_kb = head_dim * 4e-3, all_us = (double)pairs * kv_len * row_kb * (ragged ? 0.71 : 1.0) / 6500.0;
  const double beside = head_dim == 64 ? 0.3 : 1.37;
  double least = 0.0;
  for (int want = 1, most = max(1, min(max_splits(batch, kv_heads), kv_len / GRAIN)); want <= most; ++want) {
    const int rows = ceil_div(ceil_div(kv_len, want), GRAIN) * GRAIN, splits = ceil_div(kv_len, rows);   // splits <= want
    const double rate = head_dim != 64 ? 43.5 : splits == 1 && eight_waves(batch, kv_heads, kv_len, head_dim, group) ? 42.0 : 29.0;
    const int64_t on_cu = ceil_div64(pairs * splits, cus);                   // on the fullest CU; of uneven lengths, on the average
    const double share = ragged ? fmax(1.0, (double)(pairs * splits) / cus) : (double)on_cu;
    const double us = fmax(min(rows, kv_len) * row_kb / rate * (1.0 + beside * sqrt(share - 1.0)) + 1.2 * (on_cu - 1), all_us) +
                      (splits > 1 ? 3.5 : 0.0);
    if (want == 1 || us < least) { least = us; best = SplitPlan{splits, rows}; }
  }
  return best;
}
// Upper bound of plan_splits(.., len).splits over every len <= kv_len: the number of ranges is
// not monotone in the length (the range size is rounded up to GRAIN), the scratch size must be,
// because a generation loop sizes its scratch once, for the capacity of its cache.
inline int splits_bound(int batch, int kv_heads, int kv_len) {
  return kv_len < MIN_CUT_ROWS ? 1 : min(max_splits(batch, kv_heads), kv_len / GRAIN);
}

// Query heads per block for `group` heads sharing one cache head: the whole group up to 8, else
// its largest divisor up to 8 -- several blocks then each stream that cache head for their share of
// the query heads (16 heads: two passes of 8).  More than four passes (a prime group above 8) are
// left to the vector-ALU kernel.
constexpr int MAX_G = 8, MAX_PASSES = 4;
inline int heads_per_block(int group) {
  if (group <= MAX_G) return group;
  for (int d = MAX_G; d >= 1; --d)
    if (group % d == 0) return group / d <= MAX_PASSES ? d : 0;
  return 0;
}
// blocks per sequence and range: cache heads x passes (the split plan counts these)
inline int block_heads(int q_heads, int kv_heads) {
  const int gb = heads_per_block(q_heads / kv_heads);
  return gb > 0 ? q_heads / gb : kv_heads;
}

template <int DH, int G>
forge_status launch_dg(const AttnArgs& a, const SplitPlan& pl, hipStream_t s) {
  const int yheads = a.q_heads / G;
  DecParams p;
  p.q = (const bf16*)a.q;
  p.k = (const bf16*)a.k;
  p.v = (const bf16*)a.v;
  p.part = (float*)a.workspace;
  p.out = (bf16*)a.out;
  p.q_heads = a.q_heads;
  p.kv_heads = yheads;
  p.passes = yheads / a.kv_heads;
  p.kv_len = a.kv_len;
  p.splits = pl.splits;
  p.rows_per_split = pl.rows_per_split;
  p.kv_bs = a.kv_batch_stride;
  p.kv_hs = a.kv_head_stride;
  p.scale_log2e = a.scale * 1.4426950408889634f;
  p.kv_pos = a.kv_pos;
  // Ranges are the fastest block index, except two or four of them in a grid that is not whole rounds over the CUs:
  // blocks go round-robin over the 8 XCDs, so with an even count every XCD gets the same ranges of all heads,
  // and the last ones are short or empty where the lengths differ (us, ranges | heads fastest, merge included: 21
  // sequences up to 1400 rows of 16 heads 39.5 | 33.7, 5 up to 1400 of 16 16.0 | 12.2, 24 up to 700 of 8 14.0 | 12.8).
  // Elsewhere heads first keeps the same rows of all heads in flight at once and loses as often as it
  // wins (1 sequence of 4096, 32 heads, 16 ranges 18.0 | 22.1; 3 up to 4508 in a cache of 8192, 8 heads, 12 ranges
  // 13.8 | 17.1; 16 up to 6556, 16 heads, 512 blocks 107.6 | 117.5; 21 up to 4096, 12 heads, 3 ranges 38.1 | 40.9).
  const int64_t blocks = (int64_t)p.splits * yheads * a.batch;
  p.heads_first = (p.splits == 2 || p.splits == 4) && blocks % compute_units() != 0;
  p.batch = a.batch;
  // By length: where some CU gets a second block and the rows are worth the look at all lengths.  us, batch order | by length:
  // 25 x 12 heads of 128 up to 899 rows 26.0 | 21.2, 31 x 12 of 64 up to 1897 29.5 | 25.1, 51 x 16 of 128 up to 1392 86 | 74, 39 x 8
  // of 128 up to 2410 62.4 | 55.4; of 170 drawn caches in one and two ranges 7 % less in the geometric mean, seven of them 2 to 6 %
  // more.  Of more ranges the last ones of a short sequence are empty, and its length says little about the first: 12 drawn
  // ones with heads of 128 2.3 % less, 33 with heads of 64 2.8 % more, up to 19 % (15 x 12 up to 4200).  Not, times batch order, up
  // to 552 rows of 60 x 8 heads of 128 1.04, 584 of 44 x 16 1.05, 699 of 61 x 8 1.05, 792 of 61 x 16 1.02, 513 of 64 x 12 of 64 1.10.
  const int cus = compute_units();
  const int64_t least = blocks > 3 * cus ? 131072 / DH : blocks * 5 > cus * 8 ? max(65536 / DH, 768) : 65536 / DH;    // rows
  p.by_length = a.kv_pos != nullptr && a.batch <= 64 && blocks > cus && (p.splits <= 2 || DH == 128) && a.kv_len >= least ? cus : 0;
  const dim3 grid = p.heads_first ? dim3(yheads, a.batch, p.splits) : dim3(p.splits, yheads, a.batch);
  bool eight = false;
  if constexpr (DH == 64 && G == 1) {
    eight = p.splits == 1 && eight_waves(a.batch, yheads, a.kv_len, DH, G);
    if (eight) attn_decode_kernel<DH, G, 8><<<grid, 8 * 64, 0, s>>>(p);
  }
  // Loads left to the scheduler: short caches of heads of 128, one query head each, in more blocks than CUs; waves without a tile
  // then request nothing (us, in place | free: 64 x 32 up to 64 rows 18.7 | 16.9, 51 x 32 up to 119 17.3 | 15.9; 66 drawn calls up to
  // 128 rows 5.4 % less, 48 up to 300 1.3 %, longer ones alike; with a block per CU at most 15 x 16 up to 73 4.5 | 4.9).  A branch
  // around the loads in place does the same for those and makes every wait of the loop a full one: 33 x 8 up to 358 11.1 | 12.5.
  bool free_loads = false;
  if constexpr (DH == 128 && G == 1) {
    free_loads = p.splits == 1 && blocks > cus && a.kv_len <= 256;
    if (free_loads) attn_decode_kernel<DH, G, 4, true><<<grid, 4 * 64, 0, s>>>(p);
  }
  if (!eight && !free_loads) attn_decode_kernel<DH, G, 4><<<grid, 4 * 64, 0, s>>>(p);
  if (p.splits == 1) return launch_status();
  if (hipGetLastError() != hipSuccess) return FORGE_ERR_HIP;
  attn_decode_combine<DH><<<dim3(a.q_heads, a.batch), DH, 0, s>>>(p.part, (bf16*)a.out, a.q_heads,
                                                                  yheads, p.splits);
  return launch_status();
}

template <int DH>
forge_status launch_d(const AttnArgs& a, const SplitPlan& pl, hipStream_t s) {
  switch (heads_per_block(a.q_heads / a.kv_heads)) {
    case 1: return launch_dg<DH, 1>(a, pl, s);
    case 2: return launch_dg<DH, 2>(a, pl, s);
    case 3: return launch_dg<DH, 3>(a, pl, s);
    case 4: return launch_dg<DH, 4>(a, pl, s);
    case 5: return launch_dg<DH, 5>(a, pl, s);
    case 6: return launch_dg<DH, 6>(a, pl, s);
    case 7: return launch_dg<DH, 7>(a, pl, s);
    case 8: return launch_dg<DH, 8>(a, pl, s);
    default: return FORGE_ERR_UNSUPPORTED;
  }
}

}  // namespace

namespace {
// partial rows of (query head, range) pairs, with their maximum and sum
inline size_t partial_bytes(int64_t pairs, int head_dim) { return (size_t)pairs * (head_dim + 2) * sizeof(float); }

// Groups that run on the vector-ALU kernel write no partials.  Their sizes stay those by which calls have been
// accepted and refused, the fixed array's among them: ranges of 256 rows, two blocks per CU.
inline size_t vector_group_bytes(int batch, int q_heads, int kv_heads, int kv_len, int head_dim) {
  const int64_t two_per_cu = ceil_div64(2 * (int64_t)compute_units(), (int64_t)batch * kv_heads);
  const int splits = (int)min(min(two_per_cu, (int64_t)MAX_SPLITS), (int64_t)(kv_len / 256));
  return splits > 1 ? partial_bytes((int64_t)batch * q_heads * splits, head_dim) : 0;
}
}  // namespace

// what a call of this batch has to bring: room for the ranges of any cache up to kv_len
size_t attn_decode_needed_bytes(int batch, int q_heads, int kv_heads, int kv_len, int head_dim) {
  if (heads_per_block(q_heads / kv_heads) == 0) return vector_group_bytes(batch, q_heads, kv_heads, kv_len, head_dim);
  const int splits = splits_bound(batch, block_heads(q_heads, kv_heads), kv_len);
  return splits > 1 ? partial_bytes((int64_t)batch * q_heads * splits, head_dim) : 0;   // else the blocks write the output
}

// The size to ask for: also what any smaller batch needs, which is cut into more ranges (24 sequences of 8 heads run
// uncut, 16 in two ranges): b * splits_bound(b) over all b <= batch is at most b + (2 CUs - 1) / heads, and 64 ranges of each;
// a batch of two blocks per CU is not cut.
size_t attn_decode_workspace_bytes(int batch, int q_heads, int kv_heads, int kv_len, int head_dim) {
  if (heads_per_block(q_heads / kv_heads) == 0) return vector_group_bytes(batch, q_heads, kv_heads, kv_len, head_dim);
  const int per_head = (2 * compute_units() - 1) / block_heads(q_heads, kv_heads);
  if (per_head < 1 || kv_len < MIN_CUT_ROWS) return 0;
  const int64_t b = min(batch, per_head);
  return partial_bytes(min(b + per_head, b * min(MAX_SPLITS, kv_len / GRAIN)) * q_heads, head_dim);
}

// ---- scratch that nobody allocates -----------------------------------------------------------
// For callers that can neither allocate nor bring a workspace: the split-KV partials go to a
// fixed array in the library's own device image.  Each GPU holds its own copy at its own address;
// the name below is only a host-side handle for it, so host code looks the address up once per
// device (with that device current) and passes the pointer on, as it would a caller's workspace.
constexpr size_t kStaticScratchBytes = (size_t)4 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;

size_t attn_decode_static_scratch_bytes() { return kStaticScratchBytes; }

forge_status attn_decode_static_scratch(void** ptr) {
  static std::atomic<void*> per_device[kMaxDevices];   // zero-initialised; filled on first use
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return FORGE_ERR_HIP;
  if (dev < 0 || dev >= kMaxDevices) return FORGE_ERR_UNSUPPORTED;
  void* p = per_device[dev].load(std::memory_order_acquire);
  if (p == nullptr) {
    // racing first calls look the same address up twice: harmless
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return FORGE_ERR_HIP;
    per_device[dev].store(p, std::memory_order_release);
  }
  *ptr = p;
  return FORGE_OK;
}

forge_status launch_attn_decode_bf16(const AttnArgs& a, hipStream_t s) {
  if (heads_per_block(a.q_heads / a.kv_heads) == 0) return launch_attn_simple_bf16(a, s);   // no pass count covers the group
  // what THIS launch writes (at most attn_decode_needed_bytes of any cache >= kv_len)
  const SplitPlan pl = plan_splits(a.batch, block_heads(a.q_heads, a.kv_heads), a.kv_len, a.head_dim,
                                   heads_per_block(a.q_heads / a.kv_heads), a.kv_pos != nullptr);
  const size_t need = pl.splits == 1 ? 0 : partial_bytes((int64_t)a.batch * a.q_heads * pl.splits, a.head_dim);
  if (need > 0 && (a.workspace == nullptr || a.workspace_bytes < need)) return FORGE_ERR_WORKSPACE;
  if (a.head_dim == 64) return launch_d<64>(a, pl, s);
  if (a.head_dim == 128) return launch_d<128>(a, pl, s);
  return FORGE_ERR_UNSUPPORTED;
}

}  // namespace forge
