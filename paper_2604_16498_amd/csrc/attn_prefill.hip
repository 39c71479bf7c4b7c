// bf16 fused causal attention for prefill on the gfx950 matrix cores: scores, scale, mask,
// softmax and the product with V in one kernel; S and P live only in registers.
//
// Work split: a block owns 32 consecutive queries per wave of one (batch, head), and each wave walks the
// keys in tiles of 64 up to its diagonal.  Blocks of 8 waves (one per CU) run the two waves of a SIMD half a
// tile apart (Pipeline, below); blocks of 4 or 2 waves run a tile's steps in order and leave the overlap to the other
// blocks of their CU.  launch_dh says which takes a call.
//
// Both contractions are computed TRANSPOSED so that the two MFMAs chain without any data
// movement:
//   S^T[key, query] = K . Q^T   : A operand = K rows (LDS, 128-bit reads along dh),
//                                 B operand = Q^T, i.e. each lane's own query row (registers).
//   O^T[d, query]   = V^T . P^T : B operand = P^T, which is exactly the accumulator layout of
//                                 S^T (lane = query, registers = keys) rounded to bf16;
//                                 A operand = V^T, read from the row-major V tile in LDS with
//                                 the transposing LDS read (ds_read_b64_tr_b16: within 16 lanes,
//                                 lane 4q+r receives element r of the 8-byte rows addressed by
//                                 lanes q, q+4, q+8, q+12).
// A lane therefore owns ONE query throughout: its 32 scores per tile sit in its own registers,
// the row maximum needs a single exchange with lane^32 (the other half of the keys), the row
// sum is kept as a per-lane partial and combined once at the end, and the rescale factor of
// the online softmax is a per-lane scalar (applied only when some lane's maximum moved).
//
// The contraction order over keys inside a 16-key MFMA step is permuted (the same permutation
// on both operands, so the sum is unchanged): element e of lane-half h is key
// 16 s + 8 (e / 4) + 4 h + e % 4, which is what the S^T accumulator registers 8 (s % 2) + e hold.
//
// Pipeline (8 waves): per wave and tile of 64 keys the softmax is ~1000 cycles of vector ALU work and the two
// contractions ~1100 cycles of MFMA, and a wave issues in order.  The matrix pipe and the vector ALU
// of a SIMD do overlap when they are fed by two DIFFERENT waves (measured: the MFMA stream keeps its
// pace, the vector stream loses about a quarter), so the work of a tile is cut into a pure vector
// phase (mask, maximum, rescale, all exponentials, rounding of P) and a pure matrix phase
// (P.V of that tile, then S of the next one), and the two waves that share a SIMD (w and w+4) run
// the same sequence HALF A TILE APART: while one is in its vector phase the other is in its matrix
// phase.  A block barrier ends every half tile.  Only one set of score registers is alive per wave.
//
// LDS: K tile rows padded by 16 B and V tile rows by 64 B (32 at head_dim 64) so that the row reads (K) and the
// 4-rows-by-64-B transposing reads (V) of a half wave fall on disjoint banks; two buffers each.
// Tiles go HBM -> registers -> LDS, moved by the early waves (0-3): K(t+1) is stored at the start of
// the softmax step of tile t and the loads of K(t+2) go out right behind it, V likewise at the start
// of the matrix step, so a load has a whole tile to arrive, across two barriers (which wait for LDS
// only: lds_barrier).  With the loads issued and stored inside one step, 1 x 32 heads x 4096 took 148.2 us
// against 145.8, 777 queries behind 2500 keys 96.4 against 92.2, and a dense mask (8 x 12 heads x 1000,
// whose loads the old barrier drained) 92.2 against 75.6.  (The same loads issue two to four times slower from waves 4-7, and
// direct-to-LDS loads were measured slower still: +15 %.)
//
// Blocks of 4 and 2 waves: all waves copy, one barrier per tile, and S, the softmax and P.V of a tile follow each other in a
// wave.  At head_dim 64 the vector work is twice the matrix work, the 8-wave kernel left two waves per SIMD
// with it (154 registers) and its blocks filled the chip in 1.5 rounds at 8 x 12 heads x 1024; three blocks of 4 waves fit a
// CU (133 registers, 39 KB).  us, 8 waves | 4 waves: 8 x 12 heads of 64 x 1024 causal 31.8 | 27.7, x 600 20.4 | 16.0, the
// same dense 54 | 41.5, masked 82.6 | 60; head_dim 128 (two blocks per CU): 32 heads x 300 15.1 | 11.2, x 1500 49.6 | 42.4.
#include "common.hpp"

namespace forge {
namespace {

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

struct AttnParams {
  const bf16* q;
  const bf16* k;
  const bf16* v;
  bf16* out;
  int batch, q_heads, kv_heads, q_len, kv_len;
  int64_t kv_bs, kv_hs;
  float scale, scale_log2e;
  int causal;
  int n_qblocks;
  const float* mask;        // additive, fp32 [*, *, q_len, kv_len]; only read by the MASKED kernel
  int64_t mask_bs, mask_hs;
  float* part;              // SPLIT: fp32 partial rows [splits][batch * q_heads * q_len][dh], then (max, sum) pairs
  int splits;
  int round;                // > 0: every other round of this many blocks runs backwards
};

__device__ inline float xchg32_max(float x) {
  // max over the lane pair (l, l^32)
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float xchg32_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// MASKED: an additive mask (the optional mask node of the paper's attention chain) is added to
// the scaled scores before the softmax.  A lane's 32 mask values of a tile (its query row, the keys
// its score registers hold: 8 groups of 4 consecutive keys) are requested at the end of the
// preceding matrix phase, 16 bytes per load, and arrive behind the half-tile barrier.
// SPLIT: block z of a query block walks only its share of the key tiles and writes unnormalised fp32
// rows with their (maximum, sum); attn_prefill_merge adds the shares.  For calls with fewer query blocks
// than CUs (a turn of 777 tokens has 4 per head).
// head_dim 64, 4 waves: three blocks on a CU, with a mask by one register (168, left to itself 169; us, two blocks | three:
// 8 x 12 heads of 64 x 1000 masked 68.6 | 62.7, 7 x 12 x 800 53.7 | 48.7, 11 x 12 x 500 36.0 | 31.4, with at most two to
// place, 6 x 12 x 700 and fewer, alike).
template <int DH, bool MASKED, bool SPLIT, int WAVES>
__global__ __launch_bounds__(WAVES * 64, WAVES == 8 ? 1 : DH == 128 || (MASKED && WAVES == 2) ? 2 : 3) void attn_prefill_kernel(AttnParams p) {
  constexpr int BQ = WAVES * 32, BKV = 64;
  constexpr int CPR = DH / 8;                 // 16-byte chunks per row
  constexpr int KS = DH * 2 + 16;             // K row stride in LDS (bytes)
  constexpr int VS = DH * 2 + (DH == 64 ? 32 : 64);   // V row stride in LDS (bytes)
  constexpr int K_BYTES = BKV * KS, V_BYTES = BKV * VS;
  // chunks per thread, tensor and tile: the early waves move the tiles (measured: the same loads
  // issue two to four times slower from the second wave of a SIMD)
  constexpr int COPY = WAVES < 4 ? WAVES * 64 : 256;   // copying threads
  constexpr int LPT = BKV * CPR / COPY;       // per thread of the early waves; the late waves copy nothing
  constexpr int NKS = DH / 16;                // MFMA k-steps over dh
  constexpr int NDT = DH / 32;                // 32-row tiles of O^T
  extern __shared__ __attribute__((aligned(16))) char smem[];   // [K0 | K1 | V0 | V1]
  char* const kbuf = smem;
  char* const vbuf = smem + 2 * K_BYTES;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int fr = lane & 31, fh = lane >> 5;
  // late (long) query blocks first, over all heads: they carry the most key tiles under the
  // causal mask, and blocks are handed out in launch order
  // (and the blocks that are resident from the start are dealt there and back over the CUs: a CU's later blocks come a round of
  // the chip after its first, and forwards some would hold the longest of every round)
  int at = blockIdx.x;
  const int pairs = p.batch * p.q_heads;
  constexpr bool ROUNDS = DH == 64 && WAVES == 4 && !SPLIT;
  if (ROUNDS && p.round > 0) {
    const int from = at - at % p.round;
    if ((at / p.round) & 1) at = 2 * from + min((int)gridDim.x - from, p.round) - 1 - at;
  }
  int qb = p.n_qblocks - 1 - at / pairs;
  int h = at % pairs % p.q_heads, b = at % pairs / p.q_heads;
  if (MASKED && p.mask_hs == 0) {
    // One mask for all heads: within a row of query blocks, those of neighbouring heads run on one XCD (blocks are dealt
    // round-robin over the 8), whose L2 then fetches their mask rows once; dealt over all of them, every L2 fetched
    // the whole mask (8 x 12 heads x 1000: 83 -> 70 us by this alone).  Every XCD gets its share of each row, so that a last
    // row that is mostly padding does not leave some of them idle (3 x 64 heads of 128 x 541 90 us with whole rows per XCD, 81).
    // Blocks r of this row with (r + o) % 8 == x are XCD x's; the k-th of them is pair (those of the XCDs before) + k.  (Where
    // every other round runs backwards x stands for XCD 7 - x in it, and a row that two rounds share has its masks in two L2s
    // there; causal 8 x 12 x 1024, rounds forwards | there and back, 46.9 | 43.1 all the same.)
    const int o = (at - at % pairs) & 7, x = at & 7, r = at % pairs;
    int item = r >> 3;
    for (int y = 0; y < x; ++y) item += (pairs - ((y - o) & 7) + 7) >> 3;
    h = item % p.q_heads;
    b = item / p.q_heads;
  }
  const int g = h / (p.q_heads / p.kv_heads);
  const int q0 = qb * BQ, q0w = q0 + wave * 32;
  const int off = p.kv_len - p.q_len;
  const bool late = WAVES == 8 && wave >= 4;                // the second wave of each SIMD runs half a tile behind (see above)

  const bf16* kbase = p.k + (int64_t)b * p.kv_bs + (int64_t)g * p.kv_hs;
  const bf16* vbase = p.v + (int64_t)b * p.kv_bs + (int64_t)g * p.kv_hs;

  // ---- this lane's query row as the B operand of S^T (registers for the whole kernel) ------
  const int my_q = q0w + fr;
  bf16x8 qf[NKS];
  {
    const int qr = min(my_q, p.q_len - 1);
    const bf16* qrow = p.q + (((int64_t)b * p.q_heads + h) * p.q_len + qr) * DH;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
      qf[ks] = *reinterpret_cast<const bf16x8*>(qrow + (2 * ks + fh) * 8);
    // pin the fragments in registers: otherwise the compiler re-loads them from global memory
    // inside the key loop and the score MFMAs wait on that latency every tile
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) asm volatile("" : "+v"(qf[ks]));
  }

  // keys a query may see: [0, limit]
  const int last_q_blk = min(q0 + BQ, p.q_len) - 1;
  const int all_tiles = ceil_div((p.causal ? last_q_blk + off : p.kv_len - 1) + 1, BKV);
  const int share = SPLIT ? ceil_div(all_tiles, p.splits) : all_tiles;
  const int t_first = SPLIT ? (int)blockIdx.z * share : 0;            // this block's tiles: [t_first, n_tiles)
  const int n_tiles = min(all_tiles, t_first + share);                // (none: neutral rows, maximum -1e30, sum 0)
  const int my_limit = p.causal ? my_q + off : p.kv_len - 1;
  const int wave_max_limit = p.causal ? min(q0w + 31, p.q_len - 1) + off : p.kv_len - 1;
  const int wave_min_limit = p.causal ? q0w + off : p.kv_len - 1;

  // ---- global -> registers -> LDS copy plan: each early wave moves a quarter of a tile -------------
  int ld_row[LPT], ld_c[LPT];
#pragma unroll
  for (int i = 0; i < LPT; ++i) {
    const int idx = (tid & (COPY - 1)) + i * COPY;
    ld_row[i] = idx / CPR;
    ld_c[i] = idx % CPR;
  }
  u32x4 rk[LPT], rv[LPT];
  auto load_rows = [&](const bf16* base, int t, u32x4 (&r)[LPT]) {
    if (late) return;
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      const int key = min(t * BKV + ld_row[i], p.kv_len - 1);   // rows past the end re-read the last key
      r[i] = *reinterpret_cast<const u32x4*>(base + (int64_t)key * DH + ld_c[i] * 8);
    }
  };
  auto store_k = [&](int buf) {
    if (late) return;
#pragma unroll
    for (int i = 0; i < LPT; ++i)
      *reinterpret_cast<u32x4*>(kbuf + buf * K_BYTES + ld_row[i] * KS + ld_c[i] * 16) = rk[i];
  };
  auto store_v = [&](int buf) {
    if (late) return;
#pragma unroll
    for (int i = 0; i < LPT; ++i)
      *reinterpret_cast<u32x4*>(vbuf + buf * V_BYTES + ld_row[i] * VS + ld_c[i] * 16) = rv[i];
  };

  floatx16 o_acc[NDT];
#pragma unroll
  for (int i = 0; i < NDT; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) o_acc[i][e] = 0.f;
  // finite start: no inf - inf anywhere; with a mask no value of it lies below (a row cut throughout by -1e30 or less has a maximum)
  float m_run = MASKED ? -__FLT_MAX__ : -1e30f, l_run = 0.f;
  // MASKED works on scaled scores with the mask added (s * scale + mask, one instruction), so the factor inside the softmax
  // is log2e there; the difference to the maximum is taken first and exactly: a mask may hold any finite value, and maximum * log2e
  // rounded by itself is off by 440 at -1e10
  const float c = MASKED ? 1.4426950408889634f : p.scale_log2e;
  const float* mask_row = nullptr;
  if (MASKED)
    mask_row = p.mask + b * p.mask_bs + h * p.mask_hs + (int64_t)min(my_q, p.q_len - 1) * p.kv_len;
  floatx4 mk[MASKED ? 8 : 1];      // mask values of the tile whose vector phase comes next
  // (a 16-byte load needs 4-byte alignment only, so rows of any length are read this way; the end of a
  // ragged row goes element by element.  8 x 12 heads x 1001: 254 -> 81 us, 2 x 16
  // heads of 128 x 511: 67 -> 32; x 1000, which was read this way before, 79 against 76)
  auto mask_prefetch = [&](int t) {
    if (!MASKED) return;
    typedef float floatx4_u __attribute__((ext_vector_type(4), aligned(4)));
    const float* mrow = mask_row + t * BKV + 4 * fh;                        // registers 4 (g8 & 3) .. + 3 of block g8 >> 2
    if ((t + 1) * BKV <= p.kv_len) {                                        // uniform
#pragma unroll
      for (int g8 = 0; g8 < 8; ++g8)
        mk[g8] = *reinterpret_cast<const floatx4_u*>(mrow + (g8 >> 2) * 32 + 8 * (g8 & 3));
    } else {
#pragma unroll
      for (int g8 = 0; g8 < 8; ++g8) {
        const int at = (g8 >> 2) * 32 + 8 * (g8 & 3), left = p.kv_len - (t * BKV + 4 * fh + at);
        floatx4 m = {0.f, 0.f, 0.f, 0.f};                                   // keys past the end are cut in the softmax
        if (left >= 4) m = *reinterpret_cast<const floatx4_u*>(mrow + at);
        else if (left > 0) {
          m[0] = mrow[at];
          if (left > 1) m[1] = mrow[at + 1];
          if (left > 2) m[2] = mrow[at + 2];
        }
        mk[g8] = m;
      }
    }
  };

  // per-lane byte offset of the transposing V read inside a tile (without key step / d tile)
  const int vt_lane = (((lane & 15) >> 2) + 4 * fh) * VS + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;

  // ---- matrix phase, part 2: S^T = K . Q^T of one tile ---------------------------------------------
  floatx16 sc[2];                  // the scores of the tile in flight, then its probabilities
  bf16x8 pf[4];                    // P^T of the tile whose vector phase has run: B operand of P.V
  auto scores = [&](int t) {
    const char* sk = kbuf + (t & 1) * K_BYTES;
    // (the first MFMA of each key block takes a zero accumulator as an inline constant)
    // K fragments run LA MFMAs ahead of their use so that no MFMA waits on an LDS read
    constexpr int NF = 2 * NKS, LA = 4;
    bf16x8 kf[LA];
    auto kread = [&](int i) {
      const int kb = i / NKS, ks = i % NKS;
      return *reinterpret_cast<const bf16x8*>(sk + (kb * 32 + fr) * KS + (2 * ks + fh) * 16);
    };
#pragma unroll
    for (int i = 0; i < LA; ++i) kf[i] = kread(i);
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      sc[i / NKS] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i % LA], qf[i % NKS], i % NKS == 0 ? zero : sc[i / NKS], 0, 0, 0);
      if (i + LA < NF) kf[i % LA] = kread(i + LA);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- vector phase: mask, online softmax, P rounded to bf16 (no matrix instruction) ----------------
  auto softmax = [&](int t) {
    const int kv0 = t * BKV;
    if (MASKED) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) sc[kb][v] = sc[kb][v] * p.scale + mk[kb * 4 + (v >> 2)][v & 3];
    }
    if (kv0 + BKV - 1 > wave_min_limit) {       // diagonal / tail tiles only
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = kv0 + kb * 32 + 8 * (v >> 2) + 4 * fh + (v & 3);
          if (key > my_limit) sc[kb][v] = -INFINITY;
        }
    }
    float mx = sc[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sc[kb][v]);
    mx = xchg32_max(mx);
    const float m_new = fmaxf(m_run, mx);
    if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {   // wave-uniform: some maximum moved
      const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c);
      l_run *= alpha;
#pragma unroll
      for (int i = 0; i < NDT; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) o_acc[i][e] *= alpha;
      m_run = m_new;
    }
    // (a row of a share may have no visible key in a tile that other rows need; its maximum is then the initial
    // -1e30, which a scale above 2.3e8 takes to -infinity, and hidden scores less it would be NaN)
    const float mc = SPLIT ? fmaxf(m_run * c, -3.4e38f) : m_run * c;
    float psum = 0.f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float pv = __builtin_amdgcn_exp2f(MASKED ? (sc[kb][v] - m_run) * c : sc[kb][v] * c - mc);
        sc[kb][v] = pv;
        psum += pv;
      }
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int e = 0; e < 8; ++e) pf[2 * kb + s2][e] = (bf16)sc[kb][8 * s2 + e];
    }
    l_run += psum;
  };

  // ---- matrix phase, part 1: O^T += V^T . P^T --------------------------------------------------------
  auto pv_mm = [&](int t) {
    const char* sv = vbuf + (t & 1) * V_BYTES;
    // V^T fragments (two transposing reads each) run LA MFMAs ahead of their use
    constexpr int NF = 4 * NDT, LA = 4;
    typedef short v8i16 __attribute__((ext_vector_type(8)));
    v4i16 lo[LA], hi[LA];
    auto vread = [&](int i, v4i16& l, v4i16& hh) {
      const int s = i / NDT, dt = i % NDT;
      const char* va = sv + vt_lane + (16 * s) * VS + dt * 64;
      l = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(va));
      hh = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(va + 8 * VS));
    };
#pragma unroll
    for (int i = 0; i < LA; ++i) vread(i, lo[i], hi[i]);
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      const v4i16 l = lo[i % LA], hh = hi[i % LA];
      v8i16 both = {l[0], l[1], l[2], l[3], hh[0], hh[1], hh[2], hh[3]};
      o_acc[i % NDT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pf[i / NDT], o_acc[i % NDT], 0, 0, 0);
      if (i + LA < NF) vread(i + LA, lo[i % LA], hi[i % LA]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto wave_needs = [&](int t) { return t < n_tiles && t * BKV <= wave_max_limit; };   // wave-uniform

  // ---- prologue: the first tile's K and V in LDS, the second's on their way, the first's S in registers ----
  load_rows(kbase, t_first, rk);
  load_rows(vbase, t_first, rv);
  store_k(t_first & 1);
  store_v(t_first & 1);
  load_rows(kbase, t_first + 1, rk);   // (tiles past the end re-read the last key: a branch around the
  load_rows(vbase, t_first + 1, rv);   // loads would make the waits of the loop drain them all)
  if (WAVES < 8 && wave_needs(t_first)) mask_prefetch(t_first);
  lds_barrier();
  if constexpr (WAVES < 8) {
    // Tile t + 1 goes into the other buffers, whose last readers finished tile t - 1 before the barrier; the
    // register loads of tile t + 2 follow.  One barrier per tile.
    for (int t = t_first; t < n_tiles; ++t) {
      if (t + 1 < n_tiles) {
        store_k((t + 1) & 1);
        store_v((t + 1) & 1);
      }
      load_rows(kbase, t + 2, rk);
      load_rows(vbase, t + 2, rv);
      if (wave_needs(t)) {
        scores(t);
        softmax(t);
        if (wave_needs(t + 1)) mask_prefetch(t + 1);
        if (!MASKED) pv_mm(t);
      }
      // (with a mask in a branch of its own: masked 8 x 12 heads of 64 x 1000 65.5 us in the one above, 62.7; without a mask the
      // second branch costs: 2 x 12 x 267 8.0 | 7.75, 1 x 12 x 578 12.3 | 11.9)
      if (MASKED && wave_needs(t)) pv_mm(t);
      lds_barrier();
    }
  } else {
    if (wave_needs(t_first)) {
      scores(t_first);
      mask_prefetch(t_first);
    }
    lds_barrier();

    // Steps of half a tile, a block barrier after each; the late waves run one step behind:
    //   step 2t   : early waves  softmax(t), copy of K(t+1)           late waves  P.V(t-1), S(t)
    //   step 2t+1 : early waves  P.V(t), S(t+1), copy of V(t+1)      late waves  softmax(t)
    // K(t+1) goes into K buffer (t+1)&1 in step 2t; its last reader was the late waves' S(t-1) in step
    // 2t-2, and it is first read by the early waves' S(t+1) in step 2t+1.  V(t+1) goes into V buffer (t+1)&1
    // in step 2t+1; last read by the late waves' P.V(t-1) in step 2t, first read by the early waves'
    // P.V(t+1) in step 2t+3.  The register loads of tile t+2 follow each store.
    auto matrix_phase = [&](int t) {
      if (wave_needs(t)) pv_mm(t);
      if (wave_needs(t + 1)) {
        scores(t + 1);
        mask_prefetch(t + 1);
      }
    };
    if (!late) {
      for (int t = t_first; t < n_tiles; ++t) {
        if (t + 1 < n_tiles) store_k((t + 1) & 1);
        load_rows(kbase, t + 2, rk);
        if (wave_needs(t)) softmax(t);
        lds_barrier();
        if (t + 1 < n_tiles) store_v((t + 1) & 1);
        load_rows(vbase, t + 2, rv);
        matrix_phase(t);
        lds_barrier();
      }
      lds_barrier();                     // the late waves' last step
    } else {
      lds_barrier();                     // the early waves' first step
      for (int t = t_first; t < n_tiles; ++t) {
        if (wave_needs(t)) softmax(t);
        lds_barrier();
        matrix_phase(t);
        lds_barrier();
      }
    }
  }

  // ---- normalise and store: lane owns query my_q; registers 4g..4g+3 are 4 consecutive d -----
  const float l_tot = xchg32_sum(l_run);
  if constexpr (SPLIT) {
    if (my_q >= p.q_len) return;
    const int64_t rows = (int64_t)pairs * p.q_len, row = (int64_t)(b * p.q_heads + h) * p.q_len + my_q;
    float* prow = p.part + ((int64_t)blockIdx.z * rows + row) * DH;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int gg = 0; gg < 4; ++gg)
        *reinterpret_cast<floatx4*>(prow + dt * 32 + 8 * gg + 4 * fh) =
            floatx4{o_acc[dt][4 * gg], o_acc[dt][4 * gg + 1], o_acc[dt][4 * gg + 2], o_acc[dt][4 * gg + 3]};
    if (fh == 0) {
      floatx2* ml = reinterpret_cast<floatx2*>(p.part + (int64_t)p.splits * rows * DH);
      ml[(int64_t)blockIdx.z * rows + row] = floatx2{m_run * c, l_tot};
    }
    return;
  }
  if (my_q < p.q_len) {
    const float inv = 1.0f / l_tot;
    bf16* orow = p.out + ((int64_t)b * p.q_len + my_q) * ((int64_t)p.q_heads * DH) + (int64_t)h * DH;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int gg = 0; gg < 4; ++gg) {
        u32x2 pk;
        pk[0] = pack_bf2(o_acc[dt][4 * gg] * inv, o_acc[dt][4 * gg + 1] * inv);
        pk[1] = pack_bf2(o_acc[dt][4 * gg + 2] * inv, o_acc[dt][4 * gg + 3] * inv);
        *reinterpret_cast<u32x2*>(orow + dt * 32 + 8 * gg + 4 * fh) = pk;
      }
  }
}

constexpr int MAX_SHARES = 8;

// Merge of the key shares: DH / 8 lanes per row, 8 columns each; shares in order.
template <int DH>
__global__ __launch_bounds__(256) void attn_prefill_merge(const float* __restrict__ part, bf16* __restrict__ out,
                                                          int q_heads, int q_len, int64_t rows, int splits) {
  constexpr int LPR = DH / 8;
  const int64_t row = (int64_t)blockIdx.x * (256 / LPR) + threadIdx.x / LPR;
  const int c = threadIdx.x % LPR;
  if (row >= rows) return;
  // all maxima and sums and the rows of the first P shares in one round trip, from clamped addresses
  const floatx2* ml = reinterpret_cast<const floatx2*>(part + (int64_t)splits * rows * DH);
  constexpr int P = 4;
  floatx2 t[MAX_SHARES];
  float v[P][8];
#pragma unroll
  for (int z = 0; z < MAX_SHARES; ++z) t[z] = ml[min(z, splits - 1) * rows + row];
#pragma unroll
  for (int z = 0; z < P; ++z) Vec8<float>::load(part + (min(z, splits - 1) * rows + row) * DH + c * 8, v[z]);
  float mx = t[0][0];
#pragma unroll
  for (int z = 1; z < MAX_SHARES; ++z) mx = fmaxf(mx, t[z][0]);
  float o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, l = 0.f;
#pragma unroll
  for (int z0 = 0; z0 < MAX_SHARES; z0 += P) {
    if (z0 >= splits) break;
    if (z0 > 0) {
#pragma unroll
      for (int z = 0; z < P; ++z) Vec8<float>::load(part + (min(z0 + z, splits - 1) * rows + row) * DH + c * 8, v[z]);
    }
#pragma unroll
    for (int z = 0; z < P; ++z) {                           // (selects: a weight of 0 would turn an infinite output into NaN)
      const bool in = z0 + z < splits;
      const float w = __builtin_amdgcn_exp2f(t[z0 + z][0] - mx);
      l += in ? t[z0 + z][1] * w : 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] += in ? v[z][e] * w : 0.f;
    }
  }
  const float inv = 1.0f / l;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] *= inv;
  const uint32_t bh = (uint32_t)row / (uint32_t)q_len, b = bh / (uint32_t)q_heads, h = bh - b * q_heads;   // (shares: few rows)
  const int64_t q = (uint32_t)row - bh * (uint32_t)q_len;
  Vec8<bf16>::store(out + (((int64_t)b * q_len + q) * q_heads + h) * DH + c * 8, o);
}

template <int DH, bool MASKED, bool SPLIT, int WAVES>
forge_status launch_split(const AttnArgs& a, int splits, hipStream_t s) {
  AttnParams p;
  p.q = (const bf16*)a.q;
  p.k = (const bf16*)a.k;
  p.v = (const bf16*)a.v;
  p.out = (bf16*)a.out;
  p.batch = a.batch;
  p.q_heads = a.q_heads;
  p.kv_heads = a.kv_heads;
  p.q_len = a.q_len;
  p.kv_len = a.kv_len;
  p.kv_bs = a.kv_batch_stride;
  p.kv_hs = a.kv_head_stride;
  p.scale = a.scale;
  p.scale_log2e = a.scale * 1.4426950408889634f;
  p.causal = a.causal;
  p.n_qblocks = ceil_div(a.q_len, WAVES * 32);
  const int64_t grid_x = (int64_t)a.q_heads * a.batch * p.n_qblocks;
  p.part = (float*)a.workspace;
  p.splits = splits;
  p.mask = a.mask;
  p.mask_bs = a.mask_batch_stride;
  p.mask_hs = a.mask_head_stride;
  // There and back where up to three blocks per CU, all resident from the start, differ in many steps of length: 2 to 3 rounds of the
  // chip and 7 query blocks per head or more (17 drawn calls 1 to 7 % faster, us 8 x 12 heads of 64 x 1024 31.0 | 28.9, 6 x 12
  // x 902 22.7 | 21.4).  Fewer query blocks: 28 x 12 x 210 12.9 | 14.4, 13 x 12 x 418 16.8 | 17.7; more than three blocks, which
  // are handed out as others end: 16 x 12 x 1024 52.4 | 56, 4 x 32 x 1500 63.8 | 66; up to two rounds, and with two blocks per CU
  // (heads of 128) within the spread of the runs.
  p.round = DH == 64 && WAVES == 4 && !SPLIT && a.causal && p.n_qblocks >= 7 && grid_x > 2 * compute_units() && grid_x <= 3 * compute_units()
                ? compute_units() : 0;
  constexpr int smem = 2 * 64 * ((DH * 2 + 16) + (DH * 2 + (DH == 64 ? 32 : 64)));
  auto kern = attn_prefill_kernel<DH, MASKED, SPLIT, WAVES>;
  static std::atomic<uint64_t> lds_raised{0};   // per kernel instantiation
  if (raise_lds_limit(reinterpret_cast<const void*>(kern), smem, lds_raised) != FORGE_OK) return FORGE_ERR_HIP;
  dim3 grid((unsigned)grid_x, 1, splits), block(WAVES * 64);
  kern<<<grid, block, smem, s>>>(p);
  if (!SPLIT) return launch_status();
  if (hipGetLastError() != hipSuccess) return FORGE_ERR_HIP;
  const int64_t rows = (int64_t)a.batch * a.q_heads * a.q_len;
  attn_prefill_merge<DH><<<(unsigned)ceil_div64(rows, 256 / (DH / 8)), 256, 0, s>>>(p.part, p.out, a.q_heads, a.q_len, rows, splits);
  return launch_status();
}

// Blocks of w waves that a call has.
inline int64_t query_blocks(int batch, int q_heads, int q_len, int w) { return (int64_t)batch * q_heads * ceil_div(q_len, 32 * w); }

// Key shares of a call on blocks of w (4 or 8) waves: only where its query blocks leave CUs idle, at most 8 and none shorter than
// 256 keys.  What a 64-key tile takes a block depends on how many of them a CU holds, the merge launch costs 4.5 us and
// a share's partial rows go out and back at about 5 TB/s; the count with the least time is non-decreasing
// in kv_len (fewer tiles per share against a fixed cost).  us, merge included, unsplit | shares: 80 queries behind 1000 keys
// (12 heads of 64) 17.9 | 11.2 (4), 30 behind 2500 37.6 | 13.2 (8), 2 x 777 behind 2500 50 | 36 (3); heads of 128, 32 of them: 80 behind
// 4000 87 | 24.6 (8), 300 behind 1000 32.5 | 26.9 (2), 500 behind 2500 69 | 45 (4), 777 behind 0 23.2 | 29.4 (2).
inline int plan_shares(int batch, int q_heads, int q_len, int kv_len, int head_dim, int w) {
  const int64_t cus = compute_units(), blocks = query_blocks(batch, q_heads, q_len, w);
  const int per_cu = w == 8 ? 1 : head_dim == 128 ? 2 : 3;
  const int most = (int)min(min(per_cu * cus / blocks, (int64_t)kv_len / 256), (int64_t)MAX_SHARES);
  const double tiles = kv_len / 64.0, share_us = (double)((int64_t)batch * q_heads * q_len) * head_dim * 8 / 5e6;
  auto tile_us = [&](int n) {
    const int64_t r = ceil_div64(blocks * n, cus);       // blocks on the fullest CU
    if (w == 8) return 1.5;
    if (head_dim == 128) return r <= 1 ? 1.4 : 1.9;
    return r <= 1 ? 0.95 : r == 2 ? 1.35 : 1.9;
  };
  int best = 1;
  double least = tile_us(1) * tiles;
  for (int n = 2; n <= most; ++n) {
    const double us = tile_us(n) * tiles / n + 4.5 + share_us * n;
    if (us < least) { least = us; best = n; }
  }
  return best;
}

// head_dim 128: blocks of 8 waves where they fill the chip.  With key shares: at least 1700 keys, query blocks not mostly
// padding, nine tenths of the chip, or of up to three shares seven tenths without the padding (us, 8 waves | 4, 32 heads: 988
// queries over 1564 keys 41.3 | 40.5, 777 over 1777 44.6 | 46.6, over 3277 67.4 | 70, 512 over 2012 34.4 | 35.7, 1024 over
// 2424 53.5 | 59.1, over 4096 84 | 91; 12 heads x 1533 over 2481, 216 blocks, 40.0 | 43.5, 2 x 16 x 750 over 1953, 192 blocks,
// 43.6 | 48.5; but 256 over 2056, 224 blocks in seven shares, 28.1 | 25.8, 600 over 3500, 192 with padding, 66 | 58,
// 300 behind 3700 49 | 46).  Unsplit: whole query blocks, well past one round of them (32 heads x 4000 153 | 167, 3 x 16 x 2048
// 71 | 75, but 32 x 2500, 1.25 rounds, 84 | 76, 3 x 32 x 1300, 15 % padding, 84 | 75, 32 x 2048, one round, 65 | 58).
inline bool eight_waves_split(int batch, int q_heads, int q_len, int kv_len, int shares) {
  if (shares < 2 || kv_len < 1700 || q_len * 10 < ceil_div(q_len, 256) * 256 * 7) return false;
  const int64_t cus = compute_units();
  return query_blocks(batch, q_heads, q_len, 8) * shares * 10 >= cus * 9 ||
         (shares <= 3 && (int64_t)batch * q_heads * q_len * shares * 10 >= cus * 256 * 7);
}
inline bool eight_waves(int batch, int q_heads, int q_len) {
  return (int64_t)q_len * 100 >= (int64_t)ceil_div(q_len, 256) * 256 * 93 &&
         query_blocks(batch, q_heads, q_len, 8) * 10 >= (int64_t)compute_units() * 14;
}

template <int DH, bool MASKED>
forge_status launch_dh(const AttnArgs& a, hipStream_t s) {
  const int64_t cus = compute_units();
  if constexpr (!MASKED) {
    // (the workspace is optional: without it, or with less, the call runs unsplit)
    const size_t room = a.workspace != nullptr ? a.workspace_bytes / attn_prefill_share_bytes(a.batch, a.q_heads, a.q_len, DH) : 0;
    auto shares_on = [&](int w) {
      const int n = plan_shares(a.batch, a.q_heads, a.q_len, a.kv_len, DH, w);
      return room >= (size_t)n ? n : a.fewer_shares ? (int)room : 1;
    };
    if constexpr (DH == 128) {
      const int n = shares_on(8);
      if (eight_waves_split(a.batch, a.q_heads, a.q_len, a.kv_len, n)) return launch_split<DH, false, true, 8>(a, n, s);
    }
    const int n = shares_on(4);
    if (n > 1) return launch_split<DH, false, true, 4>(a, n, s);
  }
  // half as many queries per block while that leaves one block per CU (us, 4 waves | 2: 12 heads of 64 x 500 11.2 | 10.5, x 128
  // 5.9 | 5.1, masked x 1000 26 | 22; 2 x 12 x 700 masked, 264 blocks, 20 | 22.5; 32 heads of 128 x 80 7.5 | 6.2)
  if constexpr (!(MASKED && DH == 128)) {
    if (query_blocks(a.batch, a.q_heads, a.q_len, 2) <= cus) return launch_split<DH, MASKED, false, 2>(a, 1, s);
  }
  if constexpr (DH == 128) {
    // (the mask's registers leave no room for a second block; 16 heads x 1000 46 | 36, 3 x 16 x 700, 288 blocks of 4 waves, 36 | 40)
    // blocks of one length (no causal cut, or few new queries) that are one round of 8 waves or less, and more than one per CU
    // of 4: the half-filled CUs of the smaller blocks cost more than the larger ones' idle ones (us, 4 waves | 8, not causal:
    // 16 heads x 2499 behind 2502 keys 158 | 139, 3 x 16 x 944 38.8 | 35.2, 5 x 32 x 134 behind 670 33.3 | 29.4)
    const bool even = !a.causal || a.kv_len / 3 >= a.q_len;
    const int64_t blocks4 = query_blocks(a.batch, a.q_heads, a.q_len, 4), blocks8 = query_blocks(a.batch, a.q_heads, a.q_len, 8);
    if (MASKED ? blocks4 > cus : eight_waves(a.batch, a.q_heads, a.q_len) || (even && blocks4 > cus && blocks8 <= cus))
      return launch_split<DH, MASKED, false, 8>(a, 1, s);
  }
  return launch_split<DH, MASKED, false, 4>(a, 1, s);
}

}  // namespace

forge_status launch_attn_prefill_bf16(const AttnArgs& a, hipStream_t s) {
  if (a.head_dim == 64) return a.mask ? launch_dh<64, true>(a, s) : launch_dh<64, false>(a, s);
  if (a.head_dim == 128) return a.mask ? launch_dh<128, true>(a, s) : launch_dh<128, false>(a, s);
  return FORGE_ERR_UNSUPPORTED;
}

// Non-decreasing in kv_len (both share counts are), so that a buffer sized for a cache's capacity serves
// every shorter length.
size_t attn_prefill_workspace_bytes(int batch, int q_heads, int q_len, int kv_len, int head_dim) {
  int shares = plan_shares(batch, q_heads, q_len, kv_len, head_dim, 4);
  if (head_dim == 128) shares = max(shares, plan_shares(batch, q_heads, q_len, kv_len, head_dim, 8));
  return shares > 1 ? shares * attn_prefill_share_bytes(batch, q_heads, q_len, head_dim) : 0;
}

}  // namespace forge
