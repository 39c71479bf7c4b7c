// bf16 / weight-only-int8 linear for at most 64 rows of x (a decode step), and for some prompts of up to 128 rows in two chunks.
//
// HBM-bound: the weight is streamed once and nothing else of its size moves.  What the kernel is
// built around is that so few rows of x fit in REGISTERS: a block of 8 waves owns one k range of up
// to 4096 elements (2048 above 32 rows), every wave a contiguous eighth of it, and a wave holds its
// share of x as the B operands of v_mfma_f32_16x16x32_bf16 for its whole life.  The block then walks
// over tiles of 16 weight rows without a barrier between them.  Per tile a wave loads its part of the
// 16 rows straight from HBM in the A operand's layout (lane = row l%16, 16-byte chunk l/16: 64
// contiguous bytes of each row per load, no LDS) and refills each register from further on as soon as
// it has been multiplied: a tile's steps per wave, up to 10 KB (half of them above that: 8 KB at 4096 elements),
// are always in flight, 1 KB per step, and no vector-memory request is spent on re-reading activations,
// which is what holds back the slab-wise streaming kernel.
// The 8 partial sums of up to 8 tiles are collected in LDS; then every wave adds those of one tile in
// wave order and finishes its outputs (weight scale, bias, activation, residual, head split, rotation).
// Up to 4096 elements of K that is the whole reduction: no partial planes and no second launch.
// Beyond that, or where a row norm follows, each k range writes an fp32 plane for the reduce kernels.
//
// Measured against the slab-wise kernel and its reduce launch (us, cold weights): 2304 x 768 at 5
// rows 10.3 -> 4.0, 2048 x 2048 at 24 rows 10.4 -> 6.3, gated 28672 x 4096 at 5 rows 50 -> 43
// (5.5 TB/s), the same on int8 weights at 24 rows 35.8 -> 27.3.  Small ones are bound by the chain
// launch, x, weights, sums; large ones by HBM.
//
// Tile rows: a head split with rotation takes 8 columns of the first half of a head and their 8
// partners, the gated activation 8 gate rows and their 8 up rows, so that both members of a pair
// are in one tile (lanes l and l^32 of the finishing wave).
#include <math.h>
#include <type_traits>
#include "gemm_bf16.hpp"

namespace forge {
namespace {

constexpr int NW = 8;             // waves per block
constexpr int TR = 16;            // weight rows per tile
constexpr int MAX_ROWS = 64;      // rows of x of a decode step (four B operands of 16 columns)

struct RowsParams {
  GemmParams g;                   // g.N: output columns
  int rows;                       // weight rows
  int tiles;                      // row tiles
  int spw;                        // steps per wave in use
  int act;                        // activation of a finished output
  int qkv;                        // head split
  double l2_base;                 // log2 of the rotation's base
};

// What a tile ends in.  (Separate instantiations: the fp64 angles and the activations would otherwise
// cost every variant the registers that x and the tile in flight need.)
enum Finish { FIN_RAW = 0, FIN_OUT = 1, FIN_ROPE = 2 };

// rows of x a step multiplies at once are MT groups of 16; STEPS: 64-byte steps of a weight row per wave
template <int MT, int STEPS, bool W8, int FIN>
struct Rows {
  static constexpr int XF = W8 ? 2 : 1;                   // 32-k MFMA steps per 64 bytes
  static constexpr int KE = 32 * XF;                      // k per step
  static constexpr int XREGS = MT * STEPS * XF * 4;
  static constexpr int WIN = STEPS > 10 ? STEPS / 2 : STEPS;   // loads in flight per wave
  static_assert(STEPS % WIN == 0, "a tile is whole windows");
  static_assert(XREGS + WIN * 4 <= 160, "x and the tile in flight stay in registers");
  // tiles whose partial sums are collected in LDS before they are finished: one per wave where the
  // LDS of the CU holds them
  static constexpr int SLOTS = MT <= 2 ? 8 : 16 / MT;
  static constexpr int RED = SLOTS * NW * MT * 1024;
  static constexpr int XROW = STEPS * 64 * XF + 16, PATCH = 16 * XROW;   // x staging of one wave
  static constexpr int BASE = RED > NW * PATCH ? RED : NW * PATCH;
  static constexpr int SMEM = BASE + (FIN == FIN_ROPE ? SLOTS * MT * 1024 : 0);
  static_assert(SMEM <= 160 * 1024, "fits the LDS of a CU");
  static constexpr int READS = XREGS + WIN * 4 <= 96 ? NW - 1 : 2;       // partial sums read at once (more cost registers that x needs)
};

template <int MT, int STEPS, bool W8, int FIN>
__global__ __launch_bounds__(NW * 64) void gemm_bf16_rows_kernel(RowsParams r) {
  using C = Rows<MT, STEPS, W8, FIN>;
  const GemmParams& p = r.g;
  constexpr bool RAW = FIN == FIN_RAW, ROPE = FIN == FIN_ROPE;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  floatx4* const red = reinterpret_cast<floatx4*>(smem);            // [SLOTS][NW][MT][64 lanes]
  floatx2* const cs = reinterpret_cast<floatx2*>(smem + C::BASE);    // [SLOTS][MT * 128]: cos, sin of a rotating tile's (row, pair)

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  const int N = p.N, K = p.K;
  const int mz = blockIdx.z * (16 * MT);                 // this block's rows of x: [mz, mz + M)
  const int M = min(16 * MT, p.M - mz);
  const bool gated = FIN == FIN_OUT && r.act == FORGE_ACT_SWIGLU;

  // this wave's steps: [s0, s0 + ns) of the K / KE steps of a row (ns may be 0 in the last waves)
  const int total = K / C::KE;
  const int s0 = (blockIdx.y * NW + wave) * r.spw;
  const int ns = max(0, min(r.spw, total - s0));
  const int sl = min(s0, total - STEPS);                 // first step loaded: all STEPS lie inside the row (plan_rows)
  const int skip = s0 - sl;                              // ... of which [skip, skip + ns) are this wave's

  // ---- weight rows of a tile ---------------------------------------------------------------------
  // row index behind tile row i; rows past the end re-read the last one (their outputs are dropped)
  const int half = ROPE ? p.sp.head_dim / 2 : 8, octs = half / 8;
  auto w_row = [&](int tile, int i) {
    if (gated) return i < 8 ? min(tile * 8 + i, N - 1) : N + min(tile * 8 + i - 8, N - 1);
    if (ROPE) return (tile / octs) * 2 * half + (tile % octs) * 8 + (i < 8 ? i : half + i - 8);
    return min(tile * TR + i, r.rows - 1);
  };
  const char* wb = W8 ? (const char*)p.w8 : (const char*)p.w;
  const int64_t row_bytes = (int64_t)K * (W8 ? 1 : 2);
  const int in_row = sl * 64 + lg * 16;
  auto src_of = [&](int tile) { return wb + w_row(tile, lr) * row_bytes + in_row; };
  auto load = [&](const char* src, int s) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src + s * 64)); };

  // position of x row `lane` for the rotation and of its sequence for the cache rows (fetched here: behind the weight loads
  // they would wait for them)
  const bool split = ROPE || (FIN == FIN_OUT && r.qkv);
  int my_pos = 0, my_seq_pos = 0;
  if (split) {
    const int m = p.row0 + mz + min(lane, M - 1), b = p.sp.q_len == 1 ? m : m / p.sp.q_len;
    my_seq_pos = seq_position(p.sp.pos, b, p.sp.pos0);
    my_pos = my_seq_pos + m - b * p.sp.q_len;
  }

  // ---- x: whole pieces of rows (64 consecutive lanes, consecutive 16-byte chunks), put into the operand
  // layout through a patch of LDS of this wave's own.  (Loaded in the operand's layout, 16 rows by 16
  // bytes per quarter wave, x cost a cache-line lookup per 16 bytes: 5 us of 20 for 24 rows of 4096.)
  constexpr int XCH = STEPS * 4 * C::XF;                  // 16-byte chunks of a row in this wave's range
  constexpr int XL = 16 * XCH / 64;                       // wave-wide loads per group of 16 rows
  u32x4 xt[MT][XL];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int i = 0; i < XL; ++i) {
      const int m = mt * 16 + (i * 64 + lane) / XCH, c = (i * 64 + lane) % XCH;
      // (rows past the end re-read the last one; skipped by a branch, they cost a wait per load)
      xt[mt][i] = *reinterpret_cast<const u32x4*>(p.x + (int64_t)(mz + min(m, M - 1)) * K + sl * C::KE + c * 8);
    }

  // weight row of the 4 consecutive rows that this lane finishes of a tile, and their output column n
  auto first_row = [&](int tile, int& n) {
    const int i0 = 4 * lg;
    if (gated) { n = tile * 8 + (i0 & 7); return n + (i0 < 8 ? 0 : N); }
    return n = ROPE ? w_row(tile, i0) : tile * TR + i0;
  };
  // their scales and biases: those of the first tile that this wave finishes are fetched here, long
  // before they are needed
  floatx4 sc = {1.f, 1.f, 1.f, 1.f}, bi = {0.f, 0.f, 0.f, 0.f};
  const bool vec4 = (N & 3) == 0;
  auto fetch_affine = [&](int wr0, int n) {
    if (n >= N) return;
    if (vec4) {                                           // 4 columns are all in, and aligned (pointers: 16 bytes)
      if (W8) sc = *reinterpret_cast<const floatx4*>(p.wscale + wr0);
      if (p.bias != nullptr) {
        const u32x2 b = *reinterpret_cast<const u32x2*>(p.bias + wr0);
        bi = floatx4{bf_lo(b[0]), bf_hi(b[0]), bf_lo(b[1]), bf_hi(b[1])};
      }
    } else {
      for (int e = 0; e < 4 && n + e < N; ++e) {
        if (W8) sc[e] = p.wscale[wr0 + e];
        if (p.bias != nullptr) bi[e] = (float)p.bias[wr0 + e];
      }
    }
  };
  if constexpr (!RAW) {
    int n;
    const int wr0 = first_row(blockIdx.x + wave / MT * gridDim.x, n);
    fetch_affine(wr0, n);
  }

  // angles of the block's tiles (at most SLOTS: launch_fin), spread over its lanes while x is on its way; q and k
  // heads rotate, v heads do not.  Here and once, because the fp64 arithmetic wants a hundred registers:
  // beside x's operands and the weights in flight it spilled up to 36 (a layer of 32 + 2 x 8 heads of 128,
  // d_model 4096, MLP 128, at 24 rows: bf16 61.7 -> 53.6 us, int8 53.5 -> 46.3; behind the last product
  // instead 59.5 and 48.0)
  if constexpr (ROPE) {
    const int n = ceil_div(r.tiles - (int)blockIdx.x, (int)gridDim.x) * MT * 128;
#pragma unroll 1
    for (int at = tid; at < n; at += NW * 64) {
      const int t = blockIdx.x + at / (MT * 128) * gridDim.x, m = (at / 8) % (MT * 16);
      const int pos = __shfl(my_pos, min(m, M - 1), 64);
      if (t / octs >= p.sp.q_heads + p.sp.kv_heads) continue;
      const double theta = exp2(-2.0 * (double)((t % octs) * 8 + at % 8) / (double)p.sp.head_dim * r.l2_base);
      cs[at] = cos_sin((double)pos * theta);
    }
  }

  int tile = blockIdx.x, slot = 0;
  const char* src = src_of(tile);
  u32x4 wr[C::WIN];
#pragma unroll
  for (int s = 0; s < C::WIN; ++s) wr[s] = load(src, s);
  __builtin_amdgcn_sched_barrier(0);

  // B operand of step s = row lr of a group, the k that the weight's lanes hold
  bf16x8 xf[STEPS][C::XF][MT];
  {
    char* const patch = smem + wave * C::PATCH;           // [16 rows] of XCH chunks + 16 bytes: no bank conflicts either way
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
      for (int i = 0; i < XL; ++i)
        *reinterpret_cast<u32x4*>(patch + (i * 64 + lane) / XCH * C::XROW + (i * 64 + lane) % XCH * 16) = xt[mt][i];
      wave_lds_sync();
#pragma unroll
      for (int s = 0; s < STEPS; ++s)
#pragma unroll
        for (int f = 0; f < C::XF; ++f)
          xf[s][f][mt] = *reinterpret_cast<const bf16x8*>(patch + lr * C::XROW + ((s * 4 + lg) * C::XF + f) * 16);
      wave_lds_sync();
    }
  }
  lds_barrier();                                          // the sums below are collected where the patches lie

  auto one_tile = [&](auto more_c) {
    constexpr bool MORE = decltype(more_c)::value;
    const char* next = MORE ? src_of(tile + gridDim.x) : nullptr;
    floatx4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      if (s >= skip && s < skip + ns) {                   // wave-uniform
#pragma unroll
        for (int f = 0; f < C::XF; ++f) {
          bf16x8 a;
          if constexpr (W8) a = cvt_i8x8_bf16(u32x2{wr[s % C::WIN][2 * f], wr[s % C::WIN][2 * f + 1]});
          else a = __builtin_bit_cast(bf16x8, wr[s % C::WIN]);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, xf[s][f][mt], acc[mt], 0, 0, 0);
        }
      }
      if (s + C::WIN < STEPS) wr[s % C::WIN] = load(src, s + C::WIN);
      else if (MORE) wr[s % C::WIN] = load(next, s + C::WIN - STEPS);
      __builtin_amdgcn_sched_barrier(0);                  // (hoisted past the products, loads would want second registers)
    }
    // accumulator: lane = column lr of x's rows (group mt), weight rows 4 lg .. 4 lg + 3 of the tile
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) red[((slot * NW + wave) * MT + mt) * 64 + lane] = acc[mt];
    src = next;
  };
  // the collected tiles `first`, `first` + gridDim.x, ... (n of them): one wave finishes one group of
  // rows of one tile
  auto finish = [&](int first, int n_tiles) {
#pragma unroll 1
    for (int item = wave; item < n_tiles * MT; item += NW) {
      const int at = item / MT, mt = item % MT, tile = first + at * (int)gridDim.x;
      floatx4 v = red[((at * NW) * MT + mt) * 64 + lane];
#pragma unroll C::READS
      for (int w = 1; w < NW; ++w) v += red[((at * NW + w) * MT + mt) * 64 + lane];
      const int m = mt * 16 + lr;
      const int seq_pos = split ? __shfl(my_seq_pos, min(m, M - 1), 64) : 0;
      if constexpr (RAW) {
        const int n = tile * TR + 4 * lg;
        if (m >= M || n >= r.rows) continue;
        float* dst = p.part + ((int64_t)blockIdx.y * p.M + mz + m) * r.rows + n;
        if ((r.rows & 3) == 0) *reinterpret_cast<floatx4*>(dst) = v;
        else
          for (int e = 0; e < 4 && n + e < r.rows; ++e) dst[e] = v[e];
        continue;
      }
      int n;
      const int wr0 = first_row(tile, n);
      if (item != wave || first != (int)blockIdx.x) fetch_affine(wr0, n);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (W8) v[e] *= sc[e];
        v[e] += bi[e];
      }
      if (gated || ROPE) {
        floatx4 o;                                        // the partner rows: lane l ^ 32
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = __shfl_xor(v[e], 32, 64);
        if constexpr (ROPE) {
          if (tile / octs < p.sp.q_heads + p.sp.kv_heads) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const floatx2 t = cs[(at * MT * 16 + m) * 8 + 4 * (lg & 1) + e];
              v[e] = lg < 2 ? v[e] * t[0] - o[e] * t[1] : v[e] * t[0] + o[e] * t[1];
            }
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = silu_f(v[e]) * o[e];
          if (lg >= 2) continue;                          // (the up rows' lanes have handed theirs over)
        }
      } else if (r.act != FORGE_ACT_NONE) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          switch (r.act) {
            case FORGE_ACT_GELU_TANH: v[e] = gelu_tanh_f(v[e]); break;
            case FORGE_ACT_RELU: v[e] = fmaxf(v[e], 0.0f); break;
            case FORGE_ACT_SILU: v[e] = silu_f(v[e]); break;
            default: v[e] = gelu_erf_f(v[e]); break;
          }
        }
      }
      if (m >= M || n >= N) continue;
      if (ROPE || r.qkv) {
        // 4 columns stay inside a head (head_dim % 8 == 0, n % 4 == 0; N is whole heads)
        u32x2 pk;
        pk[0] = pack_bf2(v[0], v[1]);
        pk[1] = pack_bf2(v[2], v[3]);
        *reinterpret_cast<u32x2*>(split_dst_bf16(p.sp, p.row0 + mz + m, n, seq_pos)) = pk;
        continue;
      }
      const int64_t out = (int64_t)(mz + m) * p.ldy + n;
      if (n + 4 <= N && (p.ldy & 3) == 0) {
        if (p.residual != nullptr) {
          const u32x2 rr = *reinterpret_cast<const u32x2*>(p.residual + out);
          v[0] += bf_lo(rr[0]); v[1] += bf_hi(rr[0]); v[2] += bf_lo(rr[1]); v[3] += bf_hi(rr[1]);
        }
        u32x2 pk;
        pk[0] = pack_bf2(v[0], v[1]);
        pk[1] = pack_bf2(v[2], v[3]);
        *reinterpret_cast<u32x2*>(p.y + out) = pk;
      } else {
        for (int e = 0; e < 4 && n + e < N; ++e)
          p.y[out + e] = (bf16)(v[e] + (p.residual != nullptr ? (float)p.residual[out + e] : 0.f));
      }
    }
  };
  int first = tile;
  for (;;) {
    const bool more = tile + (int)gridDim.x < r.tiles;
    if (more) one_tile(std::true_type{});
    else one_tile(std::false_type{});
    ++slot;
    if (!more || slot == C::SLOTS) {
      lds_barrier();                                      // every wave's sums of these tiles are there
      finish(first, slot);
      if (!more) return;
      lds_barrier();                                      // ... and have been read
      slot = 0;
      first = tile + gridDim.x;
    }
    tile += gridDim.x;
  }
}

template <int MT, int STEPS, bool W8, int FIN>
forge_status launch_fin(const RowsParams& r, int ranges, hipStream_t s) {
  // one block per CU, also where the registers would hold two: two blocks read x twice (6144 x 2048 at
  // 8 rows 10.7 us, at 9 rows and one block 9.5 us)
  const int chunks = ceil_div(r.g.M, 16 * MT);
  int per = ceil_div(r.tiles, max(1, compute_units() / (ranges * chunks)));      // tiles per block
  if (FIN == FIN_ROPE) per = min(per, Rows<MT, STEPS, W8, FIN>::SLOTS);                // (their angles are computed once)
  auto kern = gemm_bf16_rows_kernel<MT, STEPS, W8, FIN>;
  // (more than half the LDS of a CU, whatever is needed: with two blocks resident some CUs get two and
  // others none, 2048 x 2048 at 16 rows 7.8 instead of 5.6 us)
  constexpr int smem = Rows<MT, STEPS, W8, FIN>::SMEM > 82 * 1024 ? Rows<MT, STEPS, W8, FIN>::SMEM : 82 * 1024;
  static std::atomic<uint64_t> lds_raised{0};   // per kernel instantiation
  if (raise_lds_limit(reinterpret_cast<const void*>(kern), smem, lds_raised) != FORGE_OK) return FORGE_ERR_HIP;
  kern<<<dim3(ceil_div(r.tiles, per), ranges, chunks), NW * 64, smem, s>>>(r);
  return launch_status();
}

template <int MT, int STEPS, bool W8>
forge_status launch_steps(const RowsParams& r, int fin, int ranges, hipStream_t s) {
  if (fin == FIN_RAW) return launch_fin<MT, STEPS, W8, FIN_RAW>(r, ranges, s);
  if (fin == FIN_ROPE) return launch_fin<MT, STEPS, W8, FIN_ROPE>(r, ranges, s);
  return launch_fin<MT, STEPS, W8, FIN_OUT>(r, ranges, s);
}

template <int MT, bool W8>
forge_status launch_mt(const RowsParams& r, int fin, const RowsPlan& pl, hipStream_t s) {
  switch (pl.steps) {
#define FORGE_ROWS_CASE(STEPS)                                                     \
    case STEPS:                                                                    \
      if constexpr (STEPS * (W8 ? 2 : 1) <= (MT > 2 ? 8 : 16)) return launch_steps<MT, STEPS, W8>(r, fin, pl.ranges, s); \
      else break
    FORGE_ROWS_CASE(1);
    FORGE_ROWS_CASE(2);
    FORGE_ROWS_CASE(3);
    FORGE_ROWS_CASE(4);
    FORGE_ROWS_CASE(5);
    FORGE_ROWS_CASE(6);
    FORGE_ROWS_CASE(7);
    FORGE_ROWS_CASE(8);
    FORGE_ROWS_CASE(9);
    FORGE_ROWS_CASE(10);
    FORGE_ROWS_CASE(12);
    FORGE_ROWS_CASE(14);
    FORGE_ROWS_CASE(16);
#undef FORGE_ROWS_CASE
    default: break;
  }
  return FORGE_ERR_UNSUPPORTED;
}

}  // namespace

namespace {
RowsPlan with_steps(int total, int ranges) {
  const int spw = ceil_div(total, ranges * NW);
  static constexpr int kSteps[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 14, 16};
  for (int s : kSteps)
    if (s >= spw) return RowsPlan{ceil_div(total, spw * NW), s, spw};     // total > 8 (spw - 1), so a row has at least s steps
  return RowsPlan{0, 0, 0};
}

// Where this kernel is the faster one, against the slab-wise streaming kernel (microseconds of one
// launch list, cold weights, that one | this kernel, a following reduce launch included).  Both read x
// once per block; here a block reads all of its k range of x (M * K * 2 bytes) however few weight
// rows it has, there 64 rows of it per 128 or 256 weight rows.

// bf16, at most 4096 elements of K.  While every CU has one tile, this kernel; beyond that its 64-byte pieces of
// 16 rows stream at 4.3 to 5.0 TB/s and the slabs at 4.5 to 5.4, unless rows are a multiple of 4 KB apart, which
// puts the slabs of all blocks on the same HBM channels (3.3 to 3.8, the pieces 5.2 to 5.6: 16384 x 4096 at 4 rows
// 41.2 | 26.0, x 3840 27.2 | 29.7).
bool streams_faster(int M, int rows, int K, bool qkv) {
  const int tiles = ceil_div(rows, TR), cus = compute_units();
  if (tiles <= cus) return true;
  const bool aligned = K % 2048 == 0;
  // enough weight rows for the slab-wise kernel to finish its outputs itself: with a short K and few rows the
  // per-block start still counts (50264 x 768 at 8 rows 21.5 | 20.1, 24576 x 1536 at 4 19.2 | 16.5), otherwise only where its
  // streams collide (32768 x 4096 at 17 rows 70.6 | 50.9; x 3840 46.8 | 58.5; x 1920 at 4 25.6 | 27.9; 50304 x 832 19.8 | 22.2)
  if (ceil_div(rows, 128) * 4 >= cus * 3)
    return M <= 32 && K % (32 * NW) == 0 && (aligned || (M <= 16 && K <= 2048));
  // many tiles per CU with more rows than pay for the time between two windows of a tile
  if (tiles >= 4 * cus && M > (K < 1024 ? 16 : 32)) return false;
  // between one and two tiles per CU the last round is half empty (5120 x 3840 at 17 rows 13.7 | 17.5, 6144 x 4096
  // 15.5 | 16.1, 8192 x 4096 18.8 | 16.9); a head split saves its reduce launch there (a layer of
  // 32 + 2 x 8 heads of 128 with a small MLP: 58 | 52)
  if (qkv && tiles < 2 * cus) return true;
  if (aligned) return K <= 2048 || M <= 16 || tiles * 4 >= 7 * cus;
  return K <= (M > 16 ? 2304 : 2560);   // (10240 x 2304 at 4 rows 15.0 | 13.2, x 2560 16.0 | 15.5, at 17 rows 16.4 | 17.1, x 2816 at 4 16.1 | 16.9)
}
}  // namespace

RowsPlan plan_rows(int M, int rows, int K, bool w8, int max_ranges, bool qkv) {
  const RowsPlan none = {0, 0, 0};
  if (M > MAX_ROWS || K % (w8 ? 2 * BK : BK) != 0) return none;
  const int total = K / (w8 ? 64 : 32);                        // steps of a row
  const int cap = NW * (w8 ? 8 : 16) / (M > 32 ? 2 : 1);       // ... that one range holds: x stays in registers
  const int least = ceil_div(total, cap);
  const int tiles = ceil_div(rows, TR), cus = compute_units();
  int ranges = 1;
  if (max_ranges == 0) {
    // One range, outputs finished here.  int8: wherever one range holds K (6144 x 4096 at 32 rows
    // 17.2 | 11.8, 6144 x 2048 at 64 rows 16.1 | 9.9).
    if (least > 1 || (!w8 && !streams_faster(M, rows, K, qkv))) return none;
  } else {
    // fp32 planes for a reduce kernel: enough ranges for a block per CU and for x to stay below half the
    // weight bytes of a block (2048 x 8192 at 21 rows: 2 ranges 15.0, 8 ranges 13.4 against 15.3).
    if (w8) {
      // not past 32 rows with a long K (4096 x 14336 at 64 rows 26.5 | 29.9), nor with so many tiles that the planes
      // weigh against the weight (32768 x 2560 at 33 rows 30.6 | 36.9, 16384 x 2560 20.4 | 21.8, x 3072 22.2 | 21.8)
      if (M > 32 && (K > 8192 || 640 * (int64_t)tiles >= (int64_t)K * cus)) return none;
    } else if (K <= 4096) {
      // (4096 x 4096 at 48 rows 14.8 | 15.7)
      if (tiles >= cus && (M > 32 || !streams_faster(M, rows, K, false))) return none;
    } else {
      // not for long reductions (4096 x 14336 at 5 rows 25.8 | 28.0), nor past 32 rows or one tile per CU (15360 x 5120 at
      // 4 rows 33.4 | 45.3, 5120 x 5120 16.2 | 18.0), except few rows where the slabs collide (8192 x 8192 at 4 rows
      // 38.9 | 33.4, 16384 x 8192 73.7 | 61.9)
      const bool collide = K % 4096 == 0 && M <= 16 && tiles * 4 >= 7 * cus && ceil_div(rows, 128) * 4 < cus * 3;
      if (K > 8192 || M > 32 || (tiles >= cus && !collide)) return none;
    }
    ranges = max(ceil_div(cus, tiles), ceil_div(M * cus, 8 * tiles));
    const int most = min(max_ranges, total / (2 * NW));
    ranges = max(least, min(ranges, most));
    if (ranges > max_ranges) return none;
    // (the next count that puts a block on nearly every CU: 6 ranges of 128 tiles are 192 blocks, 8 are 256)
    for (int r = ranges; r <= most; ++r)
      if (cus / r > 0 && ceil_div(tiles, ceil_div(tiles, cus / r)) * r * 10 >= cus * 9) { ranges = r; break; }
  }
  return with_steps(total, ranges);
}

// The rows of x, then the tiles that a block walks, then the weight from HBM; fitted to 630 drawn problems of up to 8192
// weight rows (within 3 % for half of them, 7 % for nine of ten).
double rows_us(int M, int rows, int K) {
  static constexpr double kX[] = {0.68, 1.22, 1.33}, kTile[] = {0.89, 0.84, 1.54};     // per 1024 elements of K: up to 16, 32, 64 rows
  const int m = M > 32 ? 2 : M > 16 ? 1 : 0, per = ceil_div(ceil_div(rows, TR), compute_units());
  const double k = K / 1024.0;
  return 2.7 + kX[m] * k + per * (0.58 + kTile[m] * k) + (double)rows * K * 2 * 0.24 / 6e6;
}

// Prompts of 65 to 128 rows in two chunks, K of 768 to 2048: the weight is read once per chunk (the second time from cache),
// as long as a block has few tiles to walk.  us: fitted to 420 drawn problems (within 4 % for half of them, 10 % for
// nine of ten); plan_route takes them where the waves that share the k slabs are estimated slower (this | that: 100 rows
// against 12288 x 1024 15.2 | 19.2, 105 against 10240 x 2048 22.3 | 27.1).  Three chunks and more gain as often as they lose
// (553 rows against 2304 x 1536 19.2 | 22.4, 173 against 6144 x 1920 26.4 | 21.7) and stay there.
RowsPlan plan_rows_prompt(int M, int rows, int K, double* us) {
  const RowsPlan none = {0, 0, 0};
  const int steps = ceil_div(K / 32, NW), per = ceil_div(ceil_div(rows, TR), compute_units() / 2);
  if (M <= 64 || M > 128 || K % BK != 0 || steps < 4 || steps > 8 || per > 6) return none;
  const double k = steps / 4.0;
  *us = 2.6 + 1.68 * k + per * (0.76 + 1.22 * k) + (double)rows * K * 2 * 0.285 / 6e6;
  return with_steps(K / 32, 1);
}

forge_status launch_rows(const GemmParams& p, const RowsPlan& pl, int act, bool qkv, bool raw, hipStream_t s) {
  RowsParams r;
  r.g = p;
  r.rows = act == FORGE_ACT_SWIGLU ? 2 * p.N : p.N;
  r.act = act;
  r.qkv = qkv ? 1 : 0;
  const int fin = raw ? FIN_RAW : (qkv && p.sp.rope ? FIN_ROPE : FIN_OUT);
  r.l2_base = fin == FIN_ROPE ? log2((double)p.sp.rope_base) : 0.0;
  r.tiles = act == FORGE_ACT_SWIGLU && !raw ? ceil_div(p.N, 8) : ceil_div(r.rows, TR);
  r.spw = pl.spw;
  if (p.w8 != nullptr)
    return p.M > 32 ? launch_mt<4, true>(r, fin, pl, s) : p.M > 16 ? launch_mt<2, true>(r, fin, pl, s) : launch_mt<1, true>(r, fin, pl, s);
  return p.M > 32 ? launch_mt<4, false>(r, fin, pl, s) : p.M > 16 ? launch_mt<2, false>(r, fin, pl, s) : launch_mt<1, false>(r, fin, pl, s);
}

}  // namespace forge
