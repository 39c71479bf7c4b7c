// bf16 linear for prompts of some tens to some hundred rows, and for decode steps against small weights: the
// waves of a block share the k slabs.
//
// Such a problem is all latency: launch, first loads, a few products, the store.  A block of 8 waves owns
// 16 RB rows of x and 16 CB weight rows, small enough that the tiles cover the chip; the waves take the 64-element
// k slabs in turn (wave w: slabs w, w + 8, ...), each loads its slabs in whole 128-byte row pieces, DEPTH of
// them in flight in registers, turns them into the operand layout through an LDS patch of its own and
// multiplies with v_mfma_f32_16x16x32_bf16, without a block barrier; the 8 partial tiles are added
// through LDS in wave order and finished (bias, activation, residual, head split) in the one launch.
// The weight is the A operand, so that a lane holds 4 consecutive output columns of one row.
//
// us, cold weights, the kernel that took the problem before (x in registers, 128 x 128 tiles, slab-wise, with a reduce launch
// where it needed one) | this one: 128 rows against 768 x 768 7.0 | 3.8, 2304 x 768 7.4 | 5.4, 3072 x 768 8.0 | 6.0, 768 x 3072
// 10.3 | 7.8, 256 x 2048 x 2048 11.6 | 9.9, 128 x 2048 x 8192 23.1 | 19.7, 24 x 2048 x 2048 6.6 | 4.9, 64 x 4096 x 4096
// 17.4 | 13.6.  What is left at 128 rows: a start of 2.5 us, the block's operands at about 50 KB per us and CU, the exchange
// of the partial tiles.  plan_waves says where.
#include <math.h>
#include "gemm_bf16.hpp"

namespace forge {
namespace {

constexpr int NW = 8;                                // waves per block
constexpr int DEPTH = 2;                             // slabs in flight per wave
constexpr int LDB = BK * 2 + 16;                     // bytes of a patch row: 64 bf16 and padding (conflict-free 128-bit accesses)

struct WavesParams {
  GemmParams g;                                      // g.N: output columns
  int act;
  int qkv;                                           // head split
};

// SLABS: no wave has more than 1, 2 or 3; 0: every wave has 3 at least
template <int RB, int CB, bool GATED, int SLABS>
__global__ __launch_bounds__(NW * 64, RB * CB <= 4 ? 4 : 2) void gemm_bf16_waves_kernel(WavesParams r) {
  const GemmParams& p = r.g;
  constexpr int FM = 16 * RB, WR = 16 * CB;          // rows of x, weight rows
  constexpr int OUT = GATED ? WR / 2 : WR;           // output columns
  constexpr int PATCH = (FM + WR) * LDB;             // bytes
  constexpr int LDR = WR + 4;                        // floats of a row of a partial tile
  static_assert(FM * LDR * 4 <= PATCH, "the partial tiles fit where the patches lie");
  constexpr bool BIG = RB * CB >= 16;                // its slabs take long to multiply: left to the scheduler
  extern __shared__ __attribute__((aligned(16))) char smem[];   // [NW * PATCH]

  const int tid = threadIdx.x, lane = tid & 63, wave = BIG ? tid >> 6 : __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = p.M, N = p.N, K = p.K;
  const int m0 = blockIdx.y * FM, n0 = blockIdx.x * OUT;
  char* const ax = smem + wave * PATCH;
  char* const bx = ax + FM * LDB;

  // loads: 8 lanes per row piece, from clamped addresses (rows past the end re-read the last one, their outputs are dropped)
  const int lrow = lane >> 3, lcol = (lane & 7) * 16;
  uint32_t xsrc[FM / 8], wsrc[WR / 8];               // byte offsets (operands below 4 GB: choose_variant)
#pragma unroll
  for (int i = 0; i < FM / 8; ++i) xsrc[i] = (uint32_t)min(m0 + lrow + 8 * i, M - 1) * (uint32_t)K * 2 + lcol;
#pragma unroll
  for (int i = 0; i < WR / 8; ++i) {
    const int rr = lrow + 8 * i;
    const int row = GATED ? min(n0 + rr % OUT, N - 1) + (rr >= OUT ? N : 0) : min(n0 + rr, N - 1);
    wsrc[i] = (uint32_t)row * (uint32_t)K * 2 + lcol;
  }
  const int slabs = K / BK, n_slabs = slabs > wave ? (slabs - wave - 1) / NW + 1 : 0;   // of them this wave's
  u32x4 va[DEPTH][FM / 8], vb[DEPTH][WR / 8];
  auto load = [&](int i, int slot) {                 // this wave's slab i
    const uint32_t at = (uint32_t)min(wave + i * NW, slabs - 1) * (BK * 2);
#pragma unroll
    for (int i = 0; i < WR / 8; ++i) vb[slot][i] = *reinterpret_cast<const u32x4*>((const char*)p.w + (wsrc[i] + at));
#pragma unroll
    for (int i = 0; i < FM / 8; ++i) va[slot][i] = *reinterpret_cast<const u32x4*>((const char*)p.x + (xsrc[i] + at));
  };

  floatx4 acc[RB][CB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int c = 0; c < CB; ++c) acc[i][c] = floatx4{0.f, 0.f, 0.f, 0.f};

  const int fr = lane & 15, fg = lane >> 4;
  auto multiply = [&](int d) {
    if constexpr (!BIG) __builtin_amdgcn_sched_barrier(0);      // (mixed with its neighbours' loads and stores a slab wants twice the registers)
    wave_lds_sync();                                 // the previous slab has been read
#pragma unroll
    for (int i = 0; i < FM / 8; ++i) *reinterpret_cast<u32x4*>(ax + (lrow + 8 * i) * LDB + lcol) = va[d][i];
#pragma unroll
    for (int i = 0; i < WR / 8; ++i) *reinterpret_cast<u32x4*>(bx + (lrow + 8 * i) * LDB + lcol) = vb[d][i];
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      bf16x8 xf[RB], wf[CB];
#pragma unroll
      for (int i = 0; i < RB; ++i) xf[i] = *reinterpret_cast<const bf16x8*>(ax + (16 * i + fr) * LDB + (4 * k + fg) * 16);
#pragma unroll
      for (int c = 0; c < CB; ++c) wf[c] = *reinterpret_cast<const bf16x8*>(bx + (16 * c + fr) * LDB + (4 * k + fg) * 16);
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int c = 0; c < CB; ++c) acc[i][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[c], xf[i], acc[i][c], 0, 0, 0);
    }
    if constexpr (!BIG) __builtin_amdgcn_sched_barrier(0);
  };
  // bias and residual of the outputs that this thread finishes: requested behind the first slabs, long before they are
  // needed.  Unconditional (a load under a branch would make every wait behind it a full one): what is not there is read
  // from the weight and dropped.
  constexpr int ITEMS = (FM * OUT / 4 + NW * 64 - 1) / (NW * 64);
  const bool vec = (N & 3) == 0 && (p.ldy & 3) == 0;
  const bool has_bias = vec && p.bias != nullptr, has_res = vec && p.residual != nullptr;
  u32x2 bi[ITEMS], ub[ITEMS], rv[ITEMS];
  auto fetch_ends = [&] {
    const bf16* const bsrc = has_bias ? p.bias : p.w;
    const bf16* const rsrc = has_res ? p.residual : p.w;
    const int ldb = has_bias ? -1 : 0, ldr = has_res ? -1 : 0;     // masks of the offsets
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const int at = min(tid + it * NW * 64, FM * OUT / 4 - 1);
      const int m = min(m0 + at / (OUT / 4), M - 1), n = min(n0 + at % (OUT / 4) * 4, N - 4);
      bi[it] = *reinterpret_cast<const u32x2*>(bsrc + (n & ldb));
      if (GATED) ub[it] = *reinterpret_cast<const u32x2*>(bsrc + ((N + n) & ldb));
      rv[it] = *reinterpret_cast<const u32x2*>(rsrc + (int64_t)(m & ldr) * p.ldy + (n & ldr));
    }
  };
  // Past the end of K a wave loads one slab at most (in the loop of the 64 x 64 tiles three): up to three slabs per wave are straight
  // code, and the loop runs at least once and is followed by the last slabs.  (As one loop that always refills, 768 of K were 32 slabs of requests instead of 16, and a loop
  // that may be skipped makes the compiler copy the slabs in flight, a wait for each: 128 rows against 2304 x 768 6.8 -> 5.95 us,
  // 3072 x 768 7.1 -> 6.4, 768 x 3072 8.0 -> 7.8, 256 x 2048 x 2048 10.6 -> 9.9.  Three slabs in the loop load a fourth and lose to
  // refilling: 400 rows against 2560 x 1280 14.8 refilling, 15.6 in the loop, 14.0 straight, 150 against 3072 x 1088 8.2, 8.8, 8.0.)
  load(0, 0);
  if constexpr (SLABS != 1) load(1, 1);
  if constexpr (!BIG) __builtin_amdgcn_sched_barrier(0);       // (among the slabs' requests: 128 rows against 768 x 768 4.0 instead of 3.8 us)
  fetch_ends();
  if constexpr (SLABS > 0) {
    if (0 < n_slabs) multiply(0);                    // (wave-uniform)
    if (SLABS > 2) load(2, 0);
    if (SLABS > 1 && 1 < n_slabs) multiply(1);
    if (SLABS > 2 && 2 < n_slabs) multiply(0);
  } else if constexpr (BIG) {                        // (always refilling: 109 rows against 5968 x 1088 10.5 us, 12.0 as below)
    for (int i = 0; i < n_slabs; i += DEPTH) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        if (i + d < n_slabs) multiply(d);
        load(i + d + DEPTH, d);
      }
    }
  } else {                                           // (n_slabs > DEPTH)
    int i = DEPTH;
#pragma unroll 1
    do {
      multiply(0);
      load(i, 0);
      multiply(1);
      load(i + 1, 1);
      i += DEPTH;
    } while (i < n_slabs);
    if (i - 2 < n_slabs) multiply(0);
    if (i - 1 < n_slabs) multiply(1);
  }

  // ---- the 8 partial tiles, added in wave order; accumulator: row lane % 16, columns 4 (lane / 16) ... + 3 ------
  wave_lds_sync();
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int c = 0; c < CB; ++c) *reinterpret_cast<floatx4*>(ax + ((16 * i + fr) * LDR + 16 * c + 4 * fg) * 4) = acc[i][c];
  __syncthreads();
  auto unpack = [](u32x2 t) { return floatx4{bf_lo(t[0]), bf_hi(t[0]), bf_lo(t[1]), bf_hi(t[1])}; };
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const int at = tid + it * NW * 64;
    const int mr = at / (OUT / 4), nc = at % (OUT / 4) * 4, m = m0 + mr, n = n0 + nc;
    if (at >= FM * OUT / 4 || m >= M || n >= N) continue;
    floatx4 v = {0.f, 0.f, 0.f, 0.f}, u = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int z = 0; z < NW; ++z) {
      const char* src = smem + z * PATCH + (mr * LDR + nc) * 4;
      v += *reinterpret_cast<const floatx4*>(src);
      if (GATED) u += *reinterpret_cast<const floatx4*>(src + OUT * 4);
    }
    if (has_bias) {
      v += unpack(bi[it]);
      if (GATED) u += unpack(ub[it]);
    } else if (p.bias != nullptr) {
      for (int e = 0; e < 4 && n + e < N; ++e) {
        v[e] += (float)p.bias[n + e];
        if (GATED) u[e] += (float)p.bias[N + n + e];
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (GATED) { v[e] = silu_f(v[e]) * u[e]; continue; }
      switch (r.act) {
        case FORGE_ACT_GELU_TANH: v[e] = gelu_tanh_f(v[e]); break;
        case FORGE_ACT_RELU: v[e] = fmaxf(v[e], 0.0f); break;
        case FORGE_ACT_SILU: v[e] = silu_f(v[e]); break;
        case FORGE_ACT_GELU_ERF: v[e] = gelu_erf_f(v[e]); break;
        default: break;
      }
    }
    bf16* dst = r.qkv ? split_dst_bf16(p.sp, p.row0 + m, n) : p.y + (int64_t)m * p.ldy + n;   // 4 columns stay inside a head
    if (vec) {
      if (has_res) v += unpack(rv[it]);
      *reinterpret_cast<u32x2*>(dst) = u32x2{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
    } else {
      const bf16* res = p.residual != nullptr ? p.residual + (int64_t)m * p.ldy + n : nullptr;
      for (int e = 0; e < 4 && n + e < N; ++e) dst[e] = (bf16)(v[e] + (res != nullptr ? (float)res[e] : 0.f));
    }
  }
}

template <int RB, int CB, bool GATED, int SLABS>
forge_status launch_slabs(const WavesParams& r, hipStream_t s) {
  constexpr int smem = NW * 16 * (RB + CB) * LDB;
  auto kern = gemm_bf16_waves_kernel<RB, CB, GATED, SLABS>;
  static std::atomic<uint64_t> lds_raised{0};        // per kernel instantiation
  if (raise_lds_limit(reinterpret_cast<const void*>(kern), smem, lds_raised) != FORGE_OK) return FORGE_ERR_HIP;
  kern<<<dim3(ceil_div(r.g.N, GATED ? 8 * CB : 16 * CB), ceil_div(r.g.M, 16 * RB)), NW * 64, smem, s>>>(r);
  return launch_status();
}

template <int RB, int CB, bool GATED>
forge_status launch_tile(const WavesParams& r, hipStream_t s) {
  const int slabs = r.g.K / BK;
  if (slabs <= NW) return launch_slabs<RB, CB, GATED, 1>(r, s);
  if (slabs <= DEPTH * NW) return launch_slabs<RB, CB, GATED, 2>(r, s);
  if (slabs <= 3 * NW) return launch_slabs<RB, CB, GATED, 3>(r, s);
  return launch_slabs<RB, CB, GATED, 0>(r, s);
}

}  // namespace

// Tiles (row blocks, column blocks) and their times in us: a start, a round of tiles over the CUs, what 1024 elements of K add
// to a round, and what they add per tile and CU (blocks that run into each other's loads); fitted to 1100 drawn problems
// with the weight in HBM (within 5 to 8 % for half of them, 11 to 20 % for nine of ten; the tile picked is 0.6 % off the
// fastest of them in the geometric mean, K below 512 3 %).  48 rows or columns come to one round where 32 and 64 do not (us,
// 128 rows against 2304 x 768 64 x 32 5.7 | 48 x 32 5.0, 3072 x 768 5.6 | 32 x 48 5.3, 68 rows against 6144 x 2048 14.0 | 48 x 48
// 12.0); where they do not, and with very short rows, the others.
// At most 64 rows are weighed against x in registers (rows_us), whose estimate is of the same age as those of the tiles of 16, 32 and
// 64 here; both kernels are about 5 % faster now, so these keep their own constants: 28 rows against 3000 x 1024 5.1 | 4.6 there, 21
// against 8192 x 2048 10.1 | 10.5.  Those of 48 only order the tiles: 50 drawn problems of 33 to 64 rows that take one are 2 to 14 %
// faster on it than without them, 6.3 % in the geometric mean (50 x 6144 x 2048 11.4 | 10.0, 47 x 8192 x 4096 20.4 | 20.0).
namespace {
struct WavesTile { int rb, cb; double start, round, per_k, full; };
constexpr WavesTile kTiles[] = {{1, 1, 2.5, 0.36, 0.51, 0.14}, {1, 2, 2.5, 0.65, 0.81, 0.22}, {2, 2, 2.97, 0.4, 1.19, 0.34}, {4, 2, 1.35, 2.34, 2.05, 0.33},
                                {4, 4, 1.3, 3.1, 3.05, 0.73}, {2, 3, 1.4, 1.99, 1.68, 0.73}, {3, 2, 1.43, 2.09, 1.57, 0.38}, {3, 3, 1.7, 2.3, 2.12, 0.77}};
constexpr WavesTile kFewRows[] = {{1, 1, 3.5, 0.23, 0.8, 0}, {1, 2, 3.6, 0.36, 1.3, 0}, {2, 2, 3.5, 0.62, 1.64, 0}, {4, 2, 2.2, 2.46, 2.4, 0},
                                  {4, 4, 2.1, 3.8, 3.56, 0}, {2, 3, 2.3, 2.1, 2.2, 0}, {3, 2, 2.2, 2.3, 1.95, 0}, {3, 3, 2.9, 2.1, 2.7, 0}};
constexpr int kTileCount = sizeof(kTiles) / sizeof(kTiles[0]);
static_assert(sizeof(kFewRows) == sizeof(kTiles), "the same tiles in the same order");
}  // namespace

WavesPlan plan_waves(int M, int N, int K, bool gated) {
  const int rows = gated ? 2 * N : N;
  WavesPlan best = {-1, 0.0};
  double empty = 0.0;                                // share of the last of several rounds
  for (int i = gated ? 1 : 0; i < kTileCount; ++i) {
    const WavesTile& t = M > 64 ? kTiles[i] : kFewRows[i];
    const int64_t tiles = (int64_t)ceil_div(M, 16 * t.rb) * ceil_div(rows, 16 * t.cb), rounds = ceil_div64(tiles, compute_units());
    if ((t.rb == 3 || t.cb == 3) && (K < 256 || rounds > 1)) continue;
    const double k = K / 1024.0, fit = t.start + rounds * (t.round + t.per_k * k) + t.full * k * tiles / compute_units();
    // (the fit is a little hard on 48 x 48 where K is long or the output gated: us, 32 x 32 | 48 x 48 where it has them equal, 73 rows
    // against 2304 gated pairs x 768 6.4 | 6.05, 84 against 2304 x 512 5.2 | 5.0, 150 rows against 2880 x 1984 12.0 | 10.8; plain and
    // short, 214 against 2304 x 512, 4.4 | 4.85)
    const double us = fit * (t.rb * t.cb == 9 && t.full > 0 && (gated || K > 1024) ? 0.98 : 1.0);
    if (best.tile >= 0 && us >= best.us) continue;
    best = WavesPlan{i, us};
    empty = t.full > 0 && rounds > 1 ? 1.0 - (double)tiles / (rounds * compute_units()) : 0.0;
  }
  // Against other kernels: too good where the last of several rounds is mostly empty, 330 and 368 tiles over 256 CUs (690 rows against
  // 1920 x 2560 29.0 us, fitted 26.6, 1433 against 1024 x 2560 27.7, 26.0), not where it is full (294 against 6144 x 2048 24.1, 25.5).
  best.us *= 1.0 + 0.3 * empty;
  best.us += (double)rows * K * 2 * (M > 64 ? 0.73 : 0.62) / 6e6;      // the weight from HBM
  return best;
}

forge_status launch_waves(const GemmParams& p, int tile, int act, bool qkv, hipStream_t s) {
  const WavesParams r = {p, act, qkv ? 1 : 0};
  const bool gated = act == FORGE_ACT_SWIGLU;
  switch (tile) {
    case 0: return gated ? FORGE_ERR_UNSUPPORTED : launch_tile<1, 1, false>(r, s);
    case 1: return gated ? launch_tile<1, 2, true>(r, s) : launch_tile<1, 2, false>(r, s);
    case 2: return gated ? launch_tile<2, 2, true>(r, s) : launch_tile<2, 2, false>(r, s);
    case 3: return gated ? launch_tile<4, 2, true>(r, s) : launch_tile<4, 2, false>(r, s);
    case 4: return gated ? launch_tile<4, 4, true>(r, s) : launch_tile<4, 4, false>(r, s);
    case 5: return gated ? launch_tile<2, 3, true>(r, s) : launch_tile<2, 3, false>(r, s);
    case 6: return gated ? launch_tile<3, 2, true>(r, s) : launch_tile<3, 2, false>(r, s);
    case 7: return gated ? launch_tile<3, 3, true>(r, s) : launch_tile<3, 3, false>(r, s);
    default: return FORGE_ERR_UNSUPPORTED;
  }
}

const char* waves_variant(int tile) {
  constexpr const char* names[] = {"gemm_bf16_waves<1,1>", "gemm_bf16_waves<1,2>", "gemm_bf16_waves<2,2>", "gemm_bf16_waves<4,2>",
                                   "gemm_bf16_waves<4,4>", "gemm_bf16_waves<2,3>", "gemm_bf16_waves<3,2>", "gemm_bf16_waves<3,3>"};
  return names[tile];
}

}  // namespace forge
