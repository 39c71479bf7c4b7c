// fp32 fused linear:  y = act(x . w^T + bias) (+ residual), true fp32 operands on the fp32
// matrix cores (v_mfma_f32_32x32x2_f32), so the result stays within fp32 rounding of the
// definition (no reduced-precision operand shortcut).
//
// Tiling: a 256-thread block (4 waves as 2 x 2) owns a 64 x 64 tile of y; each wave owns a
// 32 x 32 accumulator.  K is walked in slabs of 32: the x slab [64,32] and the w slab [64,32]
// (both K-contiguous in memory) are copied to LDS with 128-bit accesses, rows padded to 36
// floats so that eight lanes reading the same column chunk of eight consecutive rows hit
// disjoint banks.  The MFMA contracts two k per issue (lanes 0-31 supply one, lanes 32-63 the
// other); lanes 0-31 walk k = 0..15 of the slab and lanes 32-63 walk k = 16..31, so every
// lane reads four consecutive floats per 128-bit LDS read.  The slabs are prefetched three
// ahead in registers.
//
// Most problems of up to some thousand tiles take gemm_f32_waves_kernel below instead (plan_waves says which).
// Long reductions with few tiles are split along K over grid.z: raw fp32 partial sums go to the workspace
// and a second kernel adds them in split order (fixed order, no atomics: bitwise reproducible) and
// carries the epilogue.
#include <stdint.h>
#include "common.hpp"

namespace forge {
namespace {

constexpr int BM = 64, BN = 64, BK = 32, LDK = BK + 4;

// (head_dim is 64 or 128: shifts instead of divisions)
__device__ inline void* split_dst(const QkvSplit& sp, int m, int n, size_t esz) {
  const int dh = sp.head_dim, shift = __builtin_ctz(dh), c = n & (dh - 1);
  const int b = sp.q_len == 1 ? m : m / sp.q_len, s = sp.q_len == 1 ? 0 : m - b * sp.q_len;
  int h = n >> shift;
  if (h < sp.q_heads) return (char*)sp.q + (((((int64_t)b * sp.q_heads + h) * sp.q_len + s) << shift) + c) * esz;
  h -= sp.q_heads;
  const bool is_k = h < sp.kv_heads;
  h -= is_k ? 0 : sp.kv_heads;
  char* const base = (char*)(is_k ? sp.k_cache : sp.v_cache);
  return base + (((((int64_t)b * sp.kv_heads + h) * sp.kv_cap + seq_position(sp.pos, b, sp.pos0) + s) << shift) + c) * esz;
}

template <int ACT, bool SPLIT>
__global__ __launch_bounds__(256) void gemm_f32_kernel(
    const float* __restrict__ x, const float* __restrict__ w, const float* __restrict__ bias,
    const float* residual, float* y, int M, int N, int K, int ldy, QkvSplit sp,
    int k_per_split, float* part) {
  constexpr bool SWIGLU = ACT == FORGE_ACT_SWIGLU;
  constexpr int NB = SWIGLU ? 2 : 1;
  __shared__ __attribute__((aligned(16))) float As[BM][LDK];
  __shared__ __attribute__((aligned(16))) float Bs[NB][BN][LDK];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;

  floatx16 acc[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;

  const int lrow = tid >> 3;        // 0..31
  const int lcol = (tid & 7) * 4;   // 0,4,..,28

  const int k_begin = blockIdx.z * k_per_split;           // multiple of BK
  const int k_end = min(K, k_begin + k_per_split);

  // Register prefetch, PF slabs ahead: a block of a small problem walks only a few slabs, and
  // with load -> LDS -> barrier -> multiply in sequence every slab would pay the full memory
  // latency.  Loads are unconditional from clamped (valid) addresses so that they stay
  // asynchronous; what lies outside the matrix is zeroed when the slab is written to LDS.
  constexpr int PF = 3;
  floatx4 va[PF][2], vb[PF][NB][2];
  const float* xrow[2];
  const float* wrow[NB][2];
  bool rowa_ok[2], rowb_ok[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int row = lrow + 32 * r;
    rowa_ok[r] = m0 + row < M;
    rowb_ok[r] = n0 + row < N;
    xrow[r] = x + (int64_t)min(m0 + row, M - 1) * K;
#pragma unroll
    for (int t = 0; t < NB; ++t) wrow[t][r] = w + (int64_t)(min(n0 + row, N - 1) + t * N) * K;
  }
  auto gload = [&](int k0, int slot) {
    const int kk = min(k0 + lcol, K - 4);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      va[slot][r] = *reinterpret_cast<const floatx4*>(xrow[r] + kk);
#pragma unroll
      for (int t = 0; t < NB; ++t) vb[slot][t][r] = *reinterpret_cast<const floatx4*>(wrow[t][r] + kk);
    }
  };
  auto lstore = [&](int k0, int slot) {
    const bool k_ok = k0 + lcol < K;
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int row = lrow + 32 * r;
      *reinterpret_cast<floatx4*>(&As[row][lcol]) = rowa_ok[r] && k_ok ? va[slot][r] : zero;
#pragma unroll
      for (int t = 0; t < NB; ++t)
        *reinterpret_cast<floatx4*>(&Bs[t][row][lcol]) = rowb_ok[r] && k_ok ? vb[slot][t][r] : zero;
    }
  };
#pragma unroll
  for (int d = 0; d < PF; ++d) gload(k_begin + d * BK, d);
  for (int kb = k_begin; kb < k_end; kb += PF * BK) {
#pragma unroll
    for (int d = 0; d < PF; ++d) {
      const int k0 = kb + d * BK;
      if (k0 < k_end) {                       // block-uniform
        lstore(k0, d);
        __syncthreads();
        const int r = lane & 31, hk = (lane >> 5) * 16;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const floatx4 a = *reinterpret_cast<const floatx4*>(&As[wm * 32 + r][hk + 4 * j]);
          floatx4 b[NB];
#pragma unroll
          for (int t = 0; t < NB; ++t) b[t] = *reinterpret_cast<const floatx4*>(&Bs[t][wn * 32 + r][hk + 4 * j]);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int t = 0; t < NB; ++t)
              acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[t][e], acc[t], 0, 0, 0);
        }
        __syncthreads();
      }
      gload(k0 + PF * BK, d);                 // slab k0 + PF slabs into the registers just consumed
    }
  }

  const int n = n0 + wn * 32 + (lane & 31);
  if (n >= N) return;
  if (part != nullptr) {       // split-K: raw partial sums [split, M, NB * N]; the reduce kernel does the rest
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int m = m0 + wm * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
      if (m >= M) continue;
      float* dst = part + ((int64_t)blockIdx.z * M + m) * (NB * N) + n;
      dst[0] = acc[0][v];
      if (SWIGLU) dst[N] = acc[NB - 1][v];
    }
    return;
  }
  // epilogue on the accumulator: + bias, activation, + residual, store
  float bv = 0.f, bv2 = 0.f;
  if (bias != nullptr) {
    bv = bias[n];
    if (SWIGLU) bv2 = bias[n + N];
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int m = m0 + wm * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
    if (m >= M) continue;
    float val = acc[0][v] + bv;
    if (SWIGLU) val = silu_f(val) * (acc[NB - 1][v] + bv2);
    else val = apply_act<ACT>(val);
    if (SPLIT) {
      *reinterpret_cast<float*>(split_dst(sp, m, n, sizeof(float))) = val;
    } else {
      if (residual != nullptr) val += residual[(int64_t)m * ldy + n];
      y[(int64_t)m * ldy + n] = val;
    }
  }
}

// Second stage of the split: one thread per output element.
template <int ACT, bool SPLIT>
__global__ __launch_bounds__(256) void gemm_f32_reduce_kernel(
    const float* __restrict__ part, const float* __restrict__ bias, const float* residual, float* y,
    int M, int N, int ldy, int splits, QkvSplit sp) {
  constexpr bool SWIGLU = ACT == FORGE_ACT_SWIGLU;
  const int ncols = SWIGLU ? 2 * N : N;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (int64_t)M * N) return;
  const int m = (int)(gid / N), n = (int)(gid % N);
  const int64_t plane = (int64_t)M * ncols;
  const float* src = part + (int64_t)m * ncols + n;
  float a = 0.f, u = 0.f;
  for (int z = 0; z < splits; ++z) {
    a += src[z * plane];
    if (SWIGLU) u += src[z * plane + N];
  }
  if (bias != nullptr) {
    a += bias[n];
    if (SWIGLU) u += bias[n + N];
  }
  float val = SWIGLU ? silu_f(a) * u : apply_act<ACT>(a);
  if (SPLIT) {
    *reinterpret_cast<float*>(split_dst(sp, m, n, sizeof(float))) = val;
  } else {
    if (residual != nullptr) val += residual[(int64_t)m * ldy + n];
    y[(int64_t)m * ldy + n] = val;
  }
}

// ---- k slabs shared by the waves of a block ---------------------------------------------------------
// A layer of a few hundred fp32 rows has fewer 64 x 64 tiles than the chip has CUs, and each of them is a
// serial chain of slabs with two block barriers per slab, a partial plane and a second launch.  Here a
// block of 8 waves owns 32 rows x 16 CB weight rows and the waves take the 32-element k slabs in turn (wave w:
// slabs w, w + 8, ...): every wave loads, stages (in an LDS patch of its own) and multiplies its slabs
// without a block barrier, DEPTH slabs in flight in registers, and the 8 partial tiles are added through LDS in
// wave order at the end, where the outputs are finished.  v_mfma_f32_16x16x4_f32: lane l supplies row
// l%16 and the k of its quarter, 8 (l/16) ... + 7 of the slab.  The gated activation takes 16 gate rows and
// their 16 up rows as the two column blocks.
// Bound by latency: the start of a block (5 us for 768 k, 1.3 of them matrix work) and the chain load, patch, product of
// each slab.  Counted at 128 rows against 2304 x 768 and 3072 x 768: matrix units 14 and 18 % busy, LDS 2.5 and 3.4 us of
// the 14.3 and 13.9 us under a profiler (a quarter of that bank conflicts).  Tiles of 64 x 32 and 64 x 64 halve the LDS
// traffic and are slower (2304 x 768 at 128 rows 11.9 and 22 us against 10.6); two blocks per CU need the 128 registers.
// The four products of a 128-row layer of 768 (MLP 3072): 60.4 us with their reduce launches before, 39.6 on tiles of one
// and two column blocks with requests past the end, 37 now; the layer 76.8 -> 57.6 and 55.3 -> 51.9 by these.
constexpr int FW = 8;                                // waves per block
constexpr int FM = 32, RB = FM / 16;                 // rows of x per block

constexpr int slabs_in_flight(int cb) { return cb == 1 ? 3 : 2; }   // per wave (up to CB 2 in 128 registers: two blocks per CU)

// SHORT: no wave has more than DEPTH slabs; otherwise every wave has DEPTH at least (CB 2: any number)
template <int CB, int ACT, bool SPLIT, bool SHORT>
__global__ __launch_bounds__(FW * 64, CB > 2 ? 2 : 4) void gemm_f32_waves_kernel(
    const float* __restrict__ x, const float* __restrict__ w, const float* __restrict__ bias,
    const float* residual, float* y, int M, int N, int K, int ldy, QkvSplit sp) {
  constexpr bool SWIGLU = ACT == FORGE_ACT_SWIGLU;
  static_assert(!SWIGLU || CB == 2, "gate and up rows are the two column blocks");
  constexpr int WR = 16 * CB;                        // weight rows per block
  constexpr int OUT = SWIGLU ? 16 : WR;              // output columns per block
  constexpr int DEPTH = slabs_in_flight(CB);
  // the 32 x 32 tiles run two to a CU in several rounds: left to the scheduler, in a loop that always refills (us, 255 rows against
  // 2304 x 768 18.2 as the others | 16.3, 742 against 3072 x 768 46.7 | 40.7; short rows too: 190 against 4096 x 512 16.7 | 15.1,
  // 73 against 2048 gated pairs x 512 9.7 | 8.9, 300 against 768 x 256 4.6 | 4.4)
  constexpr bool REFILL = CB == 2;
  constexpr int CHAINS = CB == 2 ? 2 : 4;            // sums per output of a wave: shorter chains, smaller rounding error
  constexpr int PATCH = (FM + WR) * LDK;             // floats of one wave's patch; rows padded as above
  constexpr int LDR = WR + 4;                        // row of a partial tile
  static_assert(FM * LDR <= PATCH, "the partial tiles fit where the patches lie");
  extern __shared__ __attribute__((aligned(16))) float lds[];   // [FW * PATCH]

  const int tid = threadIdx.x, lane = tid & 63, wave = REFILL ? tid >> 6 : __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = blockIdx.y * FM, n0 = blockIdx.x * OUT;
  float* const ax = lds + wave * PATCH;
  float* const bx = ax + FM * LDK;

  // loads: 8 lanes per row piece of 32 floats, unconditional from clamped addresses (rows past the end
  // re-read the last one and are dropped at the store; k past the end is zeroed on the way into LDS)
  const int lrow = lane >> 3, lcol = (lane & 7) * 4;
  uint32_t xsrc[FM / 8], wsrc[WR / 8];               // byte offsets of the rows (below 4 GB: the host has checked)
#pragma unroll
  for (int i = 0; i < FM / 8; ++i) xsrc[i] = (uint32_t)min(m0 + lrow + 8 * i, M - 1) * (uint32_t)K * 4;
#pragma unroll
  for (int i = 0; i < WR / 8; ++i) {
    const int r = lrow + 8 * i;
    const int row = SWIGLU ? min(n0 + (r & 15), N - 1) + (r >= 16 ? N : 0) : min(n0 + r, N - 1);
    wsrc[i] = (uint32_t)row * (uint32_t)K * 4;
  }
  floatx4 va[DEPTH][FM / 8], vb[DEPTH][WR / 8];
  auto gload = [&](int k0, int slot) {
    const uint32_t kk = 4 * min(k0 + lcol, K - 4);
#pragma unroll
    for (int i = 0; i < FM / 8; ++i) va[slot][i] = *reinterpret_cast<const floatx4*>((const char*)x + (xsrc[i] + kk));
#pragma unroll
    for (int i = 0; i < WR / 8; ++i) vb[slot][i] = *reinterpret_cast<const floatx4*>((const char*)w + (wsrc[i] + kk));
  };
  floatx4 acc[CHAINS][RB][CB];
#pragma unroll
  for (int h = 0; h < CHAINS; ++h)
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < CB; ++j) acc[h][i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  auto multiply = [&](int i, int d) {                // slab i of this wave, from slot d
    if constexpr (!REFILL) __builtin_amdgcn_sched_barrier(0);               // (mixed with its neighbours' loads and stores a slab wants more registers)
    const bool k_ok = (wave + i * FW) * BK + lcol < K;
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
    wave_lds_sync();                                 // the previous slab has been read
#pragma unroll
    for (int i = 0; i < FM / 8; ++i) *reinterpret_cast<floatx4*>(ax + (lrow + 8 * i) * LDK + lcol) = k_ok ? va[d][i] : zero;
#pragma unroll
    for (int i = 0; i < WR / 8; ++i) *reinterpret_cast<floatx4*>(bx + (lrow + 8 * i) * LDK + lcol) = k_ok ? vb[d][i] : zero;
    wave_lds_sync();
    const int r = lane & 15, kq = (lane >> 4) * 8;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      floatx4 a[RB], b[CB];
#pragma unroll
      for (int i = 0; i < RB; ++i) a[i] = *reinterpret_cast<const floatx4*>(ax + (16 * i + r) * LDK + kq + 4 * j);
#pragma unroll
      for (int c = 0; c < CB; ++c) b[c] = *reinterpret_cast<const floatx4*>(bx + (16 * c + r) * LDK + kq + 4 * j);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
          for (int c = 0; c < CB; ++c)
            acc[(j + 2 * e) % CHAINS][i][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], b[c][e], acc[(j + 2 * e) % CHAINS][i][c], 0, 0, 0);
    }
    if constexpr (!REFILL) __builtin_amdgcn_sched_barrier(0);
  };
  // bias and residual of the outputs that this thread finishes, behind the first slabs: unconditional (a load under a branch would
  // make every wait behind it a full one), what is not there is read from the weight and dropped
  constexpr int ITEMS = FM * OUT / (FW * 64);
  const int has_bias = bias != nullptr ? -1 : 0, has_res = residual != nullptr ? -1 : 0;      // masks of the offsets
  float bi[ITEMS], ub[ITEMS], rv[ITEMS];
  auto fetch_ends = [&] {
    const float* const bsrc = has_bias ? bias : w;
    const float* const rsrc = has_res ? residual : w;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const int at = tid + it * FW * 64, m = min(m0 + at / OUT, M - 1), n = min(n0 + at % OUT, N - 1);
      bi[it] = bsrc[n & has_bias];
      if (SWIGLU) ub[it] = bsrc[(N + n) & has_bias];
      rv[it] = rsrc[(int64_t)(m & has_res) * ldy + (n & has_res)];
    }
  };
  // Past the end of K a wave of short rows loads what DEPTH exceeds its slabs by, one of long rows at most DEPTH - 1, or DEPTH where
  // it has just DEPTH (one loop that always refills made 768 of K 48 slabs of requests instead of 24; one that may be skipped
  // makes the compiler copy the slabs in flight, a wait for each: 128 rows against 3072 x 768 14.6 -> 12.4 us, 2304 x 768
  // 12.4 -> 11.8, 768 x 3072 13.2 -> 12.9).
  const int n_slabs = (K + BK - 1) / BK > wave ? ((K + BK - 1) / BK - wave - 1) / FW + 1 : 0;
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) gload((wave + d * FW) * BK, d);
  fetch_ends();
  if constexpr (SHORT) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
      if (d < n_slabs) multiply(d, d);               // (wave-uniform)
  } else if constexpr (REFILL) {
    for (int i = 0; i < n_slabs; i += DEPTH)
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        if (i + d < n_slabs) multiply(i + d, d);
        gload((wave + (i + d + DEPTH) * FW) * BK, d);
      }
  } else {                                           // (n_slabs >= DEPTH)
    int i = DEPTH;
#pragma unroll 1
    do {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        multiply(i - DEPTH + d, d);
        gload((wave + (i + d) * FW) * BK, d);        // into the registers just consumed
      }
      i += DEPTH;
    } while (i < n_slabs);
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
      if (i - DEPTH + d < n_slabs) multiply(i - DEPTH + d, d);
  }

  // ---- the 8 partial tiles, added in wave order; accumulator: column lane%16, rows 4 (lane/16) ... + 3 --------
  wave_lds_sync();
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int c = 0; c < CB; ++c) {
#pragma unroll
      for (int h = 1; h < CHAINS; ++h) acc[0][i][c] += acc[h][i][c];
#pragma unroll
      for (int v = 0; v < 4; ++v) ax[(16 * i + 4 * (lane >> 4) + v) * LDR + 16 * c + (lane & 15)] = acc[0][i][c][v];
    }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const int at = tid + it * FW * 64;
    const int mr = at / OUT, nc = at % OUT, m = m0 + mr, n = n0 + nc;
    float v = 0.f, u = 0.f;
#pragma unroll
    for (int z = 0; z < FW; ++z) {
      v += lds[z * PATCH + mr * LDR + nc];
      if (SWIGLU) u += lds[z * PATCH + mr * LDR + 16 + nc];
    }
    if (m >= M || n >= N) continue;
    if (has_bias) {
      v += bi[it];
      if (SWIGLU) u += ub[it];
    }
    v = SWIGLU ? silu_f(v) * u : apply_act<ACT>(v);
    if (SPLIT) {
      *reinterpret_cast<float*>(split_dst(sp, m, n, sizeof(float))) = v;
    } else {
      if (has_res) v += rv[it];
      y[(int64_t)m * ldy + n] = v;
    }
  }
}

// k ranges for a problem: none while the tiles fill the chip; otherwise towards two blocks per
// CU, each with at least four slabs.
struct SplitPlan { int splits, k_per_split; };
SplitPlan plan_split(int M, int N, int K) {
  const int tiles = ceil_div(M, BM) * ceil_div(N, BN);
  const int slabs = ceil_div(K, BK);
  int want = tiles >= 256 ? 1 : min(ceil_div(256, tiles), slabs / 4);
  want = max(1, want);
  const int per = ceil_div(slabs, want);
  return SplitPlan{ceil_div(slabs, per), per * BK};
}

}  // namespace

namespace {
template <int CB, int ACT, bool SPLIT, bool SHORT>
forge_status launch_slabs(const float* x, const float* w, const float* bias, const float* res, float* y, int M, int N,
                         int K, int ldy, const QkvSplit& sp, hipStream_t s) {
  constexpr int smem = FW * (FM + 16 * CB) * LDK * (int)sizeof(float);
  auto kern = gemm_f32_waves_kernel<CB, ACT, SPLIT, SHORT>;
  static std::atomic<uint64_t> lds_raised{0};   // per kernel instantiation
  if (raise_lds_limit(reinterpret_cast<const void*>(kern), smem, lds_raised) != FORGE_OK) return FORGE_ERR_HIP;
  const int cols = ACT == FORGE_ACT_SWIGLU ? 8 * CB : 16 * CB;
  kern<<<dim3(ceil_div(N, cols), ceil_div(M, FM)), FW * 64, smem, s>>>(x, w, bias, res, y, M, N, K, ldy, sp);
  return launch_status();
}
template <int CB, int ACT, bool SPLIT>
forge_status launch_tile(const float* x, const float* w, const float* bias, const float* res, float* y, int M, int N,
                         int K, int ldy, const QkvSplit& sp, hipStream_t s) {
  if constexpr (CB != 2) {
    if (ceil_div(K, BK) <= slabs_in_flight(CB) * FW) return launch_slabs<CB, ACT, SPLIT, true>(x, w, bias, res, y, M, N, K, ldy, sp, s);
  }
  return launch_slabs<CB, ACT, SPLIT, false>(x, w, bias, res, y, M, N, K, ldy, sp, s);
}
template <int ACT, bool SPLIT>
forge_status launch_waves(int cb, const float* x, const float* w, const float* bias, const float* res, float* y, int M, int N,
                          int K, int ldy, const QkvSplit& sp, hipStream_t s) {
  if constexpr (ACT != FORGE_ACT_SWIGLU) {
    if (cb == 3) return launch_tile<3, ACT, SPLIT>(x, w, bias, res, y, M, N, K, ldy, sp, s);
    if (cb == 1) return launch_tile<1, ACT, SPLIT>(x, w, bias, res, y, M, N, K, ldy, sp, s);
  }
  return launch_tile<2, ACT, SPLIT>(x, w, bias, res, y, M, N, K, ldy, sp, s);
}
// Column blocks (1, 2 or 3) of the wave-shared tiles, or 0 for the 64 x 64 tiles.  Times are rounds of tiles over the
// CUs times slabs plus a start, in units of 0.1 us as measured (7 per round of 64 x 64 tiles and slab, 1.9 and 1.2 per round
// of 32 x 32 and 32 x 16; us, 64 x 64 with its reduce | wave-shared: 128 rows against 2304 x 768 15.1 | 10.6, 768 x 768 9.8 | 5.2,
// 3072 x 768 18.1 | 10.9, 768 x 3072 17.4 | 12.9; 512 rows against 3072 x 768 34.3 | 29.4, 2048 rows 99 | 108, 256 rows
// against 6144 x 72 9.2 | 10.1).  A long reduction with few tiles stays cut over the grid (64 rows against 768 x 8192
// 21.9 | 28.7, 256 x 4096 at one row 13.8 | 15.0; from 24 tiles on 32.7 | 30.5), a gated one sooner (24 rows against 256 pairs x
// 2560 15.7 | 19.3).  Past four rounds the last one no longer counts as whole: blocks of 64 x 64 share CUs (1063 rows
// against 6144 x 512 70 | 82).
inline int few_tiles(int K, bool gated) { return K > 3072 ? 16 : gated && K > 2304 ? 8 : 0; }
int plan_waves(int M, int N, int K, bool gated) {
  const int64_t rows = gated ? 2 * (int64_t)N : N;
  if ((int64_t)M * K >= (1ll << 30) || rows * K >= (1ll << 30)) return 0;       // 32-bit byte offsets
  const int64_t cus = compute_units(), slabs = ceil_div(K, BK), slabs8 = (slabs + 7) / 8 * 8;
  const int64_t t64 = (int64_t)ceil_div(M, BM) * ceil_div(N, BN), mt = ceil_div(M, FM);
  if (t64 <= few_tiles(K, gated) || mt > 65535) return 0;
  const int64_t slab64 = slabs * (gated ? 14 : 7), c64 = (t64 > 4 * cus ? t64 * slab64 / cus : ceil_div64(t64, cus) * slab64) + 45;
  const int64_t c2 = ceil_div64(mt * ceil_div64(rows, 32), cus) * slabs8 * 19 / 10 + 22;
  const int64_t c1 = gated ? c2 : ceil_div64(mt * ceil_div64(N, 16), cus) * slabs8 * 12 / 10 + 21;
  // 32 x 48 where these are one round: 128 rows against 2304 x 768 32 x 16 11.9 | 11.0, 3072 x 768 12.3 | 11.1, 512 against
  // 768 x 3072 30.6 | 28.2; not in several rounds (512 against 2304 x 768 32 x 32 26.5 | 27.0)
  const int64_t c3 = !gated && mt * ceil_div64(N, 48) <= cus ? slabs8 * 2 + 44 : INT64_MAX;
  if (c64 < c2 && c64 < c1 && c64 < c3) return 0;
  if (c3 < c1 && c3 < c2) return 3;
  return c1 < c2 ? 1 : 2;
}
}  // namespace

// fp32 planes of this very problem, 0 where it runs whole
static size_t planes_bytes(int M, int N, int K, forge_act act) {
  if (plan_waves(M, N, K, act == FORGE_ACT_SWIGLU) > 0) return 0;
  const SplitPlan sp = plan_split(M, N, K);
  if (sp.splits == 1) return 0;
  return (size_t)sp.splits * M * (act == FORGE_ACT_SWIGLU ? 2 * N : N) * sizeof(float);
}

// The size to ask for: a long reduction that this many rows run whole is cut at fewer rows, and a buffer for the larger
// problem serves the smaller ones.
size_t gemm_f32_workspace_bytes(int M, int N, int K, forge_act act) {
  const size_t own = planes_bytes(M, N, K, act);
  const int cut_rows = few_tiles(K, act == FORGE_ACT_SWIGLU) / ceil_div(N, BN) * BM;      // the most rows that are cut
  return M > cut_rows && cut_rows > 0 ? max(own, planes_bytes(cut_rows, N, K, act)) : own;
}

const char* gemm_f32_variant(int M, int N, int K, forge_act act) {
  const int cb = plan_waves(M, N, K, act == FORGE_ACT_SWIGLU);
  if (cb > 0) return cb == 1 ? "gemm_f32_waves<1>" : cb == 2 ? "gemm_f32_waves<2>" : "gemm_f32_waves<3>";
  return plan_split(M, N, K).splits > 1 ? "gemm_f32<64,64,2,2>+splitk" : "gemm_f32<64,64,2,2>";
}

forge_status launch_gemm_f32(const GemmArgs& a, hipStream_t s) {
  SplitPlan pl = plan_split(a.M, a.N, a.K);
  const size_t need = planes_bytes(a.M, a.N, a.K, a.act);
  if (need > a.workspace_bytes || (need > 0 && a.workspace == nullptr)) pl = SplitPlan{1, a.K};   // unsplit
  float* part = pl.splits > 1 ? (float*)a.workspace : nullptr;
  dim3 grid(ceil_div(a.N, BN), ceil_div(a.M, BM), pl.splits), block(256);
  const unsigned rblocks = (unsigned)ceil_div64((int64_t)a.M * a.N, 256);
  const float* x = (const float*)a.x;
  const float* w = (const float*)a.w;
  const float* bias = (const float*)a.bias;
  const float* res = (const float*)a.residual;
  float* y = (float*)a.y;
  QkvSplit sp = {};
  const int ldy = a.ldy > 0 ? a.ldy : a.N;
  const int cb = plan_waves(a.M, a.N, a.K, a.act == FORGE_ACT_SWIGLU);
  if (a.split != nullptr) {
    if (a.act != FORGE_ACT_NONE || a.residual != nullptr) return FORGE_ERR_UNSUPPORTED;
    sp = *a.split;
    if (cb > 0) return launch_waves<FORGE_ACT_NONE, true>(cb, x, w, bias, res, y, a.M, a.N, a.K, ldy, sp, s);
    gemm_f32_kernel<FORGE_ACT_NONE, true><<<grid, block, 0, s>>>(x, w, bias, res, y, a.M, a.N, a.K, ldy, sp,
                                                                 pl.k_per_split, part);
    if (part != nullptr)
      gemm_f32_reduce_kernel<FORGE_ACT_NONE, true><<<rblocks, 256, 0, s>>>(part, bias, res, y, a.M, a.N, ldy, pl.splits, sp);
    return launch_status();
  }
  switch (a.act) {
#define FORGE_CASE(ACT)                                                                                        \
  case ACT:                                                                                                    \
    if (cb > 0) return launch_waves<ACT, false>(cb, x, w, bias, res, y, a.M, a.N, a.K, ldy, sp, s);             \
    gemm_f32_kernel<ACT, false><<<grid, block, 0, s>>>(x, w, bias, res, y, a.M, a.N, a.K, ldy, sp,             \
                                                       pl.k_per_split, part);                                  \
    if (part != nullptr)                                                                                       \
      gemm_f32_reduce_kernel<ACT, false><<<rblocks, 256, 0, s>>>(part, bias, res, y, a.M, a.N, ldy, pl.splits, sp); \
    break
    FORGE_CASE(FORGE_ACT_NONE);
    FORGE_CASE(FORGE_ACT_GELU_TANH);
    FORGE_CASE(FORGE_ACT_RELU);
    FORGE_CASE(FORGE_ACT_SILU);
    FORGE_CASE(FORGE_ACT_SWIGLU);
    FORGE_CASE(FORGE_ACT_GELU_ERF);
#undef FORGE_CASE
    default: return FORGE_ERR_INVALID_ARG;
  }
  return launch_status();
}

}  // namespace forge
