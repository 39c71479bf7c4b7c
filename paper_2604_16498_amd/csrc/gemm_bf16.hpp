// What the bf16 linear kernels share: the launch parameters, the head split's addressing, the int8
// conversion and the LDS-only block barrier.  Internal to the library.
#pragma once
#include "common.hpp"

namespace forge {

constexpr int BK = 64;            // k per slab of the tile and streaming kernels

// Where column n of row m (position `pos` of its sequence: seq_position) of a head split goes.  head_dim is a power of two
// (64 or 128), and the rows of a decode step are sequences: no division then.
__device__ inline bf16* split_dst_bf16(const QkvSplit& sp, int m, int n, int pos) {
  const int dh = sp.head_dim, shift = __builtin_ctz(dh), c = n & (dh - 1);
  const int b = sp.q_len == 1 ? m : m / sp.q_len, s = sp.q_len == 1 ? 0 : m - b * sp.q_len;
  int h = n >> shift;
  if (h < sp.q_heads) return (bf16*)sp.q + (((((int64_t)b * sp.q_heads + h) * sp.q_len + s) << shift) + c);
  h -= sp.q_heads;
  const bool is_k = h < sp.kv_heads;
  h -= is_k ? 0 : sp.kv_heads;
  bf16* const base = (bf16*)(is_k ? sp.k_cache : sp.v_cache);
  return base + (((((int64_t)b * sp.kv_heads + h) * sp.kv_cap + pos + s) << shift) + c);
}
// ... the position read here
__device__ inline bf16* split_dst_bf16(const QkvSplit& sp, int m, int n) {
  return split_dst_bf16(sp, m, n, seq_position(sp.pos, sp.q_len == 1 ? m : m / sp.q_len, sp.pos0));
}

struct GemmParams {
  const bf16* x;
  const bf16* w;
  const bf16* bias;
  const bf16* residual;
  bf16* y;
  int M, N, K;        // N: output columns
  int ldy;            // row stride of y and residual (elements)
  int tiles_m, tiles_n;
  int k_per_split;    // split-K: k range of one block (multiple of 64); otherwise >= K
  int splits;         // split-K in the persistent kernel: number of k ranges
  float* part;        // split-K: fp32 partial sums [splits, M, N]
  size_t part_bytes;  // bytes behind part
  QkvSplit sp;
  NormTail nt;        // nt.y_norm == nullptr: none
  const int8_t* w8;     // weight-only int8 (M <= 64 streaming path): [N, K] bytes; w is NULL then
  const float* wscale;  // one scale per weight row, applied to the reduced sum before the bias
  int row0;             // row of the whole problem that row 0 of this launch is (head split only)
  int col0;             // column of the whole problem that column 0 of this launch is (head split only)
};

typedef __attribute__((address_space(3))) void lds_void;

// 8 signed bytes -> 8 bf16 (exact: |q| <= 127 has 7 significant bits)
__device__ inline bf16x8 cvt_i8x8_bf16(u32x2 v) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int b = (int)(int8_t)((v[e >> 2] >> (8 * (e & 3))) & 0xff);
    r[e] = (bf16)(float)b;
  }
  return r;
}

// ---- decode-sized problems with x in registers (gemm_bf16_rows.hip) ------------------------------
struct RowsPlan {
  int ranges;    // k ranges; 0: the problem does not take this path
  int steps;     // 64-byte steps of a weight row that a wave loads
  int spw;       // ... of which it multiplies at most this many
};
// rows: weight rows.  max_ranges 0: the plan of a launch that finishes its outputs itself (plain, head
// split, rotated head split), one range; otherwise of one that writes at most that many fp32 planes
// [ranges, M, rows] for the reduce kernels (raw).
RowsPlan plan_rows(int M, int rows, int K, bool w8, int max_ranges, bool qkv);
RowsPlan plan_rows_prompt(int M, int rows, int K, double* us);   // 65 to 128 rows, bf16 weights
double rows_us(int M, int rows, int K);                     // estimated time of one range, bf16, K >= 1024
forge_status launch_rows(const GemmParams& p, const RowsPlan& pl, int act, bool qkv, bool raw, hipStream_t s);

// ---- prompts of some hundred rows, small decode problems (gemm_bf16_waves.hip) ----------------------
struct WavesPlan {
  int tile;      // -1: the problem does not take this path
  double us;     // estimated time
};
WavesPlan plan_waves(int M, int N, int K, bool gated);      // K % 64 == 0, bf16 weights, operands below 4 GB
forge_status launch_waves(const GemmParams& p, int tile, int act, bool qkv, hipStream_t s);
const char* waves_variant(int tile);

}  // namespace forge
