// Fused residual add + LayerNorm / RMSNorm.
//
// HBM-bound: every element of x (and delta) is read once and h, y are written once.  A row is
// held in registers as fp32 between the read and the two writes, so the mean, the centred
// variance and the normalisation all run without a second pass over memory.
//
// Two launch shapes:
//   - one 64-lane wave per row (4 rows per 256-thread block, up to 4 chunks per lane), reductions
//     by cross-lane shuffles only: d <= 1024, and d <= 2048 when there are at least 1024 rows (no
//     block barrier and a whole row in flight per wave: 13.4 vs 14.6 us for 8192 x 2048 inside the
//     model; with few rows, or at d = 4096, the block per row is the faster one);
//   - one 256-thread block per row, wave shuffles then a 4-entry LDS exchange.
// Each lane owns CH chunks of 8 consecutive elements (one 128-bit access for bf16, two for
// fp32), chunk c of lane l covers elements 8*(l + c*G) .. +8 with G lanes per row, so that
// consecutive lanes touch consecutive 16 B.
#include "common.hpp"

namespace forge {
namespace {

// 8 elements as they lie in memory (one 128-bit access for bf16, two for fp32), unpacked after all loads are out
template <typename T> struct Raw8 {
  u32x4 r[sizeof(T) / 2];
  __device__ void load(const T* p) {
#pragma unroll
    for (int i = 0; i < (int)sizeof(T) / 2; ++i) r[i] = reinterpret_cast<const u32x4*>(p)[i];
  }
  __device__ float at(int i) const {
    if constexpr (sizeof(T) == 4) return __uint_as_float(r[i / 4][i % 4]);
    else return i % 2 == 0 ? bf_lo(r[0][i / 2]) : bf_hi(r[0][i / 2]);
  }
};

template <typename T, int CH, int G, bool RMS>
__global__ __launch_bounds__(256) void residual_norm_kernel(
    const T* __restrict__ x, const T* __restrict__ delta, const T* __restrict__ gamma,
    const T* __restrict__ beta, T* __restrict__ h_out, T* __restrict__ y, int rows, int d,
    float eps) {
  constexpr int ROWS_PER_BLOCK = 256 / G;
  const int tid = threadIdx.x;
  const int lane_in_row = tid % G;
  const int row = blockIdx.x * ROWS_PER_BLOCK + tid / G;
  const bool row_ok = row < rows;   // G == 256: uniform per block; G == 64: uniform per wave
  __shared__ float red[4];

  // Every load of the row goes out before the first is waited for, from clamped addresses: a branch per chunk made each
  // wait for its own (us in a replayed graph, reductions
  // included: 128 x 768 bf16 3.14 | 2.51, with delta 3.52 | 2.59, 8192 x 768 7.49 | 6.41, 4096 x 4096 fp32 26.9 | 25.2).  Gain and shift too where the registers are there.
  constexpr bool EARLY = CH <= 2;
  const int64_t base = (int64_t)min(row, rows - 1) * d;
  int at[CH];
  Raw8<T> xr[CH], dr[CH], gr[CH], br[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    at[c] = 8 * (lane_in_row + c * G);
    at[c] = at[c] < d ? at[c] : 0;
    xr[c].load(x + base + at[c]);
  }
  if (delta != nullptr) {
#pragma unroll
    for (int c = 0; c < CH; ++c) dr[c].load(delta + base + at[c]);
  }
  auto load_affine = [&]() {
#pragma unroll
    for (int c = 0; c < CH; ++c) gr[c].load(gamma + at[c]);
    if (!RMS && beta != nullptr) {
#pragma unroll
      for (int c = 0; c < CH; ++c) br[c].load(beta + at[c]);
    }
  };
  if (EARLY) load_affine();
  float v[CH][8];
  float sum = 0.f;
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const bool in = 8 * (lane_in_row + c * G) < d;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[c][i] = in ? xr[c].at(i) : 0.f;
    if (delta != nullptr && in) {
#pragma unroll
      for (int i = 0; i < 8; ++i) v[c][i] += dr[c].at(i);
    }
    if (h_out != nullptr && in && row_ok) Vec8<T>::store(h_out + base + at[c], v[c]);
#pragma unroll
    for (int i = 0; i < 8; ++i) sum += RMS ? v[c][i] * v[c][i] : v[c][i];
  }

  auto row_sum = [&](float s) -> float {
    s = wave_sum(s);
    if (G == 256) {
      __syncthreads();            // protects red[] between the two uses
      if ((tid & 63) == 0) red[tid >> 6] = s;
      __syncthreads();
      s = red[0] + red[1] + red[2] + red[3];
    }
    return s;
  };

  const float inv_d = 1.0f / (float)d;
  float mean = 0.f, rstd;
  if (RMS) {
    rstd = rsqrtf(row_sum(sum) * inv_d + eps);
  } else {
    mean = row_sum(sum) * inv_d;
    float sq = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int e = 8 * (lane_in_row + c * G);
      if (e < d) {
#pragma unroll
        for (int i = 0; i < 8; ++i) { float t = v[c][i] - mean; sq += t * t; }
      }
    }
    rstd = rsqrtf(row_sum(sq) * inv_d + eps);
  }

  if (!EARLY) load_affine();
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    if (!row_ok || 8 * (lane_in_row + c * G) >= d) continue;
    float o[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (v[c][i] - mean) * rstd * gr[c].at(i);
    if (!RMS && beta != nullptr) {
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] += br[c].at(i);
    }
    Vec8<T>::store(y + base + at[c], o);
  }
}

template <typename T, int CH, int G>
forge_status launch_g(const void* x, const void* delta, const void* gamma, const void* beta,
                      void* h_out, void* y, int rows, int d, float eps, forge_norm kind,
                      hipStream_t s) {
  const int rows_per_block = 256 / G;
  dim3 grid(ceil_div(rows, rows_per_block)), block(256);
  if (kind == FORGE_NORM_RMSNORM)
    residual_norm_kernel<T, CH, G, true><<<grid, block, 0, s>>>(
        (const T*)x, (const T*)delta, (const T*)gamma, (const T*)beta, (T*)h_out, (T*)y, rows, d, eps);
  else
    residual_norm_kernel<T, CH, G, false><<<grid, block, 0, s>>>(
        (const T*)x, (const T*)delta, (const T*)gamma, (const T*)beta, (T*)h_out, (T*)y, rows, d, eps);
  return launch_status();
}

template <typename T>
forge_status launch_t(const void* x, const void* delta, const void* gamma, const void* beta,
                      void* h_out, void* y, int rows, int d, float eps, forge_norm kind,
                      hipStream_t s) {
  const int chunks = d / 8;
#define FORGE_NORM_CASE(CH, G) \
  return launch_g<T, CH, G>(x, delta, gamma, beta, h_out, y, rows, d, eps, kind, s)
  if (chunks <= 64) FORGE_NORM_CASE(1, 64);
  if (chunks <= 128) FORGE_NORM_CASE(2, 64);
  if (chunks <= 256 && rows >= 1024) FORGE_NORM_CASE(4, 64);
  if (chunks <= 256) FORGE_NORM_CASE(1, 256);
  if (chunks <= 512) FORGE_NORM_CASE(2, 256);
  if (chunks <= 1024) FORGE_NORM_CASE(4, 256);
  if (chunks <= 2048) FORGE_NORM_CASE(8, 256);
#undef FORGE_NORM_CASE
  return FORGE_ERR_UNSUPPORTED;
}

}  // namespace

forge_status launch_residual_norm(const void* x, const void* delta, const void* gamma,
                                  const void* beta, void* h_out, void* y, int rows, int d,
                                  float eps, forge_norm kind, forge_dtype dt, hipStream_t s) {
  if (dt == FORGE_BF16) return launch_t<bf16>(x, delta, gamma, beta, h_out, y, rows, d, eps, kind, s);
  return launch_t<float>(x, delta, gamma, beta, h_out, y, rows, d, eps, kind, s);
}

}  // namespace forge
