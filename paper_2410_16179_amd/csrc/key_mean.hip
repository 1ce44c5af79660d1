// Key centering vector mu = (1/n) sum_i k_i per (batch, KV head) (Sec. 4.3 "Data
// pre-processing").  HBM-bound streaming read of the K cache: each thread sums up to
// kMeanChunkRows/16 rows of one 8-element column group in float32, the workgroup and the
// chunks are combined in float64 in a fixed order, so the result is reproducible.
#include "mp_common.h"
#include "device_utils.h"

namespace mp {

template <int ET, bool NT>
__global__ __launch_bounds__(256) void key_mean_partial_kernel(MeanArgs a) {
  __shared__ double red[16][kHeadDim];
  const int unit = blockIdx.y, chunk = blockIdx.x;
  const int cg = threadIdx.x & 15, rl = threadIdx.x >> 4;
  const int64_t base = (int64_t)(unit / a.n_kv_heads) * a.stride_b + (int64_t)(unit % a.n_kv_heads) * a.stride_h;
  const int64_t r0 = (int64_t)chunk * kMeanChunkRows;
  const int64_t r1 = r0 + kMeanChunkRows < a.n ? r0 + kMeanChunkRows : a.n;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (r1 - r0 == kMeanChunkRows) {
    // a whole chunk: unrolled, so that as many of a thread's rows as 64 registers hold are on their way at once
    Frag f[kMeanChunkRows / 16];
#pragma unroll
    for (int j = 0; j < kMeanChunkRows / 16; ++j) frag_load<ET, NT>(a.Kc, base + (r0 + rl + 16 * j) * a.stride_n + cg * 8, f[j]);
#pragma unroll
    for (int j = 0; j < kMeanChunkRows / 16; ++j) {
      float v[8];
      frag_to_float<ET>(f[j], v);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += v[e];
    }
  } else {
#pragma unroll 4
    for (int64_t i = r0 + rl; i < r1; i += 16) {
      float v[8];
      load8<ET>(a.Kc, base + i * a.stride_n + cg * 8, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += v[e];
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[rl][cg * 8 + e] = (double)acc[e];
  __syncthreads();
  if (threadIdx.x < kHeadDim) {
    double s = 0.0;
    for (int r = 0; r < 16; ++r) s += red[r][threadIdx.x];
    a.partial[((int64_t)unit * a.nchunk + chunk) * kHeadDim + threadIdx.x] = s;
  }
}

// Sums the chunk partials of COLS elements of one (batch, KV head) in a fixed order: 1024 / COLS groups of COLS
// lanes take every (1024 / COLS)-th chunk (independent loads), the groups of a wavefront are added by
// rotations, LDS joins the rest.  Many chunks need many groups (8 KV heads x 384 chunks, 48 one after the other
// per thread with COLS = 128: 7.5 us; 16: 4.6); with few, one workgroup per unit is enough and eight are launches
// of idle threads (the call, 512 units x 2 chunks: 16 19.4 us, 128 13.1).
template <int COLS>
__global__ __launch_bounds__(1024) void key_mean_final_kernel(MeanArgs a) {
  constexpr int kGroups = 1024 / COLS, kRows = COLS < 64 ? 16 : kGroups;
  __shared__ double red[kRows][COLS];
  const int unit = blockIdx.x;
  const int d = threadIdx.x & (COLS - 1), grp = threadIdx.x / COLS;
  const int col = blockIdx.y * COLS + d;
  double s = 0.0;
#pragma unroll 4
  for (int c = grp; c < a.nchunk; c += kGroups) s += a.partial[((int64_t)unit * a.nchunk + c) * kHeadDim + col];
  if constexpr (COLS < 64) {
#pragma unroll
    for (int o = COLS; o < 64; o <<= 1) s += __shfl_xor(s, o);
    if ((threadIdx.x & 63) < COLS) red[threadIdx.x >> 6][d] = s;
  } else {
    red[grp][d] = s;
  }
  __syncthreads();
  if (grp == 0) {
    double t = 0.0;
#pragma unroll
    for (int r = 0; r < kRows; ++r) t += red[r][d];
    a.mu[(int64_t)unit * kHeadDim + col] = a.n > 0 ? (float)(t / (double)a.n) : 0.f;
  }
}

hipError_t launch_key_mean(const MeanArgs& a, hipStream_t s) {
  if (a.units <= 0) return hipSuccess;
  if (a.nchunk > 0) {
    dim3 grid((unsigned)a.nchunk, (unsigned)a.units);
    // Keys that do not fit the 32 MB of L2 are read with the non-temporal hint (201 MB: 41.5 -> 33.5 us,
    // 6.0 TB/s; without the hint 40.8); smaller caches stay in L2 for the key hashing that reads them next
    // (4096 float32 keys: the two calls 1.5 us longer with the hint).
    const int et = a.is_fp32 ? kFP32 : (a.kv_fp8 ? kFP8 : kBF16);
    const bool nt = (int64_t)a.units * a.n * kHeadDim * elem_bytes(et) > (int64_t)32 << 20;
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, a); };
    if (et == kFP32) nt ? go(key_mean_partial_kernel<kFP32, true>) : go(key_mean_partial_kernel<kFP32, false>);
    else if (et == kFP8) nt ? go(key_mean_partial_kernel<kFP8, true>) : go(key_mean_partial_kernel<kFP8, false>);
    else nt ? go(key_mean_partial_kernel<kBF16, true>) : go(key_mean_partial_kernel<kBF16, false>);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  // (32 chunks: four per thread, which the loop requests together)
  if (a.nchunk <= 32) hipLaunchKernelGGL(key_mean_final_kernel<kHeadDim>, dim3((unsigned)a.units), dim3(1024), 0, s, a);
  else hipLaunchKernelGGL(key_mean_final_kernel<16>, dim3((unsigned)a.units, kHeadDim / 16), dim3(1024), 0, s, a);
  return hipGetLastError();
}

}  // namespace mp
