// SimHash coding of cached float32 keys on the matrix cores (Sec. 4.3 "Hash function selection").
//
// A workgroup codes 32 keys of one (batch, KV head) against the 32 K projector columns of one table
// group; a wavefront takes every fourth tile of 32 neighbouring columns (v_mfma_f32_32x32x2_f32: A
// operand = columns, B operand = keys, so an accumulator register holds one (column, key) pair with
// lane % 32 = key).  W is read as it is stored, row by row, 128 contiguous bytes per half wavefront,
// from L2: the call needs no workspace and no pass over W before it.  The sign bits of a key come out
// in column order and are regrouped into plane words through LDS.
//
// Bit-exactness.  The hash bit is the sign of the exact sum k.W_j - mu.W_j.  The B operand is
// fl(k - mu), each element within 2^-24 of its magnitude, so with x = k - mu the matrix-core result is
// within kGammaF32 |x| |W_j| of the exact sum: one rounding of the difference, one of every product
// (2^-24 each) and the accumulation of 128 products in any order and grouping, each step losing at
// most 2^-23 of the running magnitude, 2^-16 + 2^-22.4 in all; 2^-15 leaves a factor of two.
// (Cauchy-Schwarz over the terms; the floor added to it covers products below the normal range,
// kSquareSlack what their squares lose in the norms.)
// Results inside that bound are listed in LDS - the list holds every pair of the workgroup, so it
// cannot overflow - and re-evaluated in float64 from exact products, and what float64 cannot decide
// is summed exactly (exact_dot.h).
//
// 4096 keys x 600 columns (one head, (8,75)): 24.6 us, a chain of latencies (two tiles of 64 dependent
// matrix instructions per wavefront are 4 us of it); the first version, a float64 dot product per lane
// with the columns of neighbouring lanes K elements apart, took 1038 us.
#include "mp_common.h"
#include "exact_dot.h"
#include "device_utils.h"

namespace mp {

typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr float kGammaF32 = 3.0517578125e-5f;             // 2^-15
constexpr int kTileKeys = 32;

__global__ __launch_bounds__(256, 3) void hash_keys_f32_kernel(HashDirectArgs a, uint32_t tiles, uint32_t jobs) {
  __shared__ uint32_t colbits[16][kTileKeys];             // [32-column tile][key]: sign bits in column order
  __shared__ uint32_t plane[16][kTileKeys];               // last table group: its plane words
  __shared__ uint16_t list[16 * 32 * kTileKeys];          // pairs to re-evaluate: column << 5 | key
  __shared__ unsigned count;
  __shared__ long long limbs[4][kLimbs];
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int kap = lane & 31, hh = lane >> 5;
  const int unit = blockIdx.y;
  const int K = a.K, ncol = a.K * a.L, Wd = table_words(a.L);
  const int64_t first = a.first_key, last = a.first_key + a.n_keys;
  const int64_t ubase = (int64_t)(unit / a.n_kv_heads) * a.stride_b + (int64_t)(unit % a.n_kv_heads) * a.stride_h;
  const float* X = reinterpret_cast<const float*>(a.X) + ubase;
  const float* W = reinterpret_cast<const float*>(a.W);
  const float* mu = a.mu ? a.mu + (int64_t)unit * kHeadDim : nullptr;
  if (lane < kLimbs) limbs[wave][lane] = 0;

  for (uint32_t job = blockIdx.x; job < jobs; job += gridDim.x) {
    const int w = (int)(job / tiles);
    const int64_t key0 = (first / kTileKeys + (int64_t)(job % tiles)) * kTileKeys;
    const int64_t key = key0 + kap;
    const bool key_ok = key >= first && key < last;
    const int64_t krow = key_ok ? key : first;            // (any valid row for masked lanes)
    if (tid == 0) count = 0;

    // ---- B operand: k - mu, lane half hh holds the elements 64 hh .. 64 hh + 63 ----
    float B[64];
    float ss = kSquareSlack;
    {
      const float4* kr = reinterpret_cast<const float4*>(X + krow * a.stride_n + 64 * hh);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float4 v = kr[i];
        B[4 * i] = v.x; B[4 * i + 1] = v.y; B[4 * i + 2] = v.z; B[4 * i + 3] = v.w;
      }
      if (mu) {
        const float4* mr = reinterpret_cast<const float4*>(mu + 64 * hh);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float4 v = mr[i];
          B[4 * i] -= v.x; B[4 * i + 1] -= v.y; B[4 * i + 2] -= v.z; B[4 * i + 3] -= v.w;
          if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // (a few at a time: the registers are few)
        }
      }
#pragma unroll
      for (int i = 0; i < 64; ++i) ss = fmaf(B[i], B[i], ss);
    }
    ss += __shfl_xor(ss, 32);
    const float xnorm = sqrtf(ss) * 1.00002f;
    __syncthreads();                                      // count is clear

    for (int tile = wave; tile < K; tile += 4) {
      const int j = 32 * w * K + 32 * tile + kap;         // this lane's column (A operand row)
      const bool col_ok = j < ncol;
      // 16 elements of the column are requested while the 16 before them are multiplied
      const uint32_t at = (uint32_t)(64 * hh * ncol + (col_ok ? j : 0));   // (128 * 8192 elements at most)
      float A[2][16];
      float w2 = kSquareSlack;
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
      uint32_t step = (uint32_t)ncol;
      asm volatile("" : "+s"(step));                       // (row offsets are worked out here, not kept across tiles)
#pragma unroll
      for (int i = 0; i < 16; ++i) A[0][i] = (W + (uint32_t)i * step)[at];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (c < 3) {
#pragma unroll
          for (int i = 0; i < 16; ++i) A[(c + 1) & 1][i] = (W + (uint32_t)(16 * (c + 1) + i) * step)[at];
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          w2 = fmaf(A[c & 1][i], A[c & 1][i], w2);
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(A[c & 1][i], B[16 * c + i], acc, 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      w2 += __shfl_xor(w2, 32);
      const float bound = key_ok ? kGammaF32 * xnorm * (sqrtf(wave_max(w2)) * 1.00002f) + 1e-30f : -1.f;
      // register r: column 8 (r / 4) + 4 hh + r % 4 of the tile
      uint32_t neg = 0, fl = 0;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        neg |= (uint32_t)(acc[r] < 0.f) << r;
        fl |= (uint32_t)!(fabsf(acc[r]) > bound) << r;
      }
      auto spread = [&](uint32_t m) {
        return ((m & 0xfu) | (m & 0xf0u) << 4 | (m & 0xf00u) << 8 | (m & 0xf000u) << 12) << (4 * hh);
      };
      const int left = ncol - (32 * w * K + 32 * tile);   // columns from the first of the tile on
      const uint32_t real = left >= 32 ? ~0u : (left > 0 ? (1u << left) - 1u : 0u);
      uint32_t bits = spread(~neg & 0xffffu);
      bits |= __shfl_xor(bits, 32);
      uint32_t close = key_ok ? spread(fl) & real : 0u;
      if (hh == 0) colbits[tile][kap] = bits & real;
      if (close) {
        unsigned pos = atomicAdd(&count, (unsigned)__popc(close));
        for (; close; close &= close - 1) list[pos++] = (uint16_t)((32 * tile + __ffs(close) - 1) << 5 | kap);
      }
    }
    __syncthreads();

    // ---- re-evaluation: 16 lanes per pair ----
    const unsigned cnt = count;
    int ln = lane;
    asm volatile("" : "+v"(ln));
    for (unsigned i0 = wave * 4; i0 < cnt; i0 += 16) {
      const unsigned i = i0 + (ln >> 4);
      const bool on = i < cnt;
      const int e = list[on ? i : i0], col = e >> 5, ek = e & 31, sl = ln & 15;
      const int j = 32 * w * K + col;
      const float* kr = X + (key0 + ek) * a.stride_n;
      float kv[8], wv[8], mv[8];
      load8<kFP32>(kr, sl * 8, kv);
#pragma unroll
      for (int d = 0; d < 8; ++d) wv[d] = W[(int64_t)(sl * 8 + d) * ncol + j];
      if (mu) load8<kFP32>(mu, sl * 8, mv);
      double s = 0.0, mag = 0.0;
#pragma unroll
      for (int d = 0; d < 8; ++d) {
        const double p = (double)kv[d] * (double)wv[d];   // exact
        s += p;
        mag += fabs(p);
        if (mu) {
          const double pm = (double)mv[d] * (double)wv[d];   // exact
          s -= pm;
          mag += fabs(pm);
        }
      }
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) {
        s += __shfl_xor(s, o);
        mag += __shfl_xor(mag, o);
      }
      bool bit = s >= 0.0;
      uint64_t pending = __ballot(on && sl == 0 && mag > 0.0 && fabs(s) <= kF64Slack * mag);
      while (pending) {
        const int src = __ffsll((unsigned long long)pending) - 1;
        const int sj = __shfl(j, src), sk = __shfl(ek, src);
        const float* skr = X + (key0 + sk) * a.stride_n;
        const bool r = exact_sign_nonneg_wave(
            limbs[wave], [&](int d) { return (double)skr[d]; }, [&](int d) { return (double)W[(int64_t)d * ncol + sj]; },
            [&](int d) { return mu ? (double)mu[d] : 0.0; }, mu != nullptr);
        if (lane == src) bit = r;
        pending &= pending - 1;
      }
      if (on && sl == 0) {
        if (bit) atomicOr(&colbits[col >> 5][ek], 1u << (col & 31));
        else atomicAnd(&colbits[col >> 5][ek], ~(1u << (col & 31)));
      }
    }
    __syncthreads();

    // ---- plane word b of a key: its columns b, b + K, b + 2 K, ... ----
    const bool tail = w == Wd - 1;
    int t0 = tid;
    asm volatile("" : "+v"(t0));                            // (nothing of this is kept in registers across jobs)
    for (int item = t0; item < K * kTileKeys; item += 256) {
      const int b = item >> 5, ek = item & 31;
      uint32_t word = 0;
      for (int beta = 0, pos = b; beta < 32; ++beta, pos += K)
        word |= ((colbits[pos >> 5][ek] >> (pos & 31)) & 1u) << beta;
      if (tail) plane[b][ek] = word;
      const int64_t k = key0 + ek;
      if (!tail && k >= first && k < last)
        a.codes[(unit * a.blocks_cap + k / kBlockKeys) * (kBlockKeys * (int64_t)a.NW) +
                slot_in_block(a.NW, w * K + b, (int)(k % kBlockKeys))] = word;
    }
    __syncthreads();
    if (tail) {
      // the K planes of the last group as one bit string of tail_tables bits each
      const int Lt = tail_tables(a.L), xs = tail_begin(K, a.L), nt = a.NW - xs;
      for (int item = t0; item < nt * kTileKeys; item += 256) {
        const int ek = item & 31, e = item >> 5;
        uint32_t word = 0;
        int b = 32 * e / Lt, at = 32 * e % Lt;            // plane and table of bit 32 e
        for (int have = 0; have < 32 && b < K; ++b, at = 0) {
          word |= (plane[b][ek] >> at) << have;           // (a plane's bits beyond Lt are zero)
          have += Lt - at;
        }
        const int64_t k = key0 + ek;
        if (k >= first && k < last)
          a.codes[(unit * a.blocks_cap + k / kBlockKeys) * (kBlockKeys * (int64_t)a.NW) +
                  slot_in_block(a.NW, xs + e, (int)(k % kBlockKeys))] = word;
      }
    }
  }
}

// Keys [first_key, first_key + n_keys) of every unit (n_keys > 0).
hipError_t launch_hash_keys_f32(const HashDirectArgs& a, int units, hipStream_t s) {
  const int64_t tiles = (a.first_key + a.n_keys - 1) / kTileKeys - a.first_key / kTileKeys + 1;
  const int64_t jobs = tiles * table_words(a.L);           // n_cap <= 2^31 keys: below 2^31
  const int64_t most = (int64_t)1 << 22;                   // (gridDim.x * 256 threads below 2^32; the kernel walks the rest)
  hipLaunchKernelGGL(hash_keys_f32_kernel, dim3((unsigned)(jobs < most ? jobs : most), (unsigned)units), dim3(256), 0, s, a,
                     (uint32_t)tiles, (uint32_t)jobs);
  return hipGetLastError();
}

}  // namespace mp
