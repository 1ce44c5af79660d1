// SimHash coding of cached float32 keys on the matrix cores (Sec. 4.3 "Hash function selection").
//
// A workgroup codes 32 or 64 keys of one (batch, KV head) against the 32 K projector columns of one table
// group; each of its K wavefronts takes a tile of 32 neighbouring columns (v_mfma_f32_32x32x2_f32: A
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
// A chain of latencies, so all 64 elements of a lane's column are requested at once, together with the keys, which
// wait in LDS (16 at a time, the next ones requested while those before them are multiplied, cost a round trip to
// L2 each).  us of the kernel, four wavefronts with two tiles each and the keys in registers | now: 4096 keys x 600 columns
// (one head, (8,75)) 22.9 | 16.5; 8 x 2048 keys x 1500 columns 112.8 | 96.8 (6.3 GFLOP: 40 us at the rate of the
// instruction; workgroups of 64 keys are one per compute unit there, their list taking 4096 K bytes of LDS, and spill five registers).
#include "mp_common.h"
#include "exact_dot.h"
#include "device_utils.h"

namespace mp {

typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr float kGammaF32 = 3.0517578125e-5f;             // 2^-15
constexpr int kKeyRow = kHeadDim + 4;                      // floats of a key's row in LDS (16 lanes' 16-byte pieces on 64 banks)

// LDS of a workgroup: the keys, the list of pairs to re-evaluate and the accumulators of the exact sums, by K wavefronts
static size_t hash_f32_lds(int K, int keys) {
  return (size_t)K * kLimbs * sizeof(long long) + keys * kKeyRow * sizeof(float) + (size_t)K * 32 * keys * sizeof(uint16_t);
}

// KT: 32-key tiles of a workgroup.
template <int KT>
__global__ __launch_bounds__(1024, 4) void hash_keys_f32_kernel(HashDirectArgs a, uint32_t tiles, uint32_t jobs) {
  constexpr int kTileKeys = 32 * KT;                      // keys of a workgroup
  extern __shared__ __attribute__((aligned(16))) long long lds[];
  // (the keys are written and read 16 bytes at a time: every row of them begins on such a boundary)
  static_assert(kLimbs * sizeof(long long) % 16 == 0 && kKeyRow * sizeof(float) % 16 == 0, "");
  __shared__ uint32_t colbits[16][kTileKeys];             // [32-column tile][key]: sign bits in column order
  __shared__ uint32_t plane[16][kTileKeys];               // last table group: its plane words
  __shared__ float norms[kTileKeys];
  __shared__ unsigned count;
  const int tid = threadIdx.x, nthreads = blockDim.x;      // 64 K
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int kap = lane & 31, hh = lane >> 5;
  const int unit = blockIdx.y;
  const int K = a.K, ncol = a.K * a.L, Wd = table_words(a.L);
  long long* limbs = lds + wave * kLimbs;
  float* keys = reinterpret_cast<float*>(lds + K * kLimbs);   // [key][kKeyRow]: fl(k - mu)
  uint16_t* list = reinterpret_cast<uint16_t*>(keys + kTileKeys * kKeyRow);   // column << 6 | key
  const int64_t first = a.first_key, last = a.first_key + a.n_keys;
  const int64_t ubase = (int64_t)(unit / a.n_kv_heads) * a.stride_b + (int64_t)(unit % a.n_kv_heads) * a.stride_h;
  const float* X = reinterpret_cast<const float*>(a.X) + ubase;
  const float* W = reinterpret_cast<const float*>(a.W);
  const float* mu = a.mu ? a.mu + (int64_t)unit * kHeadDim : nullptr;
  if (lane < kLimbs) limbs[lane] = 0;

  for (uint32_t job = blockIdx.x; job < jobs; job += gridDim.x) {
    const int w = (int)(job / tiles);
    const int64_t key0 = (first / kTileKeys + (int64_t)(job % tiles)) * kTileKeys;
    if (tid == 0) count = 0;

    // ---- A operand: this lane's column of the wavefront's tile, lane half hh holds the elements 64 hh ..
    // 64 hh + 63; all of them are requested here and travel together with the keys ----
    const int tile = wave;
    const int j = 32 * w * K + 32 * tile + kap;
    const bool col_ok = j < ncol;
    const uint32_t at = (uint32_t)(64 * hh * ncol + (col_ok ? j : 0));   // (128 * 8192 elements at most)
    float A[64];
    const float* wrow = W;
#pragma unroll
    for (int i = 0; i < 64; ++i) {
      A[i] = wrow[at];
      wrow += ncol;
      asm volatile("" : "+s"(wrow));                       // (row addresses are worked out one by one: the registers are few)
    }

    // ---- B operand: k - mu, staged in LDS; sixteen lanes take a row ----
    for (int p = tid; p < kTileKeys * 16; p += nthreads) {
      const int row = p >> 4, c = (p & 15) * 8;
      const int64_t rkey = key0 + row;
      float v[8], m[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      load8<kFP32>(X, (rkey >= first && rkey < last ? rkey : first) * a.stride_n + c, v);   // (any valid row for masked keys)
      if (mu) load8<kFP32>(mu, c, m);
      float ss = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[e] -= m[e];
        ss = fmaf(v[e], v[e], ss);
      }
      *reinterpret_cast<float4*>(keys + row * kKeyRow + c) = make_float4(v[0], v[1], v[2], v[3]);
      *reinterpret_cast<float4*>(keys + row * kKeyRow + c + 4) = make_float4(v[4], v[5], v[6], v[7]);
      ss = row_sum16(ss) + kSquareSlack;
      if ((p & 15) == 0) norms[row] = sqrtf(ss) * 1.00002f;
    }
    __syncthreads();                                      // (count is clear, too)

    {
      float w2 = kSquareSlack;
      f32x16 acc[KT];
#pragma unroll
      for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
      const float4* brow = reinterpret_cast<const float4*>(keys + kap * kKeyRow + 64 * hh);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        float4 b4[KT];
#pragma unroll
        for (int t = 0; t < KT; ++t) b4[t] = brow[t * 32 * (kKeyRow / 4) + i];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          w2 = fmaf(A[4 * i + e], A[4 * i + e], w2);
#pragma unroll
          for (int t = 0; t < KT; ++t) {
            const float bv = e == 0 ? b4[t].x : (e == 1 ? b4[t].y : (e == 2 ? b4[t].z : b4[t].w));
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(A[4 * i + e], bv, acc[t], 0, 0, 0);
          }
        }
        if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
      w2 += __shfl_xor(w2, 32);
      const float wnorm = kGammaF32 * (sqrtf(wave_max(w2)) * 1.00002f);
      const int left = ncol - (32 * w * K + 32 * tile);   // columns from the first of the tile on
      const uint32_t real = left >= 32 ? ~0u : (left > 0 ? (1u << left) - 1u : 0u);
      auto spread = [&](uint32_t m) {
        return ((m & 0xfu) | (m & 0xf0u) << 4 | (m & 0xf00u) << 8 | (m & 0xf000u) << 12) << (4 * hh);
      };
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        const int ek = 32 * t + kap;
        const bool key_ok = key0 + ek >= first && key0 + ek < last;
        const float bound = key_ok ? wnorm * norms[ek] + 1e-30f : -1.f;
        // register r: column 8 (r / 4) + 4 hh + r % 4 of the tile
        uint32_t neg = 0, fl = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          neg |= (uint32_t)(acc[t][r] < 0.f) << r;
          fl |= (uint32_t)!(fabsf(acc[t][r]) > bound) << r;
        }
        uint32_t bits = spread(~neg & 0xffffu);
        bits |= __shfl_xor(bits, 32);
        uint32_t close = key_ok ? spread(fl) & real : 0u;
        if (hh == 0) colbits[tile][ek] = bits & real;
        if (close) {
          unsigned pos = atomicAdd(&count, (unsigned)__popc(close));
          for (; close; close &= close - 1) list[pos++] = (uint16_t)((32 * tile + __ffs(close) - 1) << 6 | ek);
        }
      }
    }
    __syncthreads();

    // ---- re-evaluation: 16 lanes per pair ----
    const unsigned cnt = count;
    int ln = lane;
    asm volatile("" : "+v"(ln));
    for (unsigned i0 = wave * 4; i0 < cnt; i0 += 4 * K) {
      const unsigned i = i0 + (ln >> 4);
      const bool on = i < cnt;
      const int e = list[on ? i : i0], col = e >> 6, ek = e & 63, sl = ln & 15;
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
            limbs, [&](int d) { return (double)skr[d]; }, [&](int d) { return (double)W[(int64_t)d * ncol + sj]; },
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
    for (int item = t0; item < K * kTileKeys; item += nthreads) {
      const int b = item / kTileKeys, ek = item % kTileKeys;
      uint32_t word = 0;
#pragma unroll 8
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
      for (int item = t0; item < nt * kTileKeys; item += nthreads) {
        const int ek = item % kTileKeys, e = item / kTileKeys;
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
  // n_cap <= 2^31 keys: below 2^31 jobs
  auto tiles_of = [&](int keys) { return (a.first_key + a.n_keys - 1) / keys - a.first_key / keys + 1; };
  auto jobs_of = [&](int keys) { return tiles_of(keys) * table_words(a.L); };
  auto go = [&](auto kernel, int keys) {
    const int64_t jobs = jobs_of(keys);
    const int64_t most = (int64_t)1 << 21;                 // (gridDim.x * 1024 threads below 2^32; the kernel walks the rest)
    hipLaunchKernelGGL(kernel, dim3((unsigned)(jobs < most ? jobs : most), (unsigned)units), dim3(64 * a.K), hash_f32_lds(a.K, keys), s, a,
                       (uint32_t)tiles_of(keys), (uint32_t)jobs);
  };
  if (hash_f32_keys(a.K, jobs_of(32) * units, jobs_of(64) * units) == 64) go(hash_keys_f32_kernel<2>, 64);
  else go(hash_keys_f32_kernel<1>, 32);
  return hipGetLastError();
}

}  // namespace mp
