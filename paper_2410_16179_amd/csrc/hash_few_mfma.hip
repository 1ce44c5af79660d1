// SimHash coding of a few bf16 vectors on the matrix cores: the queries of a decode step
// (Algorithm 1 "Encode(q, W)") and the newest keys of every (batch, KV head), which join the hash
// structure behind the frozen centering vector (Sec. 4.3 "Data pre-processing"; Sec. 4.4 (3)).
//
// The step is latency-bound (a few thousand vectors at most against 384 KB of projector), so the
// kernel is built around one memory round trip.  The projector is read in a prepared form
// (magicpig_prepare_projector, once per model): MFMA A fragments, 16 bytes per lane and load,
// grouped so that a workgroup = one group of 32 tables and a wavefront = two of its bit planes.
// A wavefront requests its two A tiles and up to 64 vectors (B operand, lane%32 = vector) at
// once, multiplies (v_mfma_f32_32x32x16_bf16), and has the 32 sign bits of a plane word inside
// one lane as in the key-hashing kernel.  Keys enter with the prepared initial accumulators
// -fl(mu.W_j) (magicpig_prepare_centering, once per sequence: the mean is frozen).
//
// Bit-exactness: as in hash_keys_mfma.hip a projection with |acc| <= kGamma (|x| + |mu|) max|W_j|
// is re-evaluated exactly.  Here the re-evaluation never leaves the compute unit: the vectors and
// the projector columns sit in the wavefronts' registers and are copied to LDS (the centering vectors
// were put there at the start), sixteen lanes per projection form the exact float64 products of eight
// elements each, rotations inside the row add them, and what float64 cannot decide goes to the exact
// accumulator (exact_dot.h).  The owning lane patches its bit before the word is stored,
// so there is no list, no overflow and no atomic.
#include "mp_common.h"
#include "exact_dot.h"
#include "device_utils.h"
#include <hip/hip_ext.h>

namespace mp {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

// Row rho of tile tau of a plane pair: plane 2p + eta, bit beta of the plane word (table 32w + beta).
// Accumulator register r = 4*(rho/8) + rho%4 of lane half eta; inserted most significant bit first.
__host__ __device__ inline void few_row_to_bit(int tau, int rho, int* eta, int* beta) {
  *eta = (rho >> 2) & 1;
  *beta = 31 - (16 * tau + 4 * (rho >> 3) + (rho & 3));
}

__global__ void prep_few_header_kernel(uint32_t* header, int K, int L) {
  if (threadIdx.x == 0) {
    header[0] = kPreparedMagic;
    header[1] = (uint32_t)K;
    header[2] = (uint32_t)L;
    header[3] = 0u;                                        // largest column norm: raised by the next kernel
  }
}

// One thread per (tile row, 8-element piece of d): fragment, transposed copy, column norm.
__global__ __launch_bounds__(256) void prep_few_fragments_kernel(const uint16_t* W, uint32_t* header, uint4* frag,
                                                                 uint4* wt, int K, int L) {
  const int gid = blockIdx.x * 256 + threadIdx.x;
  const int P = (K + 1) / 2, Wd = table_words(L);
  const int row = gid >> 4, piece = gid & 15;              // row = ((w*P + p)*2 + tau)*32 + rho
  const bool row_in = row < Wd * P * 64;
  const int rho = row & 31, tau = (row >> 5) & 1, wp = row >> 6;
  const int p = wp % P, w = wp / P;
  int eta, beta;
  few_row_to_bit(tau, rho, &eta, &beta);
  const int b = 2 * p + eta, t = 32 * w + beta;
  const bool real = row_in && b < K && t < L;
  const int ncol = K * L, j = real ? t * K + b : 0;
  uint16_t v[8];
  float ss = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    v[e] = real ? W[(int64_t)(piece * 8 + e) * ncol + j] : (uint16_t)0;
    const float f = __uint_as_float((uint32_t)v[e] << 16);
    ss += f * f;
  }
  uint4 pk;
  pk.x = v[0] | ((uint32_t)v[1] << 16); pk.y = v[2] | ((uint32_t)v[3] << 16);
  pk.z = v[4] | ((uint32_t)v[5] << 16); pk.w = v[6] | ((uint32_t)v[7] << 16);
  const int s = piece >> 1, lane = (piece & 1) * 32 + rho;
  if (row_in) frag[((int64_t)(row >> 5) * 8 + s) * 64 + lane] = pk;
  if (real) wt[(int64_t)j * 16 + piece] = pk;
  ss = row_sum16(ss);                                      // the 16 pieces of a row sit in one DPP row
  if (real && piece == 0) atomicMax(&header[3], __float_as_uint(sqrtf(ss) * 1.000001f));   // (non-negative floats order like integers)
}

__global__ __launch_bounds__(256) void prep_few_copy_kernel(const uint4* src, uint4* dst, int64_t count) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256) dst[i] = src[i];
}

// Per (batch, KV head): initial accumulators -fl(mu.W_j) in fragment order, and |mu|.
__global__ __launch_bounds__(256) void prep_centering_kernel(const float* mu_all, const uint16_t* wt, float* thr,
                                                             float* munorm, int K, int L) {
  const int unit = blockIdx.y;
  const int row = blockIdx.x * 256 + threadIdx.x;
  const int P = (K + 1) / 2, Wd = table_words(L);
  const float* mu = mu_all + (int64_t)unit * kHeadDim;
  if (row == 0) {
    double ss = 0.0;
    for (int d = 0; d < kHeadDim; ++d) ss += (double)mu[d] * (double)mu[d];
    munorm[unit] = (float)sqrt(ss) * 1.000001f;
  }
  if (row >= Wd * P * 64) return;
  const int rho = row & 31, tau = (row >> 5) & 1, wp = row >> 6;
  const int p = wp % P, w = wp / P;
  int eta, beta;
  few_row_to_bit(tau, rho, &eta, &beta);
  const int b = 2 * p + eta, t = 32 * w + beta;
  float c = 0.f;                                           // rows outside the projector are masked by the kernel
  if (b < K && t < L) {
    const uint16_t* wr = wt + (int64_t)(t * K + b) * kHeadDim;
    double th = 0.0;
    for (int d = 0; d < kHeadDim; ++d) th += (double)mu[d] * (double)__uint_as_float((uint32_t)wr[d] << 16);
    c = 0.0f - (float)th;                                  // +0 when the threshold is zero
  }
  const int r = 4 * (rho >> 3) + (rho & 3);
  thr[((((int64_t)unit * Wd * P + wp) * 2 + tau) * 2 + eta) * 16 + r] = c;
}

// LDS of a workgroup besides the static arrays: the vectors (two tiles of queries, or one tile of keys
// and their 32 centering vectors), and per wavefront one or both of its A tiles and the list of its
// projections that are being re-evaluated.
constexpr int kFewList = 256;                              // entries per wavefront
constexpr int kTilePieces = 8 * 64;                        // 16-byte pieces of a tile (of the projector or of vectors)
static size_t few_lds(const HashFewArgs& a, int held_tiles) {
  return a.vector_bytes + (size_t)a.P * (held_tiles * kTilePieces * sizeof(uint4) + kFewList * sizeof(uint16_t));
}

// HELD: A tiles of a wavefront that LDS holds at once, 1 or 2.
template <int HELD>
__global__ __launch_bounds__(512) void hash_few_mfma_kernel(HashFewArgs a) {
  extern __shared__ uint4 few_mem[];
  uint4* sB = few_mem;                                     // [vector tile][k-step][lane]
  float (*sMu)[kHeadDim] = reinterpret_cast<float (*)[kHeadDim]>(few_mem + kTilePieces);   // (keys: there is no second tile)
  uint4* sA = few_mem + a.vector_bytes / 16 + (threadIdx.x >> 6) * (HELD * kTilePieces);   // [tile][k-step][lane]
  uint16_t* list = reinterpret_cast<uint16_t*>(few_mem + a.vector_bytes / 16 + a.P * HELD * kTilePieces) + (threadIdx.x >> 6) * kFewList;
  __shared__ uint32_t sTail[16][32];                       // plane words of the last table group, [plane][key]
  __shared__ long long sLimbs[8][kLimbs];
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int kap = lane & 31, hh = lane >> 5;
  const int w = blockIdx.x, p = wave;
  const bool is_key = (int)blockIdx.y >= a.q_groups;
  const int grp = is_key ? (int)blockIdx.y - a.q_groups : (int)blockIdx.y;
  int64_t first_key = a.first_key;
  if (is_key && a.n_dev) {                                 // the newest keys of a context whose length lives in device memory
    first_key = *a.n_dev - a.n_keys;
    if (first_key < 0 || first_key + a.n_keys > a.n_cap) return;    // (uniform in the workgroup, before any barrier)
  }
  if (lane < kLimbs) sLimbs[wave][lane] = 0;

  // ---- everything the wavefront needs from memory, requested at once ----
  bf16x8 A[2][8], B[2][8];
  const uint4* fr = reinterpret_cast<const uint4*>(a.frag) + (int64_t)(w * a.P + p) * 2 * 8 * 64 + lane;
#pragma unroll
  for (int tau = 0; tau < 2; ++tau)
#pragma unroll
    for (int s = 0; s < 8; ++s) A[tau][s] = __builtin_bit_cast(bf16x8, fr[(tau * 8 + s) * 64]);
  bool ok[2] = {false, false};
  const uint16_t* rp[2];
  int64_t unit = 0, key = 0;
  if (!is_key) {
#pragma unroll
    for (int bt = 0; bt < 2; ++bt) {
      const int v = grp * 64 + bt * 32 + kap;
      ok[bt] = v < a.n_q;
      rp[bt] = reinterpret_cast<const uint16_t*>(a.q) + (int64_t)(ok[bt] ? v : 0) * kHeadDim;
    }
  } else {
    const int r = grp * 32 + kap;
    ok[0] = r < a.n_krows;
    // (at most 128 key vectors: 32-bit divisions)
    const uint32_t rr = ok[0] ? (uint32_t)r : 0u, nk = (uint32_t)a.n_keys, hk = (uint32_t)a.n_kv_heads;
    unit = rr / nk;
    key = first_key + rr % nk;
    rp[0] = reinterpret_cast<const uint16_t*>(a.Kc) + (int64_t)((uint32_t)unit / hk) * a.stride_b +
            (int64_t)((uint32_t)unit % hk) * a.stride_h + key * a.stride_n;
    rp[1] = rp[0];
  }
  const bool key8 = is_key && a.kv_fp8;                    // the key rows are e4m3 bytes (wave-uniform)
  const bool two = !is_key && grp * 64 + 32 < a.n_q;       // a second tile of vectors (wave-uniform)
  if (key8) {
    // (same element offset, one byte per element; widened to the same values in bf16)
    const uint8_t* row8 = reinterpret_cast<const uint8_t*>(a.Kc) + (rp[0] - reinterpret_cast<const uint16_t*>(a.Kc)) + hh * 8;
    uint2 r8[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) r8[s] = *reinterpret_cast<const uint2*>(row8 + s * 16);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      B[0][s] = __builtin_bit_cast(bf16x8, fp8x8_to_bf16x8(r8[s].x, r8[s].y));
      B[1][s] = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
    }
  } else {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      B[0][s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(rp[0] + s * 16 + hh * 8));
      if (two) B[1][s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(rp[1] + s * 16 + hh * 8));
      else B[1][s] = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
    }
  }
  const bool centered = is_key && a.mu != nullptr;
  f32x16 acc[2][2];
#pragma unroll
  for (int tau = 0; tau < 2; ++tau)
#pragma unroll
    for (int r = 0; r < 16; ++r) { acc[tau][0][r] = 0.f; acc[tau][1][r] = 0.f; }
  float munorm = 0.f;
  if (centered) {
    const float* tp = a.thr + ((((int64_t)unit * a.Wd * a.P + (w * a.P + p)) * 2) * 2 + hh) * 16;
#pragma unroll
    for (int tau = 0; tau < 2; ++tau)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        const float4 t4 = *reinterpret_cast<const float4*>(tp + tau * 32 + v4 * 4);
        acc[tau][0][v4 * 4] = t4.x; acc[tau][0][v4 * 4 + 1] = t4.y; acc[tau][0][v4 * 4 + 2] = t4.z; acc[tau][0][v4 * 4 + 3] = t4.w;
      }
    munorm = a.munorm[unit];
    // the centering vectors themselves, for the exact re-evaluation
    for (int i = tid; i < 32 * 32; i += blockDim.x) {
      const int kk = i >> 5, piece = i & 31;
      const int r = grp * 32 + kk;
      if (r < a.n_krows)
        reinterpret_cast<float4*>(sMu[kk])[piece] =
            reinterpret_cast<const float4*>(a.mu + (int64_t)((uint32_t)r / (uint32_t)a.n_keys) * kHeadDim)[piece];
    }
  }
  const float wmax = __uint_as_float(a.header[3]);
  // the vectors to LDS, for the same: wavefront v writes the k-steps v, v + P, ...
  uint32_t my_steps = 0;
  for (int s = wave; s < 8; s += a.P) my_steps |= 1u << s;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    if (!(my_steps >> s & 1)) continue;
    sB[s * 64 + lane] = __builtin_bit_cast(uint4, B[0][s]);
    if (two) sB[(8 + s) * 64 + lane] = __builtin_bit_cast(uint4, B[1][s]);
  }

  // ---- error bound per vector: kGamma (|x| + |mu|) max|W_j| ----
  // (|x|^2 by v_dot2_f32_bf16, two exact products per instruction, float32 accumulation: the
  // relative error of the norm, below 1e-5, is inside the margin of kGamma)
  float bnd[2] = {-1.f, -1.f};
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
#pragma unroll
  for (int bt = 0; bt < 2; ++bt) {
    if (bt == 1 && !two) break;
    float ss = kSquareSlack;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const uint4 raw = __builtin_bit_cast(uint4, B[bt][s]);
      const uint32_t u[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bf16x2 v2 = __builtin_bit_cast(bf16x2, u[i]);
        ss = __builtin_amdgcn_fdot2_f32_bf16(v2, v2, ss, false);
      }
    }
    ss += __shfl_xor(ss, 32);                              // the other half of the row
    const float xnorm = sqrtf(ss) * 1.00002f;
    bnd[bt] = ok[bt] ? (kGamma * (xnorm + munorm) * (wmax + kNormSlack)) * 1.000001f + 1e-30f : -1.f;
  }

  // ---- multiply ----
#pragma unroll
  for (int tau = 0; tau < 2; ++tau)
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      acc[tau][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[tau][s], B[0][s], acc[tau][0], 0, 0, 0);
      if (two) acc[tau][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[tau][s], B[1][s], acc[tau][1], 0, 0, 0);
    }
  // sign bits and "too close to zero" flags, most significant bit first (bit beta of the plane
  // word): neg = 1 where the projection is negative.  The accumulator starts from +0 or a
  // non-zero threshold and round-to-nearest never produces -0 from a sum, so the sign bit is the
  // test "< 0".
  // The flags cost as much as the signs and are almost always all zero: the smallest |acc| of a
  // lane is compared with its bound first, and the per-bit flags are formed only by wavefronts
  // in which some lane has one below it.
  uint32_t neg[2] = {0, 0}, fl[2] = {0, 0};
  bool close_lane = false;
#pragma unroll
  for (int bt = 0; bt < 2; ++bt) {
    if (bt == 1 && !two) break;
    float lo = INFINITY;
#pragma unroll
    for (int tau = 0; tau < 2; ++tau)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        neg[bt] = __builtin_amdgcn_alignbit(neg[bt], __float_as_uint(acc[tau][bt][r]), 31);
        lo = fminf(lo, fabsf(acc[tau][bt][r]));
      }
    close_lane |= lo < bnd[bt];
  }
  if (__ballot(close_lane)) {
#pragma unroll
    for (int bt = 0; bt < 2; ++bt) {
      if (bt == 1 && !two) break;
#pragma unroll
      for (int tau = 0; tau < 2; ++tau)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          fl[bt] = __builtin_amdgcn_alignbit(fl[bt], __float_as_uint(fabsf(acc[tau][bt][r]) - bnd[bt]), 31);
    }
  }
  // this lane half's plane and the tables that exist in this group
  const int b_my = 2 * p + hh;
  const uint32_t tmask = (w == a.Wd - 1 && (a.L & 31)) ? (1u << (a.L & 31)) - 1u : ~0u;
  const uint32_t vmask = b_my < a.K ? tmask : 0u;
  fl[0] &= vmask;
  fl[1] &= two ? vmask : 0u;
  // ---- exact re-evaluation of the flagged projections, from LDS, four at a time ----
  // The vectors are in LDS, the A tiles of a wavefront that has flagged something go there; its flags become
  // a list, and sixteen lanes take an entry, eight elements each.
  // (One at a time - the two lanes that hold the vector and the two that hold the column wrote them to
  // LDS, the wavefront formed two products per lane - an entry cost 0.7 us, and a group of 32 keys has up to
  // eight of them in a wavefront.)
  __syncthreads();
  // (tile 0 of the wavefront holds bits 31 .. 16 of a plane word, tile 1 the others)
#pragma unroll 1
  for (int tile0 = 0; tile0 < 2; tile0 += HELD) {
    const uint32_t held = HELD == 2 ? ~0u : (tile0 == 0 ? 0xffff0000u : 0x0000ffffu);
    if (!__ballot(((fl[0] | fl[1]) & held) != 0u)) continue;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      sA[s * 64 + lane] = __builtin_bit_cast(uint4, HELD == 2 || tile0 == 0 ? A[0][s] : A[1][s]);
      if (HELD == 2) sA[kTilePieces + s * 64 + lane] = __builtin_bit_cast(uint4, A[1][s]);
    }
    do {
      // entry: owner lane | vector tile << 6 | bit << 7 (| result << 15)
      const int mine = __popc(fl[0] & held) + __popc(fl[1] & held);
      const int incl = half_prefix_sum32(mine);
      const int low = __builtin_amdgcn_readlane(incl, 31), cnt_all = low + __builtin_amdgcn_readlane(incl, 63);
      const int pos0 = incl - mine + (hh ? low : 0);
      const int cnt = cnt_all < kFewList ? cnt_all : kFewList;
      int pos = pos0;
#pragma unroll
      for (int bt = 0; bt < 2; ++bt)
        for (uint32_t f = fl[bt] & held; f && pos < kFewList; f &= f - 1) list[pos++] = (uint16_t)(lane | bt << 6 | (__ffs(f) - 1) << 7);
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
      __builtin_amdgcn_wave_barrier();
      const int slot = lane >> 4, sl = lane & 15;
      for (int i0 = 0; i0 < cnt; i0 += 4) {
        const bool on = i0 + slot < cnt;
        const int e = list[on ? i0 + slot : i0];
        const int el = 31 - (e >> 7 & 31), r = el & 15, hsrc = e >> 5 & 1, kap0 = e & 31;
        const int rho = 8 * (r >> 2) + 4 * hsrc + (r & 3);                    // tile row of the projection
        // elements 8 sl .. 8 sl + 7: k-step sl / 2, lane half sl % 2
        const int at16 = (sl >> 1) * 64 + (sl & 1) * 32;
        const uint4 xr = sB[(e >> 6 & 1) * kTilePieces + at16 + kap0], wr = sA[((el >> 4) - tile0) * kTilePieces + at16 + rho];
        const uint32_t xu[4] = {xr.x, xr.y, xr.z, xr.w}, wu[4] = {wr.x, wr.y, wr.z, wr.w};
        float mv[8];
        if (centered) {
          const float4 m0 = *reinterpret_cast<const float4*>(&sMu[kap0][sl * 8]), m1 = *reinterpret_cast<const float4*>(&sMu[kap0][sl * 8 + 4]);
          mv[0] = m0.x; mv[1] = m0.y; mv[2] = m0.z; mv[3] = m0.w; mv[4] = m1.x; mv[5] = m1.y; mv[6] = m1.z; mv[7] = m1.w;
        }
        double t = 0.0, g = 0.0;
#pragma unroll
        for (int d = 0; d < 8; ++d) {
          const double x = (double)__uint_as_float(d & 1 ? xu[d >> 1] & 0xffff0000u : xu[d >> 1] << 16);
          const double w64 = (double)__uint_as_float(d & 1 ? wu[d >> 1] & 0xffff0000u : wu[d >> 1] << 16);
          const double pr = x * w64;                                          // exact
          t += pr;
          g += fabs(pr);
          if (centered) {
            const double m = (double)mv[d] * w64;                             // exact
            t -= m;
            g += fabs(m);
          }
        }
        t = row_sum16(t);
        g = row_sum16(g);
        bool bit = t >= 0.0;
        // (what float64 cannot decide, one at a time)
        for (uint64_t pending = __ballot(on && sl == 0 && g > 0.0 && fabs(t) <= kF64Slack * g); pending; pending &= pending - 1) {
          const int at = __ffsll((unsigned long long)pending) - 1;
          const int pe = __builtin_amdgcn_readlane(e, at), pel = 31 - (pe >> 7 & 31), pr = pel & 15;
          const uint4* pw = sA + ((pel >> 4) - tile0) * kTilePieces + 8 * (pr >> 2) + 4 * (pe >> 5 & 1) + (pr & 3);
          const uint4* px = sB + (pe >> 6 & 1) * kTilePieces + (pe & 31);
          auto elem = [](const uint4* base, int d) {
            const uint16_t v = reinterpret_cast<const uint16_t*>(base + (d >> 4) * 64 + (d >> 3 & 1) * 32)[d & 7];
            return (double)__uint_as_float((uint32_t)v << 16);
          };
          const bool rb = exact_sign_nonneg_wave(
              sLimbs[wave], [&](int d) { return elem(px, d); }, [&](int d) { return elem(pw, d); },
              [&](int d) { return centered ? (double)sMu[pe & 31][d] : 0.0; }, centered);
          if (lane == at) bit = rb;
        }
        if (on && sl == 0 && bit) list[i0 + slot] = (uint16_t)(e | 0x8000);
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
      __builtin_amdgcn_wave_barrier();
      // the owners take their bits back
      pos = pos0;
#pragma unroll
      for (int bt = 0; bt < 2; ++bt)
        for (uint32_t f = fl[bt] & held; f && pos < kFewList; f &= f - 1) {
          const uint32_t m = f & -f;
          if (list[pos++] & 0x8000) neg[bt] &= ~m;
          else neg[bt] |= m;
          fl[bt] &= ~m;
        }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
      __builtin_amdgcn_wave_barrier();
    } while (__ballot(((fl[0] | fl[1]) & held) != 0u));
  }

  // ---- store ----
  if (!is_key) {
    // queries: plane words as they are, the tables beyond L set to 1 (they never collide)
    const uint32_t pad = b_my < a.K ? ~tmask : 0u;
    const uint32_t c0 = (~neg[0] & vmask) | pad, c1 = (~neg[1] & vmask) | pad;
    // lanes < 32 hold plane 2p of vectors kap / 32 + kap, lanes >= 32 plane 2p + 1: one half-swap
    // leaves lane l with both words of vector l
    const auto sw = __builtin_amdgcn_permlane32_swap(c0, c1, false, false);
    const int v = grp * 64 + lane;
    if (v < a.n_q) {
      uint32_t* dst = a.qcodes + (int64_t)v * a.NQ + w * a.K + 2 * p;
      dst[0] = sw[0];
      if (2 * p + 1 < a.K) dst[1] = sw[1];
    }
    return;
  }
  const uint32_t code = ~neg[0] & vmask;
  uint32_t* kdst = a.kcodes + (unit * a.blocks_cap + key / kBlockKeys) * (kBlockKeys * (int64_t)a.NW);
  const int kr = (int)(key % kBlockKeys);
  if (w < a.Wd - 1) {
    if (ok[0] && b_my < a.K) kdst[slot_in_block(a.NW, w * a.K + b_my, kr)] = code;
    return;
  }
  // keys, last table group: the K planes are stored as one bit string of tail_tables bits each
  sTail[b_my][kap] = code;                                 // b_my < 2P <= 16
  __syncthreads();
  if (wave == 0 && hh == 0 && ok[0]) {
    const int Lt = tail_tables(a.L);
    BitString bs;
    int xo = tail_begin(a.K, a.L);
    for (int b = 0; b < a.K; ++b) {
      uint32_t full;
      if (bs.append(sTail[b][kap], Lt, &full)) kdst[slot_in_block(a.NW, xo++, kr)] = full;
    }
    if (bs.nbits > 0) kdst[slot_in_block(a.NW, xo, kr)] = (uint32_t)bs.acc;
  }
}

hipError_t launch_prepare_projector(const void* W, void* prepared, int K, int L, hipStream_t s) {
  const PreparedLayout l = prepared_layout(K, L, false);
  char* base = reinterpret_cast<char*>(prepared);
  uint32_t* header = reinterpret_cast<uint32_t*>(base);
  hipLaunchKernelGGL(prep_few_header_kernel, dim3(1), dim3(64), 0, s, header, K, L);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int rows = l.Wd * l.P * 64;
  hipLaunchKernelGGL(prep_few_fragments_kernel, dim3((unsigned)((rows * 16 + 255) / 256)), dim3(256), 0, s,
                     reinterpret_cast<const uint16_t*>(W), header, reinterpret_cast<uint4*>(base + l.frag_off),
                     reinterpret_cast<uint4*>(base + l.wt_off), K, L);
  return hipGetLastError();
}

hipError_t launch_prepare_projector_fp32(const void* W, void* prepared, int K, int L, hipStream_t s) {
  const PreparedLayout l = prepared_layout(K, L, true);
  char* base = reinterpret_cast<char*>(prepared);
  hipLaunchKernelGGL(prep_few_header_kernel, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t*>(base), K, L);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t count = (int64_t)K * L * kHeadDim * 4 / 16;     // K*L*128 floats: a whole number of 16-byte pieces
  hipLaunchKernelGGL(prep_few_copy_kernel, dim3(64), dim3(256), 0, s, reinterpret_cast<const uint4*>(W),
                     reinterpret_cast<uint4*>(base + l.wt_off), count);
  return hipGetLastError();
}

hipError_t launch_prepare_centering(const float* mu, const void* prepared, void* centering, int K, int L, int units,
                                    hipStream_t s) {
  if (units <= 0) return hipSuccess;
  const PreparedLayout l = prepared_layout(K, L, false);
  const CenteringLayout c = centering_layout(K, L, (size_t)units);
  const char* pb = reinterpret_cast<const char*>(prepared);
  char* cb = reinterpret_cast<char*>(centering);
  const int rows = l.Wd * l.P * 64;
  hipLaunchKernelGGL(prep_centering_kernel, dim3((unsigned)((rows + 255) / 256), (unsigned)units), dim3(256), 0, s, mu,
                     reinterpret_cast<const uint16_t*>(pb + l.wt_off), reinterpret_cast<float*>(cb + c.thr_off),
                     reinterpret_cast<float*>(cb + c.munorm_off), K, L);
  return hipGetLastError();
}

hipError_t launch_hash_few(const HashFewArgs& a0, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  HashFewArgs a = a0;
  a.q_groups = (a.n_q + 63) / 64;
  const int k_groups = (a.n_krows + 31) / 32;
  if (a.q_groups + k_groups <= 0) return hipSuccess;
  const dim3 grid((unsigned)a.Wd, (unsigned)(a.q_groups + k_groups)), block(64 * a.P);
  a.vector_bytes = (a.n_krows > 0 && a.mu ? 8 + 16 : 16) * 1024;
  // Both A tiles at once, unless there are more workgroups than compute units and the room for one tile lets
  // more of them share one: the registers allow eight wavefronts, that is 8 / P workgroups.  32768 queries,
  // (8,75): 36.8 us with both tiles, 25.7 with one; with few workgroups the second pass over the flags costs more.
  const bool one = (int64_t)grid.x * grid.y > kNumCU && (a.P == 1 || a.P == 2 || a.P == 4);
  const size_t lds = few_lds(a, one ? 1 : 2);
  auto go = [&](auto kernel) {
    if (start || stop) hipExtLaunchKernelGGL(kernel, grid, block, lds, s, start, stop, 0, a);
    else hipLaunchKernelGGL(kernel, grid, block, lds, s, a);
  };
  if (one) go(hash_few_mfma_kernel<1>);
  else go(hash_few_mfma_kernel<2>);
  return hipGetLastError();
}

}  // namespace mp
