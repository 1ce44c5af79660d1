// SimHash coding of cached bf16 keys on the matrix cores (Sec. 4.3 "Hash function
// selection"; Sec. 4.4 (3): the K*L random projections are the compute-bound step).
//
// The projection is a [keys x 128] x [128 x K*L] contraction.  It runs as bf16 MFMA
// (v_mfma_f32_32x32x16_bf16) with the projector as the A operand and 32 keys as the B
// operand, so an accumulator register of a lane holds one (projection, key) pair with
// lane%32 = key: the 32 sign bits of a code word are assembled inside one lane with one
// funnel shift per element and no cross-lane traffic.  Rows of the A operand are
// arranged (prep_hash_keys_kernel) so that the two lane halves of two consecutive MFMA
// tiles produce two complete code words; one half-swap then gives every lane the four
// words of "its" key and a wavefront stores a contiguous kilobyte of the code layout.
//
// Bit-exactness.  The hash bit is the sign of the exact sum  k.W_j - mu.W_j.  The MFMA
// result acc ~ k.W_j - fl(mu.W_j) (the threshold enters as the initial accumulator) differs
// from it by at most  kGamma * (|k_i| max_j |W_j| + max_j |mu.W_j|) + kThresholdSlack |mu| max_j |W_j|:
// every bf16 product is exact in float32, the accumulation inside the matrix core loses at most kGamma
// of the sum of magnitudes whatever its order and grouping (mp_common.h), the threshold is one term of
// that sum, and the other terms' magnitudes sum to |k_i| |W_j| at most (Cauchy-Schwarz); the largest
// threshold is that of the quad of tiles at hand.  The threshold itself is a float64 sum of 128 exact
// products: where they cancel, its error (127 roundings of 2^-53 of sum_d |mu_d W_dj| <= |mu| |W_j|) is
// what remains of the last term.  (Bounding the threshold by |mu| |W_j|, as if it were summed here,
// listed 1.4e-3 of the projections instead of 0.9e-3.)
// Elements with |acc| below that bound are listed in LDS and re-evaluated
// at the end of the workgroup in float64 with the exact fallback of exact_dot.h, which
// patches the bit.  Pairs beyond the LDS list go to a global list and finish_hash_keys_kernel
// (hash_direct.hip); if that overflows too, that kernel redoes the whole call in float64.
#include "mp_common.h"
#include "recheck_pairs.h"

namespace mp {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int kListCapLocal = 1536;       // flagged elements a workgroup can hold in LDS

// Projection handled by row rho (0..31) of MFMA tile T: tile pair T/2 makes code words
// x = 2*(T/2) + eta, eta = (rho/4)%2 being the lane half that receives the row; the row is
// accumulator register r = 4*(rho/8) + rho%4 of that half, inserted as element 16*(T%2) + r
// of the word, most significant bit first.
__host__ __device__ inline void tile_row_to_bit(int T, int rho, int* x, int* beta) {
  const int eta = (rho >> 2) & 1;
  const int r = 4 * (rho >> 3) + (rho & 3);
  *x = 2 * (T >> 1) + eta;
  *beta = 31 - (16 * (T & 1) + r);
}

// One launch prepares a call.
// The first `proj_blocks` workgroups (16 tile rows each): A-operand fragments, transposed bf16 copy
// of W for the recheck, largest column norm of the 16 rows.  One thread per (tile row, 8-element piece
// of d).  The first also clears the counters the later kernels of the call add to.
// The next, 256 projector columns of one (batch, KV head) each: initial accumulators -fl(mu.W_j) in
// fragment order and the same sums in float64.  A thread takes a column, neighbouring threads
// neighbouring columns, so that W is read in whole lines as it is stored.  (As two launches, the second
// reading the transposed copy row by row, they took 4.8 + 9.4 us.)
// With a centering vector units / 4 more, |mu| of four each.
__global__ __launch_bounds__(256) void prep_hash_keys_kernel(HashMfmaArgs a, int proj_blocks, int thr_blocks) {
  __shared__ float smax[4];
  const int tid = threadIdx.x;
  const int ncol = a.K * a.L;
  const uint16_t* W = reinterpret_cast<const uint16_t*>(a.W);
  if ((int)blockIdx.x < proj_blocks) {
    const int gid = blockIdx.x * 256 + tid;
    if (gid == 0) {
      *a.list_count = 0u;
      *a.overflow = 0;
      *a.flagged_total = 0u;
    }
    const int row = gid >> 4, piece = gid & 15;        // row = T*32 + rho  (ntiles is a multiple of four: no partial workgroup)
    const int T = row >> 5, rho = row & 31;
    int x, beta;
    tile_row_to_bit(T, rho, &x, &beta);
    const int t = 32 * (x / a.K) + beta;
    const bool real = x < a.NQ && t < a.L;
    const int j = real ? t * a.K + x % a.K : 0;
    uint16_t v[8];
    float ss = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v[e] = real ? W[(int64_t)(piece * 8 + e) * ncol + j] : (uint16_t)0;
      const float f = __uint_as_float((uint32_t)v[e] << 16);
      ss += f * f;
    }
    // fragment order: k-step s = piece/2, lane = (piece%2)*32 + rho, eight bf16 per lane
    const int s = piece >> 1, lane = (piece & 1) * 32 + rho;
    uint4 pk;
    pk.x = v[0] | ((uint32_t)v[1] << 16); pk.y = v[2] | ((uint32_t)v[3] << 16);
    pk.z = v[4] | ((uint32_t)v[5] << 16); pk.w = v[6] | ((uint32_t)v[7] << 16);
    reinterpret_cast<uint4*>(a.afrag)[((int64_t)T * 8 + s) * 64 + lane] = pk;
    if (real) reinterpret_cast<uint4*>(a.wt)[(int64_t)j * 16 + piece] = pk;
    ss = wave_max(row_sum16(ss));                      // the 16 pieces of a row sit in one DPP row; padding rows: 0
    if ((tid & 63) == 0) smax[tid >> 6] = ss;
    __syncthreads();
    if (tid == 0) a.rownorm[blockIdx.x] = sqrtf(fmaxf(fmaxf(smax[0], smax[1]), fmaxf(smax[2], smax[3]))) * 1.000001f;
    return;
  }
  const int at = (int)blockIdx.x - proj_blocks;
  if (at >= thr_blocks * a.units) {
    const int unit = (at - thr_blocks * a.units) * 4 + (tid >> 6), lane = tid & 63;
    if (unit < a.units) {
      const float* mu = a.mu + (int64_t)unit * kHeadDim;
      const float ss = wave_sum(fmaf(mu[lane], mu[lane], mu[lane + 64] * mu[lane + 64])) + kSquareSlack;
      if (lane == 0) a.munorm[unit] = sqrtf(ss) * 1.00002f;   // (infinite beyond 1.8e19: everything is then listed)
    }
    return;
  }
  const int unit = at / thr_blocks;
  const float* mu = a.mu ? a.mu + (int64_t)unit * kHeadDim : nullptr;
  // column i of the whole table groups (32 K columns each), then the words that pad the last quad
  const int i = at % thr_blocks * 256 + tid;
  if (i >= a.ntiles * 32) return;
  const bool grouped = i < 32 * a.NQ;
  const int w = i / (32 * a.K), rem = i % (32 * a.K);
  const int x = grouped ? w * a.K + rem % a.K : i >> 5, beta = grouped ? rem / a.K : i & 31;
  float c = -INFINITY;                                 // pad rows: never >= 0, never flagged
  if (i < ncol) {                                      // (i is the projector column itself)
    double th = 0.0, mg = 0.0;
    if (mu) {
#pragma unroll 32
      for (int d = 0; d < kHeadDim; ++d) {
        const double pm = (double)mu[d] * (double)__uint_as_float((uint32_t)W[(uint32_t)d * (uint32_t)ncol + (uint32_t)i] << 16);   // exact
        th += pm;
        mg += fabs(pm);
      }
    }
    c = 0.0f - (float)th;                              // +0 when the threshold is zero
    // for the exact re-evaluation: the same sum in float64 and a float32 upper bound of its magnitude sum
    a.thr64[(int64_t)unit * ncol + i] = th;
    a.magmu[(int64_t)unit * ncol + i] = mg > 0.0 ? (float)mg * 1.000001f + 2e-45f : 0.f;   // (2e-45: what the conversion loses below the normal range)
  }
  // word x, bit beta: tile 2 (x / 2) + el / 16, lane half x % 2, register el % 16, el = 31 - beta
  const int el = 31 - beta, T = 2 * (x >> 1) + (el >> 4);
  a.thr[(((int64_t)unit * a.ntiles + T) * 2 + (x & 1)) * 16 + (el & 15)] = c;
}

// One pair of tiles (2 tiles x 8 k-steps x 64 lanes x 16 bytes = 16 KB of fragments), global -> LDS
// without passing through registers: lane l of a wavefront supplies the address of its 16
// bytes, the hardware writes them to (wave-uniform LDS base) + 16 l.  The caller waits for
// the vector-memory counter before the barrier that publishes the stage.
__device__ inline void stage_pair(const uint4* gpair, uint4* stage, int tid, int wave) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void*)(gpair + i * 256 + tid),
        (__attribute__((address_space(3))) void*)(stage + i * 256 + wave * 64), 16, 0, 0);
}

// Three workgroups per compute unit: 166 registers, 46 KB of LDS (two 16 KB stages, the list).
// With stages of four tiles (80 KB, two workgroups per compute unit) the kernel was 10 % slower:
// a workgroup goes through its phases (load and norm the keys, sweep, queue, re-evaluate) one
// after the other, and a third resident workgroup fills more of the gaps.
__global__ __launch_bounds__(256, 3) void hash_keys_mfma_kernel(HashMfmaArgs a) {
  __shared__ uint4 sA0[2 * 8 * 64], sA1[2 * 8 * 64];     // two stages of a tile pair: 2 tiles x 8 k-steps each
  __shared__ float sThr[2][4 * 2 * 16];
  __shared__ unsigned long long sList[kListCapLocal];
  __shared__ unsigned sCount;
  __shared__ long long sLimbs[4][kLimbs];

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int unit = blockIdx.y;
  const int kap = lane & 31, hh = lane >> 5;
  const int64_t first = a.first_key, last = a.first_key + a.n_keys;   // [first, last)
  const int64_t cb = first / kBlockKeys + (int64_t)blockIdx.x * 4 + wave;   // my code block
  const bool wave_on = cb * kBlockKeys < last;
  if (tid == 0) sCount = 0;

  const int q0 = a.part_begin[blockIdx.z], nquads = a.part_begin[blockIdx.z + 1];   // quads of this workgroup
  const uint4* gA = reinterpret_cast<const uint4*>(a.afrag);
  const float* gThr = a.thr + (int64_t)unit * a.ntiles * 32;
  stage_pair(gA + (int64_t)q0 * 2 * 1024, sA0, tid, wave);
  if (tid < 128) sThr[q0 & 1][tid] = gThr[q0 * 128 + tid];

  // ---- B operand: my 64 keys, resident in registers for the whole kernel ----
  const uint16_t* Kc = reinterpret_cast<const uint16_t*>(a.Kc);
  const int64_t ubase = (int64_t)(unit / a.n_kv_heads) * a.stride_b + (int64_t)(unit % a.n_kv_heads) * a.stride_h;
  bf16x8 B[2][8];
  int64_t key[2];
  bool key_ok[2];
#pragma unroll
  for (int bt = 0; bt < 2; ++bt) {
    key[bt] = cb * kBlockKeys + bt * 32 + kap;
    key_ok[bt] = wave_on && key[bt] >= first && key[bt] < last;
    const int64_t krow = key_ok[bt] ? key[bt] : first;  // any valid row for masked lanes
    if (a.kv_fp8) {                                      // e4m3 bytes, widened to the same values in bf16
      const uint8_t* row8 = reinterpret_cast<const uint8_t*>(a.Kc) + ubase + krow * a.stride_n + hh * 8;
      uint2 r8[8];
#pragma unroll
      for (int s = 0; s < 8; ++s) r8[s] = *reinterpret_cast<const uint2*>(row8 + s * 16);
#pragma unroll
      for (int s = 0; s < 8; ++s) B[bt][s] = __builtin_bit_cast(bf16x8, fp8x8_to_bf16x8(r8[s].x, r8[s].y));
    } else {
#pragma unroll
      for (int s = 0; s < 8; ++s)
        B[bt][s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(Kc + ubase + krow * a.stride_n + s * 16 + hh * 8));
    }
  }
  // largest column norm of the projector (of every 16 tile rows; requested together with the keys)
  float wmax = 0.f;
  for (int i = lane; i < a.ntiles * 2; i += 64) wmax = fmaxf(wmax, a.rownorm[i]);
  const float munorm = a.mu ? a.munorm[unit] : 0.f;
  float knorm[2];
#pragma unroll
  for (int bt = 0; bt < 2; ++bt) {
    // |k|^2 by v_dot2_f32_bf16 (two exact products per instruction, float32 accumulation: the
    // relative error of the norm, below 1e-5, is inside the margin of kGamma)
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
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
    ss += __shfl_xor(ss, 32);                            // the other half of the row
    knorm[bt] = sqrtf(ss) * 1.00002f;
  }

  const int NW = a.NW;
  uint32_t* blk_codes = a.codes + ((int64_t)unit * a.blocks_cap + cb) * (kBlockKeys * (int64_t)NW);
  wmax = wave_max(wmax);
  if (blockIdx.x == 0 && unit == 0 && blockIdx.z == 0 && tid == 0) *a.wmax_bits = __float_as_uint(wmax);   // statistics only
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  // flagged iff |acc| < bnd = bnd0 + kGamma * largest threshold of the quad, just above the rigorous
  // bound (so "<=" is covered); masked keys are never flagged
  float bnd0[2];
#pragma unroll
  for (int bt = 0; bt < 2; ++bt) bnd0[bt] = key_ok[bt] ? ((kGamma * knorm[bt] + kThresholdSlack * munorm) * (wmax + kNormSlack)) * 1.000001f + 1e-30f : -INFINITY;

  // The four words a quad produces are stored one quad later, so that the wait for the
  // staged fragments at the end of a quad does not also wait for a store just issued.
  uint4 pend = make_uint4(0, 0, 0, 0);
  const int64_t mykey = cb * kBlockKeys + lane;
  const bool store_on = wave_on && mykey >= first && mykey < last;
  // Plane words below the last table group are stored as they are (whole quads as 16 bytes);
  // the planes of the last group go through a bit string that keeps only the real tables.
  const int xs = tail_begin(a.K, a.L), Lt = tail_tables(a.L), NQ = a.NQ;
  BitString tail;
  int tail_x = xs;                                       // next key word the bit string fills
  uint4 tbuf = make_uint4(0, 0, 0, 0);                   // words of the 16-byte group being filled
  // Words leave in increasing order, starting at a group boundary: whole groups of four are
  // stored as 16 bytes, the words of the final 1-3 word group one by one.
  auto emit = [&](int x, uint32_t wv) {
    if ((x >> 2) < (NW >> 2)) {
      switch (x & 3) {
        case 0: tbuf.x = wv; break;
        case 1: tbuf.y = wv; break;
        case 2: tbuf.z = wv; break;
        default:
          tbuf.w = wv;
          if (store_on) *reinterpret_cast<uint4*>(blk_codes + (x >> 2) * 256 + lane * 4) = tbuf;
      }
    } else if (store_on) {
      blk_codes[slot_in_block(NW, x, lane)] = wv;
    }
  };
  auto store_quad = [&](int q) {
    const int x0 = q * 4;
    if (x0 + 4 <= xs) {
      if (store_on) *reinterpret_cast<uint4*>(blk_codes + q * 256 + lane * 4) = pend;
      return;
    }
    const uint32_t w4[4] = {pend.x, pend.y, pend.z, pend.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int x = x0 + i;
      if (x >= NQ) break;
      if (x < xs) {
        emit(x, w4[i]);
      } else {
        uint32_t full;
        if (tail.append(w4[i], Lt, &full)) emit(tail_x++, full);
      }
    }
    if (x0 + 4 >= NQ && tail.nbits > 0) emit(tail_x, (uint32_t)tail.acc);   // last quad: the rest
  };
  // One quad: 4 MFMA tiles (2 pairs = 4 code words) against the 64 keys of this wavefront.  The
  // fragments travel in stages of a pair: pair 2q sits in sA0 when the quad starts (published by
  // the last barrier), pair 2q + 1 goes to sA1 while the first pair is multiplied, and the first
  // pair of the next quad goes to sA0 while the second is.
  auto do_quad = [&](int q) {
    const int cur = q & 1;
    const bool more = q + 1 < nquads;
    float stt = -INFINITY;
    if (q > q0) store_quad(q - 1);
    stage_pair(gA + ((int64_t)q * 2 + 1) * 1024, sA1, tid, wave);
    if (more && tid < 128) stt = gThr[(q + 1) * 128 + tid];

    float bnd[2];
    {
      const float t0 = fabsf(sThr[cur][lane]), t1 = fabsf(sThr[cur][64 + lane]);   // (padding rows: infinite)
      const float most = wave_max(fmaxf(t0 < INFINITY ? t0 : 0.f, t1 < INFINITY ? t1 : 0.f));
      bnd[0] = fmaf(kGamma * 1.000001f, most, bnd0[0]);
      bnd[1] = fmaf(kGamma * 1.000001f, most, bnd0[1]);
    }
    uint32_t wd[2][2];                                   // [pair][key tile] inverted bits, MSB first
    uint32_t fl[2][2];                                   // same bit positions: |acc| <= bound
#pragma unroll
    for (int pair = 0; pair < 2; ++pair) {
      wd[pair][0] = 0; wd[pair][1] = 0;
      fl[pair][0] = 0; fl[pair][1] = 0;
      if (pair == 1) {
        // (every wavefront of the workgroup, working or not, passes here) the second pair has
        // landed in sA1 and everybody is done with sA0: the first pair of the next quad may go there
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (more) stage_pair(gA + ((int64_t)q * 2 + 2) * 1024, sA0, tid, wave);
      }
      if (wave_on) {
        const uint4* sTile = pair ? sA1 : sA0;
#pragma unroll
        for (int tau = 0; tau < 2; ++tau) {
          const int tile = pair * 2 + tau;
          f32x16 c;
#pragma unroll
          for (int v4 = 0; v4 < 4; ++v4) {
            const float4 t4 = *reinterpret_cast<const float4*>(&sThr[cur][(tile * 2 + hh) * 16 + v4 * 4]);
            c[v4 * 4] = t4.x; c[v4 * 4 + 1] = t4.y; c[v4 * 4 + 2] = t4.z; c[v4 * 4 + 3] = t4.w;
          }
          f32x16 acc0 = c, acc1 = c;
          // the A fragment of k-step s + 2 is requested from LDS before the MFMAs of step s are
          // issued (left to itself the compiler emits read, wait, two MFMAs, read, wait, ...)
          bf16x8 ring[3];
          ring[0] = __builtin_bit_cast(bf16x8, sTile[(tau * 8) * 64 + lane]);
          ring[1] = __builtin_bit_cast(bf16x8, sTile[(tau * 8 + 1) * 64 + lane]);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int s = 0; s < 8; ++s) {
            if (s + 2 < 8) ring[(s + 2) % 3] = __builtin_bit_cast(bf16x8, sTile[(tau * 8 + s + 2) * 64 + lane]);
            acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[s % 3], B[0][s], acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[s % 3], B[1][s], acc1, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            // funnel shift: word = (word << 1) | sign(x).  For the code bit x = acc: the sign
            // is exact for ">= 0" because the accumulator starts from +0 or a non-zero
            // threshold, never -0.  For the flag x = |acc| - bound', negative iff |acc| <= bound.
            wd[pair][0] = __builtin_amdgcn_alignbit(wd[pair][0], __float_as_uint(acc0[r]), 31);
            wd[pair][1] = __builtin_amdgcn_alignbit(wd[pair][1], __float_as_uint(acc1[r]), 31);
            fl[pair][0] = __builtin_amdgcn_alignbit(fl[pair][0], __float_as_uint(fabsf(acc0[r]) - bnd[0]), 31);
            fl[pair][1] = __builtin_amdgcn_alignbit(fl[pair][1], __float_as_uint(fabsf(acc1[r]) - bnd[1]), 31);
          }
        }
        wd[pair][0] = ~wd[pair][0];
        wd[pair][1] = ~wd[pair][1];
      }
    }
    if (wave_on) {
      // lanes < 32 hold words x0 (pair 0) and x0+2 (pair 1) of keys kap / 32+kap, lanes >= 32
      // hold x0+1 and x0+3: one half-swap per pair leaves lane l with the words of key l
      const auto s0 = __builtin_amdgcn_permlane32_swap(wd[0][0], wd[0][1], false, false);
      const auto s1 = __builtin_amdgcn_permlane32_swap(wd[1][0], wd[1][1], false, false);
      pend = make_uint4(s0[0], s0[1], s1[0], s1[1]);     // stored at the start of the next quad
      // Projections too close to zero are queued once per quad, after the staged fragments
      // have landed (the list lives in LDS too).
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const int nfl = __popc(fl[0][0]) + __popc(fl[0][1]) + __popc(fl[1][0]) + __popc(fl[1][1]);
      if (__ballot(nfl != 0)) {
        unsigned pos = 0;
        if (nfl) pos = atomicAdd(&sCount, (unsigned)nfl);  // one reservation per lane and quad
        int64_t gpos = -1;
        const unsigned end = pos + (unsigned)nfl;
#pragma unroll
        for (int pair = 0; pair < 2; ++pair) {
          const unsigned xw = (unsigned)(2 * (q * 2 + pair) + hh) << 5;   // code word of this lane half
#pragma unroll
          for (int bt = 0; bt < 2; ++bt) {
            uint32_t f = fl[pair][bt];
            while (f) {
              const int beta = __ffs(f) - 1;
              f &= f - 1;
              const unsigned long long ent =
                  ((unsigned long long)unit << 48) | ((unsigned long long)key[bt] << 16) | (xw + (unsigned)beta);
              if (pos < kListCapLocal) {
                sList[pos] = ent;
              } else {                                   // rare: the workgroup's list is full
                if (gpos < 0) {                          // (one reservation here too: entry by entry all lanes queue for the counter)
                  gpos = atomicAdd(a.list_count, end - pos);
                  if ((uint64_t)gpos + (end - pos) > a.list_cap) *a.overflow = 1;
                }
                if ((uint64_t)gpos < a.list_cap) a.list[gpos] = ent;
                ++gpos;
              }
              ++pos;
            }
          }
        }
      }
    }

    if (more && tid < 128) sThr[cur ^ 1][tid] = stt;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the next stage has landed in LDS
    __syncthreads();
  };
  for (int q = q0; q < nquads; ++q) do_quad(q);
  store_quad(nquads - 1);

  // ---- re-evaluate this workgroup's flagged pairs while its key rows are still in L2 ----
  // The code words were stored above; the wait holds until L2 has them, the barrier makes
  // that true for all four wavefronts, so the atomic patches below land on top of them.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __syncthreads();
  if (lane < kLimbs) sLimbs[wave][lane] = 0;
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
  const unsigned cnt = sCount;
  const unsigned keep = cnt < kListCapLocal ? cnt : kListCapLocal;
  if (tid == 0 && cnt) atomicAdd(a.flagged_total, cnt);    // statistics only
  recheck_pairs<4>(a, sLimbs[wave], keep, (uint64_t)wave * 16, 64, [&](uint64_t i) { return sList[i]; });
}

// The sweep over the projector is split over grid layers while all of them are resident at once: a
// workgroup alone on its compute unit takes 4 us per quad and 15 to 25 us besides (keys from HBM,
// norms, re-evaluation), so a few workgroups leave the chip idle for a whole sweep.  Measured for
// the call, (10,150): 128 workgroups 79 -> 46 us in six parts, 256 workgroups 80 -> 60 us in three;
// 512 workgroups 96 -> 100 us in two, 3072 workgroups 458 -> 556 us: a second round of workgroups costs
// its fixed part.  The quads of the last table group stay together (their words are one bit string).
static int split_sweep(int64_t groups, int nquads, int tail_quad, int* begin) {
  constexpr int64_t kResident = 3 * kNumCU;
  int64_t parts = kResident / groups;
  parts = parts < 1 ? 1 : (parts > kMaxSweepParts ? kMaxSweepParts : parts);
  const int per = (int)((nquads + parts - 1) / parts);
  int n = 0;
  for (int q = 0; q < nquads;) {
    begin[n++] = q;
    q = q + per < nquads && q + per <= tail_quad && n < parts ? q + per : nquads;
  }
  begin[n] = nquads;
  return n;
}

hipError_t launch_hash_keys_mfma(const HashMfmaArgs& a, hipStream_t s) {
  const int proj_blocks = a.ntiles * 2, thr_blocks = (a.ntiles * 32 + 255) / 256;   // 16 tile rows, 256 columns each
  const int64_t prep_blocks = proj_blocks + (int64_t)thr_blocks * a.units + (a.mu ? (a.units + 3) / 4 : 0);
  hipLaunchKernelGGL(prep_hash_keys_kernel, dim3((unsigned)prep_blocks), dim3(256), 0, s, a, proj_blocks, thr_blocks);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t first_blk = a.first_key / kBlockKeys;
  const int64_t last_blk = (a.first_key + a.n_keys - 1) / kBlockKeys;
  const int64_t nblk = last_blk - first_blk + 1;
  const int64_t groups = (nblk + 3) / 4 * a.units;
  HashMfmaArgs b = a;
  const int parts = split_sweep(groups, a.ntiles / 4, tail_begin(a.K, a.L) / 4, b.part_begin);
  hipLaunchKernelGGL(hash_keys_mfma_kernel, dim3((unsigned)((nblk + 3) / 4), (unsigned)a.units, (unsigned)parts), dim3(256), 0, s, b);
  return hipGetLastError();
}

}  // namespace mp
