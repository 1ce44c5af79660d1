// Exact re-evaluation of the projections that the matrix-core key hashing could not decide.
#pragma once
#include "mp_common.h"
#include "exact_dot.h"
#include "device_utils.h"

namespace mp {

// Float64 / exact re-evaluation of listed (key, projection) pairs, for one wavefront: pairs
// first, first + step, ... below count, 64/LPP of them per sweep (step = 64/LPP * wavefronts).
// LPP lanes share a pair (128/LPP elements each, read in 16-byte pieces from the key row and
// from the transposed projector row); their float64 partial sums are combined by shuffles.
// Any summation order is covered by the float64 error bound; what it cannot decide is summed
// exactly.  The bit is then set or cleared in the stored code word.
// List entry: unit (16 bits) | key (32 bits) | code word x (11 bits) | bit of the word (5 bits).
template <int LPP, class GetEntry>
__device__ inline void recheck_pairs(const HashMfmaArgs& a, long long* limb, uint64_t count,
                                     uint64_t first, uint64_t step, GetEntry get) {
  constexpr int kPieces = 16 / LPP;                      // 8-element pieces per lane
  const int lane = threadIdx.x & 63;
  const uint16_t* Kc = reinterpret_cast<const uint16_t*>(a.Kc);
  const uint16_t* WT = reinterpret_cast<const uint16_t*>(a.wt);
  const int grp = lane / LPP, sl = lane % LPP;
  for (uint64_t i0 = first; i0 < count; i0 += step) {
    const uint64_t i = i0 + grp;
    const bool on = i < count;
    const unsigned long long e = get(on ? i : i0);
    const int x = (int)((e >> 5) & 0x7ff), tbit = (int)(e & 31);
    const int j = (32 * (x / a.K) + tbit) * a.K + x % a.K;
    const int64_t unit = (int64_t)(e >> 48);
    const int64_t k = (int64_t)((e >> 16) & 0xffffffffull);
    const int ub = (int)unit / a.n_kv_heads, uh = (int)unit % a.n_kv_heads;
    const int64_t xoff = (int64_t)ub * a.stride_b + (int64_t)uh * a.stride_h + k * a.stride_n;
    // Products of two bf16 values are exact in float32; they are added in float64 (at most 128
    // roundings of 2^-53 of the magnitude sum) and the centering term mu.W_j comes ready-made in
    // float64 from the preparing launch, with the same kind of error on its own magnitude sum:
    // |s - exact| < 2^-45 (sum|k w| + sum|mu w|).  The magnitude sums are float32 upper bounds.
    uint4 kraw[kPieces], wraw[kPieces];
#pragma unroll
    for (int p = 0; p < kPieces; ++p) {
      const int d0 = (p * LPP + sl) * 8;
      if (a.kv_fp8) {                                    // e4m3 bytes, widened to the same values in bf16
        const uint2 r8 = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint8_t*>(a.Kc) + xoff + d0);
        kraw[p] = fp8x8_to_bf16x8(r8.x, r8.y);
      } else {
        kraw[p] = *reinterpret_cast<const uint4*>(Kc + xoff + d0);
      }
      wraw[p] = *reinterpret_cast<const uint4*>(WT + (int64_t)j * kHeadDim + d0);
    }
    double s = 0.0;
    float magf = 0.f;
#pragma unroll
    for (int p = 0; p < kPieces; ++p) {
      const uint32_t ku[4] = {kraw[p].x, kraw[p].y, kraw[p].z, kraw[p].w};
      const uint32_t wu[4] = {wraw[p].x, wraw[p].y, wraw[p].z, wraw[p].w};
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float p0 = __uint_as_float(ku[t] << 16) * __uint_as_float(wu[t] << 16);                 // exact
        const float p1 = __uint_as_float(ku[t] & 0xffff0000u) * __uint_as_float(wu[t] & 0xffff0000u);   // exact
        s += (double)p0;
        s += (double)p1;
        magf += fabsf(p0);
        magf += fabsf(p1);
      }
    }
#pragma unroll
    for (int o = LPP / 2; o > 0; o >>= 1) {
      s += __shfl_xor(s, o);
      magf += __shfl_xor(magf, o);
    }
    double mag = (double)(magf * 1.0001f);
    // float32 products below 2^-126 are rounded to multiples of 2^-149, 1e-42 for 128 of them, or vanish: where
    // all are about that small they are formed again in float64, exactly
    double lost = 1e-42;
    if (__ballot(on && magf < 1e-30f)) {
      double s64 = 0.0, mag64 = 0.0;
#pragma unroll
      for (int p = 0; p < kPieces; ++p) {
        const uint32_t ku[4] = {kraw[p].x, kraw[p].y, kraw[p].z, kraw[p].w};
        const uint32_t wu[4] = {wraw[p].x, wraw[p].y, wraw[p].z, wraw[p].w};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const double p0 = (double)__uint_as_float(ku[t] << 16) * (double)__uint_as_float(wu[t] << 16);
          const double p1 = (double)__uint_as_float(ku[t] & 0xffff0000u) * (double)__uint_as_float(wu[t] & 0xffff0000u);
          s64 += p0;
          s64 += p1;
          mag64 += fabs(p0);
          mag64 += fabs(p1);
        }
      }
#pragma unroll
      for (int o = LPP / 2; o > 0; o >>= 1) {
        s64 += __shfl_xor(s64, o);
        mag64 += __shfl_xor(mag64, o);
      }
      s = s64;
      mag = mag64;
      lost = 0.0;
    }
    if (a.mu) {
      s -= a.thr64[unit * (a.K * a.L) + j];
      mag += (double)a.magmu[unit * (a.K * a.L) + j];
    }
    bool bit = s >= 0.0;
    const bool unsure = on && sl == 0 && mag > 0.0 && fabs(s) <= kF64Slack * mag + lost;
    uint64_t pending = __ballot(unsure);
    while (pending) {
      const int src = __ffsll((unsigned long long)pending) - 1;
      const int64_t sx = ((int64_t)__shfl((int)(xoff >> 32), src) << 32) | (uint32_t)__shfl((int)(xoff & 0xffffffff), src);
      const int sj = __shfl(j, src);
      const int64_t su = ((int64_t)__shfl((int)(unit >> 32), src) << 32) | (uint32_t)__shfl((int)(unit & 0xffffffff), src);
      const float* smu = a.mu ? a.mu + su * kHeadDim : nullptr;
      const bool r = exact_sign_nonneg_wave(
          limb,
          [&](int d) {
            return a.kv_fp8 ? (double)fp8_to_float(reinterpret_cast<const uint8_t*>(a.Kc)[sx + d])
                            : (double)__uint_as_float((uint32_t)Kc[sx + d] << 16);
          },
          [&](int d) { return (double)__uint_as_float((uint32_t)WT[(int64_t)sj * kHeadDim + d] << 16); },
          [&](int d) { return smu ? (double)smu[d] : 0.0; }, smu != nullptr);
      if (lane == src) bit = r;
      pending &= pending - 1;
    }
    if (on && sl == 0) {
      int kword, kbit;
      key_bit_position(a.K, a.L, x, tbit, &kword, &kbit);
      const uint32_t mask = 1u << kbit;
      uint32_t* word = a.codes + (unit * a.blocks_cap + k / kBlockKeys) * (kBlockKeys * (int64_t)a.NW) +
                       slot_in_block(a.NW, kword, (int)(k % kBlockKeys));
      if (bit) atomicOr(word, mask);
      else atomicAnd(word, ~mask);
    }
  }
}

}  // namespace mp
