// Bucketed LSH hash tables in HBM (Algorithm 1: S = Query(HT, q_code); Sec. 4.4 (4)
// "Retrieval"; App. E.2: L tables per key-value head, one key index per key and table).
//
// Per (batch, KV head) and table t the keys are counting-sorted by their K-bit code:
// offsets[t][c] .. offsets[t][c+1] delimits, inside indices[t][], the keys whose code in table
// t is c.  A decode step then touches only the L buckets its query codes select (about
// L*n/2^K indices per head) instead of every key's code: the same sample S as the collision
// scan at a small fraction of its bytes.
//   With the large workspace, three launches: ht_count_kernel (codes per table, 16 bits each, into
//   the workspace; keys per bucket and window of 16384 keys), ht_offsets_kernel (fill levels of the
//   buckets at the start of every window, bucket offsets) and ht_place_kernel (one window of one
//   table per workgroup, sorted in LDS and copied out).  8 KV heads x 98304 keys at (10,150): 105 +
//   14 + 166 us, against 1806 + 455 us of the first version (one workgroup per (unit, 16 tables)
//   walking every window, and a wavefront per piece in the copy).
//   Without it, ht_build_kernel<false>: histogram of the codes of 32 (or fewer) tables in LDS ->
//   offsets; ht_build_kernel<true>: second pass, scatters key indices to their buckets (every 4-byte
//   store reaches HBM on its own).
//   lookup_gather_kernel  : the decode step's retrieval for min_hits 1 or 2: one workgroup per
//       (query head, slice of 16384 keys: one window of the build) reads the L buckets, marks the keys of its slice in
//       LDS bitmaps and gathers and weighs them right away; the few keys appended since the
//       build are found by the collision scan in the same workgroups.
//   table_lookup_kernel, table_lookup_bitmap_kernel: the lookup alone (hit counts per key in
//       LDS byte counters, or seen / seen-twice bitmaps): they emit the same 64-bit ballots
//       (count >= min_hits, key not static) that collision_scan_kernel emits, for the separate
//       gather and merge kernels; used for the count output, other min_hits, and when more
//       keys were appended than the one-launch form takes.
#include "attention_common.h"
#include <hip/hip_ext.h>
#include <type_traits>

namespace mp {

// 64-key blocks per workgroup of the counting lookup: 32 KB of hit counters, one byte per key up
// to 255 tables, two bytes beyond (a key can collide in every table)
template <int BITS> constexpr int kLookupRunBlocks = 512 * 8 / BITS;

// tables handled by one build workgroup: as many histograms of 2^K counters as fit 64 KB of LDS
__host__ __device__ inline int ht_tables_per_pass(int K) {
  const int fit = (64 * 1024) / (4 << K);
  return fit >= 32 ? 32 : (fit >= 16 ? 16 : (fit >= 8 ? 8 : 4));
}

// SCATTER = false: count codes, write offsets.  SCATTER = true: read offsets, place indices.
template <bool SCATTER>
__global__ __launch_bounds__(256) void ht_build_kernel(TableArgs a) {
  extern __shared__ uint32_t hist[];                  // [tables in this pass][2^K]
  const int unit = blockIdx.y;
  const int tpp = ht_tables_per_pass(a.K);
  const int passes = 32 / tpp;
  const int w = blockIdx.x / passes, beta0 = (blockIdx.x % passes) * tpp;
  const int nb = 1 << a.K;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  uint32_t* offs = a.offsets + (int64_t)unit * a.L * (nb + 1);
  uint32_t* idxs = a.indices + (int64_t)unit * a.L * a.n_cap;

  for (int i = tid; i < tpp * nb; i += 256) {
    const int t = 32 * w + beta0 + i / nb;
    hist[i] = (SCATTER && t < a.L) ? offs[(int64_t)t * (nb + 1) + i % nb] : 0u;
  }
  __syncthreads();

  const int64_t nblk = key_blocks(a.n);
  const uint32_t* ucodes = a.kcodes + (int64_t)unit * a.blocks_cap * (kBlockKeys * (int64_t)a.NW);
  // (the lookup reads from the header that the buckets are in no order)
  if (!SCATTER && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) a.header[0] = 0u;
  for (int64_t blk = wave; blk < nblk; blk += 4) {
    const int64_t key = blk * kBlockKeys + lane;
    const uint32_t* blkp = ucodes + blk * (kBlockKeys * (int64_t)a.NW);
    uint32_t kw[12];                                    // (tables take K <= 12)
#pragma unroll
    for (int b = 0; b < 12; ++b) kw[b] = b < a.K ? load_plane_word(blkp, a.NW, a.K, a.L, w * a.K + b, lane) : 0u;
    if (key < a.n) {
      const int here = a.L - 32 * w - beta0 < tpp ? a.L - 32 * w - beta0 : tpp;
#pragma unroll 4
      for (int bb = 0; bb < here; ++bb) {
        const int beta = beta0 + bb;
        uint32_t code = 0;
#pragma unroll
        for (int b = 0; b < 12; ++b) code |= ((kw[b] >> beta) & 1u) << b;
        const uint32_t pos = atomicAdd(&hist[bb * nb + code], 1u);
        if (SCATTER) idxs[(int64_t)(32 * w + beta) * a.n_cap + pos] = (uint32_t)key;
      }
    }
  }
  if (SCATTER) return;
  __syncthreads();
  // exclusive prefix sum of every table's histogram -> offsets (one wavefront per table)
  for (int bb = wave; bb < tpp; bb += 4) {
    const int t = 32 * w + beta0 + bb;
    if (t >= a.L) break;
    const int per = (nb + 63) / 64;                   // consecutive bins per lane
    uint32_t local = 0;
    for (int j = 0; j < per; ++j) {
      const int c = lane * per + j;
      if (c < nb) local += hist[bb * nb + c];
    }
    uint32_t incl = local;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t v = __shfl_up(incl, o);
      if (lane >= o) incl += v;
    }
    uint32_t run = incl - local;
    for (int j = 0; j < per; ++j) {
      const int c = lane * per + j;
      if (c < nb) {
        offs[(int64_t)t * (nb + 1) + c] = run;
        run += hist[bb * nb + c];
      }
    }
    if (lane == 63) offs[(int64_t)t * (nb + 1) + nb] = incl;
  }
}

// ---- the build with a workspace: count, scan, place ----
//
// Sixteen bit planes of sixteen tables -> sixteen codes.  p[i] holds plane i in its low and plane
// i + 8 in its high half (bit j = table j); on return p[j] holds the code of table j in its low and
// that of table j + 8 in its high half (a 16 x 16 bit transpose: 8 byte permutes and 12 swaps of
// four operations, 3.5 per code, against 2 K for taking the bits out one by one).
template <int D, uint32_t M>
__device__ inline void swap_bits(uint32_t (&p)[8]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = q / D * 2 * D + q % D;                // the words without bit D of their number
    const uint32_t x = p[i], y = p[i + D];
    p[i] = (x & M) | ((y << D) & ~M);
    p[i + D] = ((x >> D) & M) | (y & ~M);
  }
}
__device__ inline void planes_to_codes(uint32_t (&p)[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) p[i] = __builtin_amdgcn_perm(p[i], p[i], 0x07050604u);   // bytes 3, 1, 2, 0
  swap_bits<4, 0x0f0f0f0fu>(p);
  swap_bits<2, 0x33333333u>(p);
  swap_bits<1, 0x55555555u>(p);
}

// Workgroups of the count and place kernels come as blockIdx.y * gridDim.x + blockIdx.x with gridDim.x
// a multiple of eight, so that id % 8 is the XCD a workgroup runs on: item id / 8 of "lane" id % 8.
// (fewer than 2^31 workgroups: their output, 64 KB each, has to fit the memory of the card)
__device__ inline uint32_t linear_workgroup() { return blockIdx.y * gridDim.x + blockIdx.x; }
static dim3 linear_grid(int64_t total) {                // total: a multiple of eight
  const int64_t most = (int64_t)1 << 21;                // gridDim.x * 1024 threads stays below 2^32
  if (total <= most) return dim3((unsigned)total);
  return dim3((unsigned)most, (unsigned)((total + most - 1) / most));
}

// tables a count workgroup handles: u32 histograms of 2^K counters in at most 64 KB of LDS
constexpr int ht_count_tables(int K) { return K <= 10 ? 16 : (K == 11 ? 8 : 4); }

// The key blocks of a window, two neighbouring ones per wavefront at a time, for the tables t0 + j and
// t0 + 8 + j, j0 <= j < j0 + T/2, t0 = 32 w + 16 half.  TAIL: w is the last table group (its planes
// are one bit string).
// What it waits for is the address unit, one access per cycle and quad of lanes that leaves a 64-byte
// line: so a lane takes two neighbouring keys (lanes 0-31 one block, 32-63 the next: the store of a
// table is 256 contiguous bytes) and reads its words in the layout's 16-byte groups.
template <int K, int T, bool TAIL>
__device__ inline void ht_count_blocks(const TableArgs& a, uint32_t* hist, int unit, int win, int w, int half, int j0) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  constexpr int nb = 1 << K;
  constexpr int kGroups = K == 1 ? 1 : (K + 6) / 4;     // 16-byte groups that K words from anywhere touch, at most
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t0 = 32 * w + 16 * half;
  const int64_t nblk = key_blocks(a.n);
  constexpr int64_t kWinBlocks = kBuildWindow / kBlockKeys;
  const int64_t blk_end = nblk < (win + 1) * kWinBlocks ? nblk : (win + 1) * kWinBlocks;
  const uint32_t* ucodes = a.kcodes + (int64_t)unit * a.blocks_cap * (kBlockKeys * (int64_t)a.NW);
  const int64_t row = a.blocks_cap * kBlockKeys;        // codes16: rows of whole blocks
  uint16_t* out16 = a.codes16 + ((int64_t)unit * a.L + t0 + j0) * row + 2 * lane;
  const uint32_t pick = half ? 0x07060302u : 0x05040100u;  // this half of planes i (bytes 0-3) and i + 8 (4-7)
  const int key0 = 2 * (lane & 31);                     // keys key0 and key0 + 1 of the lane's block
  const int full = a.NW >> 2, rem = a.NW & 3;
  const int g0 = (w * K) >> 2;                          // first 16-byte group of the planes
  for (int64_t blk = win * kWinBlocks + 2 * wave; blk < blk_end; blk += 32) {
    const bool on = blk + (lane >> 5) < blk_end;        // (the second block may not exist)
    const uint32_t* blkp = ucodes + (blk + (on ? lane >> 5 : 0)) * (kBlockKeys * (int64_t)a.NW);
    // The groups of four words that hold the K planes of the lane's two keys (32 bytes apiece); the
    // words of an incomplete last group come one by one.
    uint32_t raw[2][4 * kGroups];
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      if (g0 + g < full) {
        const u32x4* src = reinterpret_cast<const u32x4*>(blkp + (g0 + g) * 256) + key0;
        const u32x4 v0 = src[0], v1 = src[1];
        raw[0][4 * g] = v0.x; raw[0][4 * g + 1] = v0.y; raw[0][4 * g + 2] = v0.z; raw[0][4 * g + 3] = v0.w;
        raw[1][4 * g] = v1.x; raw[1][4 * g + 1] = v1.y; raw[1][4 * g + 2] = v1.z; raw[1][4 * g + 3] = v1.w;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          raw[0][4 * g + i] = 0u; raw[1][4 * g + i] = 0u;
          if (g0 + g == full && i < rem) {
            raw[0][4 * g + i] = blkp[full * 256 + key0 * rem + i];
            raw[1][4 * g + i] = blkp[full * 256 + (key0 + 1) * rem + i];
          }
        }
      }
    }
    // the first plane's word to the front (register numbers are constants: the words are moved)
    auto drop = [&](int n) {                             // n is 1 or 2
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int i = 0; i < 4 * kGroups; ++i) {
          const int from = n == 1 ? i + 1 : i + 2;
          raw[e][i] = from < 4 * kGroups ? raw[e][from] : 0u;
        }
    };
    const int skip = (w * K) & 3;
    if (skip & 1) drop(1);
    if (skip & 2) drop(2);
    if constexpr (TAIL) {
      // plane i starts at bit i Lt of the string: whenever that crosses into the next word the words
      // move up by one
      int Lt = tail_tables(a.L);
      asm volatile("" : "+s"(Lt));
      uint32_t pl[2][K];
#pragma unroll
      for (int i = 0; i < K; ++i) {
        if (i > 0 && ((i * Lt) >> 5) != (((i - 1) * Lt) >> 5)) drop(1);
#pragma unroll
        for (int e = 0; e < 2; ++e) pl[e][i] = __builtin_amdgcn_alignbit(raw[e][1], raw[e][0], (uint32_t)(i * Lt) & 31u);
      }
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int i = 0; i < K; ++i) raw[e][i] = pl[e][i];
    }
    uint32_t pk[2][8];
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        // (plane b as bit b + 2: the codes come out times four, byte offsets of the counters)
        pk[e][i] = __builtin_amdgcn_perm(i + 6 < K ? raw[e][(i + 6) % (4 * kGroups)] : 0u, i >= 2 && i - 2 < K ? raw[e][(i + 4 * kGroups - 2) % (4 * kGroups)] : 0u, pick);
    planes_to_codes(pk[0]);
    planes_to_codes(pk[1]);
    if constexpr (T < 16) {                              // the T/2 words of this workgroup to the front
#pragma unroll
      for (int q = 8 - T / 2; q > 0; q -= T / 2) {
        if (j0 == q) {
#pragma unroll
          for (int j = 0; j < T / 2; ++j) { pk[0][j] = pk[0][q + j]; pk[1][j] = pk[1][q + j]; }
        }
      }
    }
    const int64_t key = (blk + (lane >> 5)) * kBlockKeys + key0;
    const bool real0 = key < a.n, real1 = key + 1 < a.n;  // (a.n ends inside the last block)
    uint16_t* o = out16 + blk * kBlockKeys;
    int left = a.L - (t0 + j0);                          // tables from the first of this workgroup on
    asm volatile("" : "+s"(left));
#pragma unroll
    for (int j = 0; j < T / 2; ++j) {
      const uint32_t c0 = pk[0][j], c1 = pk[1][j];
      if (j < left) {
        char* h = reinterpret_cast<char*>(hist + 2 * j * nb);
        if (real0) atomicAdd(reinterpret_cast<uint32_t*>(h + (c0 & 0xffffu)), 1u);
        if (real1) atomicAdd(reinterpret_cast<uint32_t*>(h + (c1 & 0xffffu)), 1u);
        if (on) *reinterpret_cast<uint32_t*>(o) = __builtin_amdgcn_perm(c1, c0, 0x05040100u);
      }
      if (j + 8 < left) {
        char* h = reinterpret_cast<char*>(hist + (2 * j + 1) * nb);
        if (real0) atomicAdd(reinterpret_cast<uint32_t*>(h + (c0 >> 16)), 1u);
        if (real1) atomicAdd(reinterpret_cast<uint32_t*>(h + (c1 >> 16)), 1u);
        if (on) *reinterpret_cast<uint32_t*>(o + 8 * row) = __builtin_amdgcn_perm(c1, c0, 0x07060302u);
      }
      o += row;
    }
  }
}

// Counts the keys of one window of 16384 per bucket for T tables, and writes every key's code of
// those tables (16 bits, table-major).  One workgroup = (unit, window, T tables): the windows are
// counted independently, so that the chip is full at one sequence (8 KV heads x 98304 keys at
// (10,150): 480 workgroups, two per compute unit; walking the windows one after the other in one
// workgroup per (unit, 16 tables), which the first version did to carry the fill levels along,
// kept 80 of 256 compute units busy).  All groups of tables of a window run on one XCD: they read the
// same code blocks, which then come from HBM once.  105 us there, 384 MB read and written (79 us at the
// rate of a large copy): what it waits for changes from address unit to LDS atomics to vector unit
// in the course of a pair of blocks, and 32 wavefronts per compute unit overlap them in part.
template <int K>
__global__ __launch_bounds__(1024, 8) void ht_count_kernel(TableArgs a) {
  extern __shared__ uint32_t hist[];                    // [T][2^K]
  constexpr int T = ht_count_tables(K), nb = 1 << K;
  constexpr int kParts = 16 / T;                        // workgroups per half group of 16 tables
  const uint32_t groups = 2 * kParts * table_words(a.L);
  const uint32_t id = linear_workgroup();
  const uint32_t vw = (id >> 3) / groups * 8 + (id & 7);   // (unit, window)
  const int grp = (int)((id >> 3) % groups);
  if (vw >= (uint32_t)a.units * (uint32_t)a.windows) return;
  const int unit = (int)(vw / (uint32_t)a.windows), win = (int)(vw % (uint32_t)a.windows);
  const int w = grp / (2 * kParts), half = (grp / kParts) & 1, j0 = (grp % kParts) * (T / 2);
  const int t0 = 32 * w + 16 * half;                    // tables t0 + j and t0 + 8 + j, j0 <= j < j0 + T/2
  if (t0 + j0 >= a.L) return;
  const int tid = threadIdx.x;
  for (int i = tid; i < T * nb; i += 1024) hist[i] = 0u;
  __syncthreads();
  if (w == table_words(a.L) - 1) ht_count_blocks<K, T, true>(a, hist, unit, win, w, half, j0);
  else ht_count_blocks<K, T, false>(a, hist, unit, win, w, half, j0);
  __syncthreads();
  for (int i = tid; i < T * nb; i += 1024) {
    const int li = i / nb, t = t0 + j0 + (li >> 1) + 8 * (li & 1);
    if (t < a.L) a.wincum[(((int64_t)unit * a.L + t) * a.windows + win) * nb + i % nb] = hist[i];
  }
}

// Per (unit, table): turns the counts of the windows into fill levels (keys of the bucket in earlier
// windows), and their totals into bucket offsets.  A few per cent of the build.
__global__ __launch_bounds__(256) void ht_offsets_kernel(TableArgs a) {
  extern __shared__ uint32_t tot[];                     // [2^K]
  __shared__ uint32_t wsum[4];
  const int t = blockIdx.x, unit = blockIdx.y;
  const int nb = 1 << a.K;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  // (the lookup reads from the header that the buckets are ordered by window)
  if (t == 0 && unit == 0 && tid == 0) a.header[0] = (uint32_t)a.windows;
  uint32_t* cum = a.wincum + ((int64_t)unit * a.L + t) * a.windows * nb;
  for (int c = tid; c < nb; c += 256) {
    // (eight windows are read before any is written back: the compiler cannot know that the places differ)
    uint32_t run = 0;
    for (int w0 = 0; w0 < a.windows; w0 += 8) {
      uint32_t n_c[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) n_c[i] = w0 + i < a.windows ? cum[(int64_t)(w0 + i) * nb + c] : 0u;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (w0 + i < a.windows) cum[(int64_t)(w0 + i) * nb + c] = run;
        run += n_c[i];
      }
    }
    tot[c] = run;
  }
  __syncthreads();
  const int per = nb / 256 > 0 ? nb / 256 : 1;          // thread = run of consecutive buckets
  uint32_t local = 0;
  for (int j = 0; j < per; ++j)
    if (tid * per + j < nb) local += tot[tid * per + j];
  uint32_t incl = local;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t v = __shfl_up(incl, o);
    if (lane >= o) incl += v;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  uint32_t at = incl - local;
  for (int v = 0; v < wave; ++v) at += wsum[v];
  uint32_t* offs = a.offsets + ((int64_t)unit * a.L + t) * (nb + 1);
  for (int j = 0; j < per; ++j) {
    const int c = tid * per + j;
    if (c < nb) {
      offs[c] = at;
      at += tot[c];
      if (c == nb - 1) offs[nb] = at;
    }
  }
}

// Places the keys of one window into the buckets of one table.  The window is counting-sorted
// by bucket in LDS (its bucket sizes are the differences of the fill levels), every entry with its
// bucket beside it, so that the sorted window is then copied out by consecutive lanes: entry i of
// bucket c goes to i + (first place of the bucket's piece in the index array - its place in the
// sorted window).  Pieces are about 16 entries, so a wavefront store covers four or five of them; the
// first version gave a wavefront one piece at a time (a quarter of the lanes at work, 455 us at 8 KV
// heads x 98304 keys, (10,150); then 176 to 182 us with 24 vector
// instructions per key; now 158 to 166 us, 18 per key and no masks in whole windows, for 790 MB read and written, 4.8 TB/s,
// about the rate of a large copy).  Two workgroups per compute unit (72 KB of LDS each at K = 10); the windows of a
// table run on one XCD, whose L2 joins the pieces of neighbouring windows into whole lines.
__global__ __launch_bounds__(1024, 8) void ht_place_kernel(TableArgs a) {
  extern __shared__ uint32_t lds[];
  const int nb = 1 << a.K;
  uint32_t* cursor = lds;                                              // [2^K] byte offset in `sorted` of the next free slot of the bucket's piece
  uint32_t* delta = lds + nb;                                          // [2^K] place in the index array - place in `sorted`
  uint32_t* sorted = delta + nb;                                       // [kBuildWindow] bucket << 16 | key inside the window
  static_assert(kBuildWindow == 1 << 14, "above 14 bits of key and two of zero an entry >> 14 is four times its bucket");
  __shared__ uint32_t wsum[16];
  const uint32_t id = linear_workgroup();
  const int win = (int)((id >> 3) % (uint32_t)a.windows);
  const int64_t ut = (id >> 3) / (uint32_t)a.windows * 8 + (id & 7);   // (unit, table)
  if (ut >= (int64_t)a.units * a.L) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t* offs = a.offsets + ut * (nb + 1);
  const uint32_t* cum = a.wincum + (ut * a.windows + win) * nb;
  const bool last = win == a.windows - 1;
  const uint16_t* codes = a.codes16 + ut * (a.blocks_cap * kBlockKeys);
  const int64_t k0 = (int64_t)win * kBuildWindow;
  const int m = (int)(k0 + kBuildWindow < a.n ? kBuildWindow : a.n - k0);   // keys of the window
  // the codes of this thread's keys (rows hold whole blocks: pieces of eight that begin below n end inside)
  uint4 raw[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int kb = (h * 1024 + tid) * 8;
    raw[h] = kb < m ? *reinterpret_cast<const uint4*>(codes + k0 + kb) : make_uint4(0, 0, 0, 0);
  }
  // bucket sizes of the window and their exclusive prefix sums (thread = run of consecutive buckets)
  const int per = nb / 1024 > 0 ? nb / 1024 : 1;                       // nb is a power of two
  uint32_t n_c[4], base_c[4], run = 0;                                 // K <= 12: at most four buckets
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c = tid * per + j;
    n_c[j] = 0; base_c[j] = 0;
    if (j < per && c < nb) {
      const uint32_t before = cum[c], first = offs[c];
      const uint32_t after = last ? offs[c + 1] - first : cum[nb + c];
      n_c[j] = after - before;
      base_c[j] = first + before;
      run += n_c[j];
    }
  }
  uint32_t incl = run;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t v = __shfl_up(incl, o);
    if (lane >= o) incl += v;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  uint32_t at = incl - run;
  for (int v = 0; v < wave; ++v) at += wsum[v];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c = tid * per + j;
    if (j < per && c < nb) {
      cursor[c] = 4 * at;
      delta[c] = base_c[j] - at;
      at += n_c[j];
    }
  }
  __syncthreads();
  // counting sort of the window's keys, and the sorted window copied out; whole windows need no masks
  uint32_t* idxs = a.indices + ut * a.n_cap;
  auto place = [&](auto whole) {
    constexpr bool kWhole = decltype(whole)::value;
    char* cur = reinterpret_cast<char*>(cursor);
    char* out = reinterpret_cast<char*>(sorted);
    const char* del = reinterpret_cast<const char*>(delta);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int kb = (h * 1024 + tid) * 8;
      const uint32_t u[4] = {raw[h].x, raw[h].y, raw[h].z, raw[h].w};
      uint32_t code4[8], pos4[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        code4[e] = (e & 1) ? u[e >> 1] >> 16 : u[e >> 1] & 0xffffu;
        if (kWhole || kb + e < m) pos4[e] = atomicAdd(reinterpret_cast<uint32_t*>(cur + code4[e]), 4u);
      }
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (kWhole || kb + e < m) *reinterpret_cast<uint32_t*>(out + pos4[e]) = (code4[e] << 14) | (uint32_t)(kb + e);
    }
    __syncthreads();
    auto copy = [&](int i) {
      const uint32_t e = sorted[i];
      idxs[*reinterpret_cast<const uint32_t*>(del + (e >> 14)) + (uint32_t)i] = (uint32_t)k0 | (e & (kBuildWindow - 1));
    };
    if constexpr (kWhole) {
#pragma unroll
      for (int i = 0; i < kBuildWindow / 1024; ++i) copy(i * 1024 + tid);
    } else {
#pragma unroll 4
      for (int i = tid; i < m; i += 1024) copy(i);
    }
  };
  if (m == kBuildWindow) place(std::true_type{});
  else place(std::false_type{});
}

template <int BITS>
__global__ __launch_bounds__(1024) void table_lookup_kernel(AttnArgs a, TableArgs tb) {
  constexpr int kLookupRunKeys = kLookupRunBlocks<BITS> * kBlockKeys;
  constexpr int kPerWord = 32 / BITS;                  // counters per 32-bit LDS word
  constexpr uint32_t kCntMask = (1u << BITS) - 1u;
  __shared__ uint32_t counters[kLookupRunKeys / kPerWord];
  __shared__ uint32_t bstart[512], blen[512];
  const Ctx cx = resolve_context(a);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int run = blockIdx.x;
  const int64_t bh = blockIdx.y;
  const int G = a.Hq / a.Hkv;
  const int64_t unit = (bh / a.Hq) * a.Hkv + (bh % a.Hq) / G;
  const int nb = 1 << a.K;
  const uint32_t* offs = tb.offsets + unit * a.L * (nb + 1);
  const uint32_t* idxs = tb.indices + unit * a.L * tb.n_cap;
  const int64_t key0 = (int64_t)run * kLookupRunKeys;

  __shared__ uint32_t qs[256];
  for (int i = tid; i < kLookupRunKeys / kPerWord; i += 1024) counters[i] = 0u;
  if (tid < a.NQ) qs[tid] = a.qcodes[bh * a.NQ + tid];   // one round trip for the query's words
  __syncthreads();
  // bucket of every table: the query's K-bit code of table t selects offsets[t][code..code+1]
  for (int t = tid; t < a.L; t += 1024) {
    const uint32_t* qw = qs + (t >> 5) * a.K;
    uint32_t code = 0;
    for (int b = 0; b < a.K; ++b) code |= ((qw[b] >> (t & 31)) & 1u) << b;
    const uint32_t s0 = offs[(int64_t)t * (nb + 1) + code], s1 = offs[(int64_t)t * (nb + 1) + code + 1];
    bstart[t] = s0;
    blen[t] = s1 - s0;
  }
  __syncthreads();

  // wavefront v reads tables v, v+16, ...: up to 128 entries of each bucket are requested
  // before any is used; longer buckets are finished in a loop
  constexpr int kMaxB = 32;                           // L <= 512 tables over 16 wavefronts
  uint32_t e0[kMaxB], e1[kMaxB];
  const uint32_t ukey0 = (uint32_t)key0;
  const int nbk = (a.L - wave + 15) >> 4;             // buckets of this wavefront
#pragma unroll
  for (int k = 0; k < kMaxB; ++k) {
    e0[k] = 0xffffffffu; e1[k] = 0xffffffffu;
    if (k < nbk) {
      const int t = wave + 16 * k;
      const uint32_t len = blen[t];
      const uint32_t* p = idxs + (int64_t)t * tb.n_cap + bstart[t];
      if ((uint32_t)lane < len) e0[k] = p[lane];
      if ((uint32_t)lane + 64 < len) e1[k] = p[lane + 64];
    }
  }
  // a key outside this run (or the "no entry" marker) wraps to a value >= kLookupRunKeys
  auto count_key = [&](uint32_t key) {
    const uint32_t rel = key - ukey0;
    if (rel < (uint32_t)kLookupRunKeys) atomicAdd(&counters[rel / kPerWord], 1u << (BITS * (rel % kPerWord)));
  };
#pragma unroll
  for (int k = 0; k < kMaxB; ++k) {
    if (k < nbk) {
      count_key(e0[k]);
      count_key(e1[k]);
      const int t = wave + 16 * k;
      if (blen[t] > 128) {
        const uint32_t* p = idxs + (int64_t)t * tb.n_cap + bstart[t];
        for (uint32_t j = 128 + lane; j < blen[t]; j += 64) count_key(p[j]);
      }
    }
  }
  __syncthreads();

  // ballots of the blocks the tables cover: a thread takes 32 consecutive keys (half a block)
  const int64_t nblk = key_blocks(cx.n);
  for (int part = tid; part < kLookupRunKeys / 32; part += 1024) {
    const int64_t kfirst = key0 + (int64_t)part * 32;
    if (kfirst >= key_blocks(tb.n) * kBlockKeys) break;
    // positions of this thread's keys that are real and outside the static set
    const int64_t lo = (a.n_sink > kfirst ? a.n_sink : kfirst) - kfirst;
    const int64_t hi_key = cx.n - a.n_local < cx.n ? cx.n - a.n_local : cx.n;
    const int64_t hi = (hi_key < kfirst + 32 ? hi_key : kfirst + 32) - kfirst;
    uint32_t elig = 0;
    if (hi > lo) elig = (hi - lo >= 32 ? 0xffffffffu : ((1u << (hi - lo)) - 1u)) << lo;
    auto count_of = [&](int j) { return (int)((counters[(part * 32 + j) / kPerWord] >> (BITS * (j % kPerWord))) & kCntMask); };
    uint32_t bits = 0;
#pragma unroll
    for (int j = 0; j < 32; ++j) bits |= (uint32_t)(a.tau <= 0 || count_of(j) >= a.tau) << j;
    bits &= elig;
    reinterpret_cast<uint32_t*>(a.masks)[(bh * nblk) * 2 + kfirst / 32] = bits;
    if (a.dbg_counts || a.dbg_cand) {                 // debug outputs only
      for (int j = 0; j < 32; ++j) {
        const int64_t i = kfirst + j;
        if (a.dbg_counts && i < cx.n) a.dbg_counts[bh * a.dbg_stride + i] = (uint16_t)count_of(j);
        if (a.dbg_cand && ((bits >> j) & 1u)) {
          const int pos = atomicAdd(&a.dbg_ncand[bh], 1);
          if (pos < a.dbg_cand_cap) a.dbg_cand[bh * a.dbg_cand_cap + pos] = (int32_t)i;
        }
      }
    }
  }
}

// Production form of the lookup for min_hits 1 or 2 (no count output): one workgroup per query
// head marks every key it meets in a "seen" bitmap of the whole indexed range and, when it was
// already marked, in a "seen twice" bitmap (both in LDS, a bit per key); the ballots are those
// bitmaps.  No bucket is read more than once per head, whatever the context length.
// Bound by latency and instruction count: two workgroups per compute unit (64 registers) so that 512 heads are
// one round; the entries of kChunk buckets requested at once, up to 64 kEntries of each (at 131072 keys and
// K = 10 a bucket holds 128 on average, and every second one made a wavefront wait for the rest of it when the
// first request took 128); what a wavefront knows of its buckets sits in its lanes, and the slots of a chunk
// that have no bucket are left by a branch (masked off instead, 11 buckets in slots of 16 took 9.8 us, with the
// branch 7.2 in slots of 8).  Kernel, us: all buckets of a wavefront at once, 128 entries each, 96 registers |
// four at a time, 192 entries, descriptors in LDS | this: 256 heads x 4096 keys, (10,170) 8.7 | 11.0 | 7.2;
// 256 x 60000, (10,170) 10.2 | 11.2 | 10.1; 256 x 20000, (10,512) 16.1 | 23.4 | 14.2; 512 x 100000, (10,150)
// 24.8 | 18.0 | 16.4.
template <int kChunk, int kEntries>
__global__ __launch_bounds__(1024, 8) void table_lookup_bitmap_kernel(AttnArgs a, TableArgs tb) {
  extern __shared__ uint32_t bitmap[];                  // seen[nw], twice[nw]
  __shared__ uint32_t bstart[512], blen[512];
  __shared__ uint32_t qs[256];
  const Ctx cx = resolve_context(a);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int64_t bh = blockIdx.x;
  const int G = a.Hq / a.Hkv;
  const int64_t unit = (bh / a.Hq) * a.Hkv + (bh % a.Hq) / G;
  const int nb = 1 << a.K;
  const uint32_t* offs = tb.offsets + unit * a.L * (nb + 1);
  const uint32_t* idxs = tb.indices + unit * a.L * tb.n_cap;
  const int nw = (int)key_blocks(tb.n) * 2;             // 32-key words of the indexed range
  uint32_t* seen = bitmap;
  uint32_t* twice = bitmap + nw;
  for (int i = tid; i < 2 * nw; i += 1024) bitmap[i] = 0u;
  if (tid < a.NQ) qs[tid] = a.qcodes[bh * a.NQ + tid];
  __syncthreads();
  for (int t = tid; t < a.L; t += 1024) {
    const uint32_t* qw = qs + (t >> 5) * a.K;
    uint32_t code = 0;
    for (int b = 0; b < a.K; ++b) code |= ((qw[b] >> (t & 31)) & 1u) << b;
    const uint32_t s0 = offs[(int64_t)t * (nb + 1) + code], s1 = offs[(int64_t)t * (nb + 1) + code + 1];
    bstart[t] = s0;
    blen[t] = s1 - s0;
  }
  __syncthreads();
  // wavefront v reads tables v, v+16, ..., kChunk at a time: up to 64 kEntries entries of each bucket
  // are requested before any is used, and the first atomics (was the key seen before?) are issued
  // together; longer buckets are finished in a loop
  const int nbk = (a.L - wave + 15) >> 4;                // at most 32: lane k holds what is known of bucket k
  const uint32_t my_start = lane < nbk ? bstart[wave + 16 * lane] : 0u, my_len = lane < nbk ? blen[wave + 16 * lane] : 0u;
  for (int k0 = 0; k0 < nbk; k0 += kChunk) {
    uint32_t e[kChunk][kEntries], before[kChunk][kEntries];
    const int here = nbk - k0;                           // (wave-uniform)
#pragma unroll
    for (int k = 0; k < kChunk; ++k) {
#pragma unroll
      for (int j = 0; j < kEntries; ++j) { e[k][j] = 0xffffffffu; before[k][j] = 0u; }
    }
#pragma unroll
    for (int k = 0; k < kChunk; ++k) {
      if (k >= here) break;
      const uint32_t len = __builtin_amdgcn_readlane(my_len, k0 + k);
      const uint32_t* p = idxs + (int64_t)(wave + 16 * (k0 + k)) * tb.n_cap + __builtin_amdgcn_readlane(my_start, k0 + k);
#pragma unroll
      for (int j = 0; j < kEntries; ++j)
        if ((uint32_t)(lane + 64 * j) < len) e[k][j] = p[lane + 64 * j];
    }
#pragma unroll
    for (int k = 0; k < kChunk; ++k) {
      if (k >= here) break;
#pragma unroll
      for (int j = 0; j < kEntries; ++j)
        if (e[k][j] != 0xffffffffu) before[k][j] = atomicOr(&seen[e[k][j] >> 5], 1u << (e[k][j] & 31));
    }
#pragma unroll
    for (int k = 0; k < kChunk; ++k) {
      if (k >= here) break;
#pragma unroll
      for (int j = 0; j < kEntries; ++j)
        if (before[k][j] >> (e[k][j] & 31) & 1u) atomicOr(&twice[e[k][j] >> 5], 1u << (e[k][j] & 31));
    }
  }
  // (what is longer than the first request)
  for (uint64_t f = __ballot(my_len > 64 * kEntries); f; f &= f - 1) {
    const int k = __ffsll((unsigned long long)f) - 1;
    const uint32_t len = __builtin_amdgcn_readlane(my_len, k);
    const uint32_t* p = idxs + (int64_t)(wave + 16 * k) * tb.n_cap + __builtin_amdgcn_readlane(my_start, k);
    for (uint32_t j = 64 * kEntries + lane; j < len; j += 64) {
      const uint32_t key = p[j], bit = 1u << (key & 31);
      if (atomicOr(&seen[key >> 5], bit) & bit) atomicOr(&twice[key >> 5], bit);
    }
  }
  __syncthreads();
  // ballots of the indexed range, 32 keys per word, static keys and keys beyond n masked out
  const int64_t nblk = key_blocks(cx.n);
  const uint32_t* hit = a.tau >= 2 ? twice : seen;
  uint32_t* mout = reinterpret_cast<uint32_t*>(a.masks) + bh * nblk * 2;
  const int64_t hi_key = cx.n - a.n_local < cx.n ? cx.n - a.n_local : cx.n;
  for (int i = tid; i < nw; i += 1024) {
    const int64_t kfirst = (int64_t)i * 32;
    const int64_t lo = (a.n_sink > kfirst ? a.n_sink : kfirst) - kfirst;
    const int64_t hi = (hi_key < kfirst + 32 ? hi_key : kfirst + 32) - kfirst;
    uint32_t elig = 0;
    if (hi > lo) elig = (hi - lo >= 32 ? 0xffffffffu : ((1u << (hi - lo)) - 1u)) << lo;
    const uint32_t bits = hit[i] & elig;
    mout[i] = bits;
    if (a.dbg_cand) {                                    // debug output only
      for (uint32_t f = bits; f; f &= f - 1) {
        const int pos = atomicAdd(&a.dbg_ncand[bh], 1);
        if (pos < a.dbg_cand_cap) a.dbg_cand[bh * a.dbg_cand_cap + pos] = (int32_t)(kfirst + __ffs(f) - 1);
      }
    }
  }
}

hipError_t launch_build_tables(const TableArgs& t, hipStream_t s) {
  if (t.units <= 0 || t.L <= 0) return hipSuccess;
  hipError_t e;
  if (t.codes16) {
    // enough workspace for every key's code per table: buckets ordered by window
    const int T = ht_count_tables(t.K);
    const int64_t groups = (int64_t)(32 / T) * table_words(t.L);
    const dim3 cgrid = linear_grid(((int64_t)t.units * t.windows + 7) / 8 * 8 * groups);
    const size_t count_lds = (size_t)T * (4u << t.K);
    switch (t.K) {
#define MP_COUNT(KT) case KT: hipLaunchKernelGGL(ht_count_kernel<KT>, cgrid, dim3(1024), count_lds, s, t); break;
      MP_COUNT(1) MP_COUNT(2) MP_COUNT(3) MP_COUNT(4) MP_COUNT(5) MP_COUNT(6)
      MP_COUNT(7) MP_COUNT(8) MP_COUNT(9) MP_COUNT(10) MP_COUNT(11)
      default: hipLaunchKernelGGL(ht_count_kernel<12>, cgrid, dim3(1024), count_lds, s, t);   // (tables take K <= 12)
#undef MP_COUNT
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(ht_offsets_kernel, dim3((unsigned)t.L, (unsigned)t.units), dim3(256), (size_t)4 << t.K, s, t);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const dim3 pgrid = linear_grid(((int64_t)t.units * t.L + 7) / 8 * 8 * t.windows);
    const size_t place_lds = ((size_t)8 << t.K) + (size_t)kBuildWindow * sizeof(uint32_t);   // <= 96 KB at K = 12
    hipLaunchKernelGGL(ht_place_kernel, pgrid, dim3(1024), place_lds, s, t);
    return hipGetLastError();
  }
  const int tpp = ht_tables_per_pass(t.K);
  const int passes = 32 / tpp;
  const size_t lds = (size_t)tpp * (4u << t.K);
  const dim3 grid((unsigned)(table_words(t.L) * passes), (unsigned)t.units);
  hipLaunchKernelGGL(ht_build_kernel<false>, grid, dim3(256), lds, s, t);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(ht_build_kernel<true>, grid, dim3(256), lds, s, t);
  return hipGetLastError();
}

// Lookup and gather in one launch for min_hits 1 or 2: a workgroup of 16 wavefronts per (query
// head, slice of kLgSliceBlocks key blocks of the indexed range).  It reads the L buckets of the
// head: of window-ordered tables (the build with a workspace) only the pieces that hold the
// keys of its slice, which is a build window, so that a head's buckets are read once in all;
// otherwise whole buckets, of which it keeps the keys of its slice.  The keys are marked in
// "seen" / "seen twice" bitmaps in LDS, and wavefront v then expands the bits of its
// kLgWaveBlocks blocks into an index list and gathers and weighs those keys
// (gather_estimate_wave) without the ballots ever leaving the compute unit: one partial per
// (head, slice, wavefront).  The keys of the static set T are dealt over these wavefronts (key
// j to wavefront j mod their number) and join the batches.  The keys appended since the build,
// 16 code blocks per slice, are found by the collision scan in the workgroups of slice 0, 1,
// ... and join the gather batches there.
// KT, WDT, LT: the collision scan's compile-time K, ceil(L/32) and tables of the last group (0: any).
template <int KT, int WDT, int LT, int ET>
__global__ __launch_bounds__(1024) void lookup_gather_kernel(AttnArgs a, TableArgs tb) {
  constexpr bool FP32 = ET == kFP32;
  constexpr int kSliceWords = kLgSliceBlocks * 2;       // 32-key words of a slice
  constexpr int kWaveWords = kLgWaveBlocks * 2;
  __shared__ uint32_t seen[kSliceWords], twice[kSliceWords];
  __shared__ uint32_t qs[256];
  __shared__ uint16_t lists[16][kLgWaveBlocks * kBlockKeys + kBlockKeys];
  const Ctx cx = resolve_context(a);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int slice = blockIdx.x;
  const int64_t bh = blockIdx.y;
  const int G = a.Hq / a.Hkv;
  const int unit = (int)((bh / a.Hq) * a.Hkv + (bh % a.Hq) / G);
  const int nb = 1 << a.K;
  const uint32_t* offs = tb.offsets + (int64_t)unit * a.L * (nb + 1);
  const uint32_t* idxs = tb.indices + (int64_t)unit * a.L * tb.n_cap;
  const uint32_t key_lo = (uint32_t)slice * (kLgSliceBlocks * kBlockKeys);
  const uint32_t qword = tid < a.NQ ? a.qcodes[bh * a.NQ + tid] : 0u;      // (requested, not yet used)
  for (int i = tid; i < kSliceWords; i += 1024) { seen[i] = 0u; twice[i] = 0u; }
  // ---- keys appended since the build: run `slice` of 16 of their code blocks, one per
  // wavefront, compared with this head's code while the query code is on its way; the
  // wavefront gathers what its block samples with its own batch ----
  uint64_t app_mask = 0;
  const int64_t app_blk = a.blk_begin + (int64_t)slice * 16 + wave;
  if (slice < a.lg_app_runs && app_blk < key_blocks(cx.n)) {
    const int hg = (int)(bh % a.Hq) % G;
    auto emit = [&](int, int64_t, uint64_t m) { app_mask = m; };
    if constexpr (KT == 0) {
      AnyWords<1> ahead;
      request_any(a, unit, app_blk, lane, ahead);
      scan_block_any<1, true>(a, cx, unit, app_blk, lane, hg, 1, ahead, false, emit);
    } else scan_blocks<KT, WDT, LT, 1, true>(a, cx, unit, app_blk, lane, hg, hg + 1, emit);
  }
  if (tid < a.NQ) qs[tid] = qword;
  __syncthreads();
  // wavefront v reads tables v, v+16, ...: lane k finds the bucket of table v + 16 k (its code
  // from the query's plane words, then two offsets); the descriptors reach the other lanes as
  // scalars.  Up to 128 entries of each bucket are requested before any is used; longer
  // buckets are finished in a loop.
  constexpr int kMaxB = 32;                             // L <= 512 tables over 16 wavefronts
  const int nbk = (a.L - wave + 15) >> 4;
  // 0: buckets in no particular order (also taken when the tables were built over another number
  // of keys than this call says: whole buckets are then read, never a piece that is not there)
  const int windows = (int)tb.header[0] == a.lg_nslices ? a.lg_nslices : 0;
  uint32_t my_start = 0, my_len = 0;
  if (lane < nbk) {
    const int t = wave + 16 * lane;
    const uint32_t* qw = qs + (t >> 5) * a.K;
    uint32_t code = 0;
    for (int b = 0; b < a.K; ++b) code |= ((qw[b] >> (t & 31)) & 1u) << b;
    const uint32_t* o = offs + (int64_t)t * (nb + 1) + code;
    my_start = o[0];
    uint32_t my_end = o[1];
    if (windows > 0) {
      // window-ordered buckets: only the piece that holds the keys of this slice
      const uint32_t* wc = tb.wincum + (((int64_t)unit * a.L + t) * windows + slice) * nb + code;
      if (slice + 1 < windows) my_end = my_start + wc[nb];
      my_start += wc[0];
    }
    my_len = my_end - my_start;
  }
  constexpr uint32_t kSliceKeys = kLgSliceBlocks * kBlockKeys;
  auto mark = [&](uint32_t key) {
    const uint32_t rel = key - key_lo;                  // absent entries and other slices: out of range
    if (rel < kSliceKeys) {
      const uint32_t bit = 1u << (rel & 31);
      if (atomicOr(&seen[rel >> 5], bit) & bit) atomicOr(&twice[rel >> 5], bit);
    }
  };
  if (windows > 0) {
    // Window-ordered tables: a piece holds about 16 keys (n 2^-K per window of 16384 keys), so
    // half a wavefront reads a piece: lanes 0..31 that of table v + 32 j, lanes 32..63 that of
    // table v + 32 j + 16.  The first atomics of all pieces are issued together and their
    // answers (was the key seen before?) used afterwards, so the LDS round trips overlap.
    // Pieces of more than 32 keys are finished in a loop.
    const int half = lane >> 5, li = lane & 31;
    uint32_t e[kMaxB / 2];
#pragma unroll
    for (int j = 0; j < kMaxB / 2; ++j) {
      e[j] = 0xffffffffu;
      if (2 * j < nbk) {
        const int k = 2 * j + half;
        const uint32_t start = __shfl(my_start, k), len = __shfl(my_len, k);   // (0 for k >= nbk)
        const uint32_t* p = idxs + (int64_t)(wave + 16 * k) * tb.n_cap + start;
        if ((uint32_t)li < len) e[j] = p[li];
      }
    }
    uint32_t before[kMaxB / 2];
#pragma unroll
    for (int j = 0; j < kMaxB / 2; ++j) {
      const uint32_t rel = e[j] - key_lo;
      before[j] = 0u;
      if (2 * j < nbk && rel < kSliceKeys) before[j] = atomicOr(&seen[rel >> 5], 1u << (rel & 31));
    }
#pragma unroll
    for (int j = 0; j < kMaxB / 2; ++j) {
      const uint32_t rel = e[j] - key_lo;
      if (2 * j < nbk && rel < kSliceKeys && ((before[j] >> (rel & 31)) & 1u)) atomicOr(&twice[rel >> 5], 1u << (rel & 31));
    }
    // (rare: the wavefront knows at once whether any of its pieces is that long)
    for (uint64_t f = __ballot(my_len > 32); f; f &= f - 1) {
      const int k = __ffsll((unsigned long long)f) - 1;
      const uint32_t len = __builtin_amdgcn_readlane(my_len, k);
      const uint32_t* p = idxs + (int64_t)(wave + 16 * k) * tb.n_cap + __builtin_amdgcn_readlane(my_start, k);
      for (uint32_t j = 32 + lane; j < len; j += 64) mark(p[j]);
    }
  } else {
    // Buckets in no particular order: up to 128 entries of each bucket are requested before any
    // is used; longer buckets are finished in a loop.
    uint32_t e0[kMaxB], e1[kMaxB];
#pragma unroll
    for (int k = 0; k < kMaxB; ++k) {
      e0[k] = 0xffffffffu; e1[k] = 0xffffffffu;
      if (k < nbk) {
        const uint32_t start = __builtin_amdgcn_readlane(my_start, k), len = __builtin_amdgcn_readlane(my_len, k);
        const uint32_t* p = idxs + (int64_t)(wave + 16 * k) * tb.n_cap + start;
        if ((uint32_t)lane < len) e0[k] = p[lane];
        if ((uint32_t)lane + 64 < len) e1[k] = p[lane + 64];
      }
    }
    // Marking: absent entries and keys of other slices fall out of range.  The first atomics of
    // eight buckets are issued together and their answers (was the key seen before?) used
    // afterwards, so the LDS round trips overlap instead of following each other.
#pragma unroll
    for (int c0 = 0; c0 < kMaxB; c0 += 8) {
      if (c0 < nbk) {
        uint32_t before[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const uint32_t rel = ((i & 1) ? e1[c0 + (i >> 1)] : e0[c0 + (i >> 1)]) - key_lo;
          before[i] = 0u;
          if (rel < kSliceKeys) before[i] = atomicOr(&seen[rel >> 5], 1u << (rel & 31));
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const uint32_t rel = ((i & 1) ? e1[c0 + (i >> 1)] : e0[c0 + (i >> 1)]) - key_lo;
          if (rel < kSliceKeys && ((before[i] >> (rel & 31)) & 1u)) atomicOr(&twice[rel >> 5], 1u << (rel & 31));
        }
      }
    }
    for (uint64_t f = __ballot(my_len > 128); f; f &= f - 1) {
      const int k = __ffsll((unsigned long long)f) - 1;
      const uint32_t len = __builtin_amdgcn_readlane(my_len, k);
      const uint32_t* p = idxs + (int64_t)(wave + 16 * k) * tb.n_cap + __builtin_amdgcn_readlane(my_start, k);
      for (uint32_t j = 128 + lane; j < len; j += 64) mark(p[j]);
    }
  }
  __syncthreads();
  // ---- gather: wavefront v takes blocks v*kLgWaveBlocks .. of the slice ----
  const uint32_t* hit = a.tau >= 2 ? twice : seen;
  const int64_t hi_key = cx.n - a.n_local < tb.n ? cx.n - a.n_local : tb.n;   // indexed, not in the local window
  const int64_t wave_key0 = (int64_t)key_lo + (int64_t)wave * (kLgWaveBlocks * kBlockKeys);
  uint16_t* list = lists[wave];
  HeadVectors<FP32> hv;
  request_head_vectors<FP32>(a, unit, bh, hv);
  uint32_t bits = 0;
  if (lane < kWaveWords) {
    const int64_t kfirst = wave_key0 + (int64_t)lane * 32;
    const int64_t lo = (a.n_sink > kfirst ? a.n_sink : kfirst) - kfirst;
    const int64_t hi = (hi_key < kfirst + 32 ? hi_key : kfirst + 32) - kfirst;
    uint32_t elig = 0;
    if (hi > lo) elig = (hi - lo >= 32 ? 0xffffffffu : ((1u << (hi - lo)) - 1u)) << lo;
    bits = hit[wave * kWaveWords + lane] & elig;
  }
  if (a.dbg_cand) {                                      // debug output only
    for (uint32_t f = bits; f; f &= f - 1) {
      const int pos = atomicAdd(&a.dbg_ncand[bh], 1);
      if (pos < a.dbg_cand_cap)
        a.dbg_cand[bh * a.dbg_cand_cap + pos] = (int32_t)(wave_key0 + lane * 32 + __ffs(f) - 1);
    }
  }
  const int c = __popc(bits);
  const int incl = half_prefix_sum32(c);                 // kWaveWords <= 32
  const int in_slice = __builtin_amdgcn_readlane(incl, 31);
  int pos = incl - c;
  for (uint32_t f = bits; f; f &= f - 1) list[pos++] = (uint16_t)(lane * 32 + __ffs(f) - 1);
  // behind them the sampled keys of the wavefront's appended block (lane = key of the block)
  if ((app_mask >> lane) & 1)
    list[in_slice + __popcll(app_mask & ((1ull << lane) - 1ull))] = (uint16_t)lane;
  const int n_sampled = in_slice + __popcll(app_mask);
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
  // static keys slot, slot + slots, ... ride along behind the sampled ones
  const int slots = a.lg_nslices * 16, slot = slice * 16 + wave;
  const int nst = static_share(cx, slot, slots);
  const WavePartial wp = gather_estimate_wave<ET, (FP32 ? 4 : 8)>(a, unit, n_sampled + nst, n_sampled, hv, [&](int cc) {
    if (cc >= n_sampled) return static_key(a, cx, slot + (int64_t)(cc - n_sampled) * slots);
    return (cc < in_slice ? wave_key0 : app_blk * kBlockKeys) + (int64_t)list[cc];
  });
  store_partial(wp, a.partial + (bh * a.nranges + slot) * kPartialStride);
}

template <int KT, int WDT, int LT>
static void launch_lookup_gather_for(const AttnArgs& a, const TableArgs& t, dim3 grid, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  auto go = [&](auto kernel) {
    if (start || stop) hipExtLaunchKernelGGL(kernel, grid, dim3(1024), 0, s, start, stop, 0, a, t);
    else hipLaunchKernelGGL(kernel, grid, dim3(1024), 0, s, a, t);
  };
  if (a.is_fp32) go(lookup_gather_kernel<KT, WDT, LT, kFP32>);
  else if (a.kv_fp8) go(lookup_gather_kernel<KT, WDT, LT, kFP8>);
  else go(lookup_gather_kernel<KT, WDT, LT, kBF16>);
}

hipError_t launch_lookup_gather(const AttnArgs& a0, const TableArgs& t, int nslices, int appended_runs, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  AttnArgs a = a0;
  a.lg_nslices = nslices;
  a.lg_app_runs = appended_runs;                       // <= nslices
  const dim3 grid((unsigned)nslices, (unsigned)((int64_t)a.B * a.Hq));
#define MP_TUNED(KT, LL) if (a.K == KT && a.L == LL) launch_lookup_gather_for<KT, words_of(LL), tail_of(LL)>(a, t, grid, s, start, stop); else
  MP_TUNED_TABLES(MP_TUNED) launch_lookup_gather_for<0, 0, 0>(a, t, grid, s, start, stop);
#undef MP_TUNED
  return hipGetLastError();
}

hipError_t launch_table_lookup(const AttnArgs& a, const TableArgs& t, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  const int64_t nblk = key_blocks(t.n);
  // two bits per key in LDS: up to 196608 indexed keys in 48 KB (5 KB more are static)
  const size_t bitmap_bytes = (size_t)nblk * 2 * 2 * sizeof(uint32_t);
  if (!a.dbg_counts && (a.tau == 1 || a.tau == 2) && bitmap_bytes <= 48 * 1024) {
    const dim3 grid((unsigned)((int64_t)a.B * a.Hq));
    auto go = [&](auto kernel) {
      if (start || stop) hipExtLaunchKernelGGL(kernel, grid, dim3(1024), bitmap_bytes, s, start, stop, 0, a, t);
      else hipLaunchKernelGGL(kernel, grid, dim3(1024), bitmap_bytes, s, a, t);
    };
    // by the average bucket, so that few are longer than the first request (256 heads x 20000 keys, (10,300): 20 on
    // average, <8, 1> 10.0 us, <8, 2> 12.2)
    const int64_t average = t.n >> a.K;
    if (average <= 40) go(table_lookup_bitmap_kernel<8, 1>);
    else if (average <= 96) go(table_lookup_bitmap_kernel<8, 2>);
    else go(table_lookup_bitmap_kernel<4, 3>);
    return hipGetLastError();
  }
  auto go = [&](auto kernel, int run_blocks) {
    const dim3 grid((unsigned)((nblk + run_blocks - 1) / run_blocks), (unsigned)((int64_t)a.B * a.Hq));
    if (start || stop) hipExtLaunchKernelGGL(kernel, grid, dim3(1024), 0, s, start, stop, 0, a, t);
    else hipLaunchKernelGGL(kernel, grid, dim3(1024), 0, s, a, t);
  };
  if (a.L <= 255) go(table_lookup_kernel<8>, kLookupRunBlocks<8>);
  else go(table_lookup_kernel<16>, kLookupRunBlocks<16>);
  return hipGetLastError();
}

}  // namespace mp
