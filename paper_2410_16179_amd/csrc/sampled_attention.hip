// One decode step of LSH-sampled attention (Algorithm 1 "MagicPIG Decoding"; Eq. "lsh
// sampling probability"; Eq. "close form"), HBM-bound.
//
// Retrieval by scanning the packed codes of every key (magicpig_sampled_attention):
//   scan_gather_kernel, then merge_partials_kernel.
// Retrieval through the hash tables (magicpig_sampled_attention_tables):
//   lookup_gather_kernel (hash_tables.hip: lookup, gather, scan of the few appended keys in one
//   launch), merge_partials_kernel; or, with many heads, for the count output and for other
//   min_hits: table lookup [+ collision_scan_kernel over the keys appended since the build],
//   gather_estimate_kernel, merge_partials_kernel.
//
// collision scan (scan_blocks)
//   One wavefront per 64-key code block, lane = key: the block is a contiguous 256*NW-byte
//   read, 16 bytes per lane and load.  For each of the G query heads of the KV head the K
//   bit planes of every table word are XNOR-ed with the query's (scalar operands) and
//   AND-ed together; a popcount adds the number of colliding tables.  Keys outside the
//   static set with count >= min_hits are reported as one 64-bit ballot per (head, block).
//   No LDS, no barrier, about 60 VGPRs.
// gather and estimate (gather_estimate_wave)
//   One wavefront per (query head, run of key blocks): the sampled keys are an index list in
//   LDS (gather_estimate_kernel expands the ballots by a wavefront prefix sum; scan_gather_kernel
//   appends to the list while it compares); the static sink and local-window keys ride
//   along in these batches; rows are gathered four at a time (a quarter wavefront holds one 128-element row)
//   with up to 32 K rows and 32 V rows in flight; q.k, q.(k-mu), |k-mu|^2 are reduced over
//   the 16 lanes of a row, the inclusion probability u_i and the logit q.k/sqrt(d) - log u_i
//   are evaluated once per candidate, and an online max/sum softmax accumulates the weighted
//   V rows.  The wavefront stores a (max, sum, output) partial.
// scan_gather_kernel does both for a run of 4 to 24 key blocks (chosen by the host) in one workgroup;
// collision_scan_kernel / gather_estimate_kernel are the two as separate launches, joined by
// the ballots in HBM.
// merge_partials_kernel combines a head's partials (the "recursive attention" merge of
//   Sec. 4.4) and writes the output row.
#include "attention_common.h"
#include <hip/hip_ext.h>
#include <type_traits>

#ifndef MP_SCAN_BPW
#define MP_SCAN_BPW 1
#endif

namespace mp {

template <int KT, int WDT, int LT, int BPW>
__global__ __launch_bounds__(256) void collision_scan_kernel(AttnArgs a) {
  const Ctx c = resolve_context(a);
  // readfirstlane tells the compiler that the wavefront index (and everything derived from
  // it: KV head, query-code address) is uniform, so those loads become scalar
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t nblk = key_blocks(c.n);
  const int unit = blockIdx.y;
  const int64_t blk0 = a.blk_begin + ((int64_t)blockIdx.x * 4 + wave) * BPW;
  if (blk0 >= nblk) return;
  const int G = a.Hq / a.Hkv;
  const int64_t head0 = (int64_t)(unit / a.Hkv) * a.Hq + (int64_t)(unit % a.Hkv) * G;
  auto emit = [&](int h, int64_t blk, uint64_t m) {
    if (lane == 0) a.masks[(head0 + h) * nblk + blk] = m;
  };
  // grid layer z compares with its share of the heads
  const int per = (G + gridDim.z - 1) / gridDim.z, h0 = blockIdx.z * per, h1 = h0 + per < G ? h0 + per : G;
  if (h0 >= h1) return;
  if constexpr (KT == 0) {
    AnyWords<WDT> ahead;
    request_any(a, unit, blk0, lane, ahead);
    scan_block_any<WDT, true>(a, c, unit, blk0, lane, h0, h1 - h0, ahead, false, emit);
  } else scan_blocks<KT, WDT, LT, BPW, true>(a, c, unit, blk0, lane, h0, h1, emit);
}

// rows per quarter wavefront and batch of the stand-alone gather: 32 K and 32 V rows in flight
template <int ET> constexpr int kGatherIters = ET == kFP32 ? 4 : 8;
// entries of a wavefront's index list: fewer than a batch left over, and all keys of a piece
template <int ET> constexpr int kGatherList = kRangeBlocks * kBlockKeys + 4 * kGatherIters<ET>;

// One wavefront = one (query head, run of g_run_blocks key blocks).  blockDim = 64 * G:
// the G wavefronts of a workgroup serve the G heads of one KV head on the same run.  The ballots of
// sixteen blocks at a time are expanded into an index list in LDS by a prefix sum; full batches of rows are taken
// from its front, and what is left waits for the next sixteen blocks.  The keys of the static set T are
// dealt over the runs (key j to run j mod runs) and join the last batch, or they have wavefronts of their own behind those of the runs
// (plan_gather).  kFull = false: runs of one piece, everything goes through the code of the last batch.
// Bound by the rows it gathers (random 256-byte rows) and by the vector unit.  512 heads x 131072 keys, (10,170), 1.3
// million rows: 152 us (643 MB at 4.2 TB/s, vector unit 73 % busy) with a wavefront for each 1024 keys, about 20 of the 32
// rows of a batch and workgroups of their own for T; now 122 us (5.3 TB/s): the estimator's arithmetic, once per
// batch, serves 32 rows, full batches need no masks, and the 16-lane sums of a batch are taken together.
// Four wavefronts per SIMD (128 registers; at 141, three, it was 40 % slower); the lists are as many as the workgroup has
// wavefronts, so that sixteen fit a compute unit with few heads too (room for eight lists in a workgroup of one
// wavefront: nine fitted; 512 heads of 512 KV heads x 16384 keys, (10,150), the step 40.3 us, now 36.6).
template <int ET, bool kFull>
__global__ __launch_bounds__(512, 4) void gather_estimate_kernel(AttnArgs a) {
  constexpr bool FP32 = ET == kFP32;
  constexpr int kIt = kGatherIters<ET>, kBatch = 4 * kIt;
  extern __shared__ uint16_t lists[];                      // [heads of the workgroup][kGatherList<ET>]
  const Ctx c = resolve_context(a);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int unit = blockIdx.y, run = blockIdx.x;
  const int b = unit / a.Hkv, g = unit % a.Hkv;
  const int G = a.Hq / a.Hkv;
  const int64_t bh = (int64_t)b * a.Hq + (int64_t)g * G + wave;
  const int64_t nblk = key_blocks(c.n);
  // wavefronts behind those of the runs take static keys only
  const int nruns = (int)gridDim.x - a.g_static_runs;
  const bool own = run >= nruns;
  const int run_blocks = own ? 0 : a.g_run_blocks;
  const int64_t blk0 = (int64_t)run * a.g_run_blocks;
  uint16_t* list = lists + wave * kGatherList<ET>;
  HeadVectors<FP32> hv;
  request_head_vectors<FP32>(a, unit, bh, hv);
  const uint64_t* masks = a.masks + bh * nblk;
  auto ballots = [&](int at) {                             // lane i < 16: block blk0 + at + i
    return lane < kRangeBlocks && at < run_blocks && blk0 + at + lane < nblk ? masks[blk0 + at + lane] : 0ull;
  };
  GatherState st;
  int have = 0;                                            // keys in the list
  uint64_t next = ballots(0);
  int64_t s0 = run;                                        // static keys of this wavefront: s0, s0 + sstep, ...
  int sstep = nruns, nst = a.g_static_runs > 0 ? 0 : static_share(c, run, nruns);
  if (own) {
    s0 = (int64_t)(run - nruns) * a.g_static_keys;
    sstep = 1;
    const int64_t left = c.n_static - s0;
    nst = left <= 0 ? 0 : (left < a.g_static_keys ? (int)left : a.g_static_keys);
  }
  if (kFull && own) {
    const int full = nst / kBatch * kBatch;
    if (full > 0) gather_estimate_keys<ET, kIt, true>(st, a, unit, full, 0, hv, [&](int cc) { return static_key(a, c, s0 + cc); });
    s0 += full;
    nst -= full;
  }
#pragma unroll 1
  for (int at = 0; at < run_blocks; at += kRangeBlocks) {
    uint64_t m = next;
    next = ballots(at + kRangeBlocks);
    const int pc = __popcll(m);
    static_assert(kRangeBlocks <= 16, "the ballots of a range are summed over one row of 16 lanes");
    const int incl = row_prefix_sum16(pc);
    int pos = have + incl - pc;
    while (m) {
      const int bit = __ffsll((unsigned long long)m) - 1;
      list[pos++] = (uint16_t)((at + lane) * kBlockKeys + bit);
      m &= m - 1;
    }
    have += __builtin_amdgcn_readlane(incl, kRangeBlocks - 1);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
    if (!kFull) continue;
    const int full = have / kBatch * kBatch, left = have - full;
    if (full > 0)
      gather_estimate_keys<ET, kIt, true>(st, a, unit, full, full, hv, [&](int cc) { return blk0 * kBlockKeys + (int64_t)list[cc]; });
    const uint16_t k = lane < left ? list[full + lane] : (uint16_t)0;   // fewer than a batch are left: to the front
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
    if (lane < left) list[lane] = k;
    have = left;
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
  gather_estimate_keys<ET, kIt, false>(st, a, unit, have + nst, have, hv, [&](int cc) {
    const int sampled = list[cc < have ? cc : 0];            // (read for static keys, too: no branch between the reads of a batch)
    const int64_t fixed = static_key(a, c, s0 + (int64_t)(cc - have) * sstep);
    return cc < have ? blk0 * kBlockKeys + sampled : fixed;
  });
  store_partial(finish_gather(st), a.partial + (bh * a.nranges + run) * kPartialStride);
}

// Wavefronts that share the keys of a run and head in the one-launch scan + gather (KT, HT: compile-time K, 0
// for the form for any, and the heads that form is laid out for): two where a workgroup serves one head.
// They join their partials in LDS.  Measured with the merge, (9,110): 32 KV heads x 20011 keys one wavefront
// 34.1 us, two 31.3 (32.1 with a partial each); one KV head x 100000 keys 18.2 (22.8 with a partial each: the
// merge of 782 partials is one workgroup's work).  Four wavefronts, or two heads shared by two each, gained nothing.
template <int KT, int HT> constexpr int kScanParts = KT == 0 && HT == 1 ? 2 : 1;

// Scan and gather in one launch (the whole context is scanned, no hash tables): a workgroup of
// four wavefronts compares a run of up to kFusedBlocks = 24 consecutive code blocks with the G
// heads' codes (scan_blocks, f_wave_blocks blocks per wavefront one after the other), appends
// the keys each head samples to that head's list in LDS as it goes, and wavefront h then gathers
// and weighs the keys that head h samples from the
// run (16 blocks: about 17 at a sampling rate of 1.6 %, one batch of the 32-row gather).  As
// separate launches the gather follows the scan with two dependent round trips of its own
// (ballots, then rows) on an idle memory system; here the rows of one workgroup travel while
// the others still stream codes, and only the gather of the last workgroups is exposed
// (measured at 32 heads x 98304 keys: 33 us against 25.6 + 13.7 us).  The host picks the run
// length, 4 to 24 blocks: the shortest whose workgroups are all resident at once (16 blocks at
// that shape).  Shorter runs measured the same kernel time there but cost more partials and
// gather batches.  What remains exposed there, after the last block of codes has arrived
// (time stamps): 0.7 us until the four wavefronts meet, 0.6 us candidate positions and row
// addresses, 1.6 us for the rows, 1.3 us estimator, 0.7 us weighted V rows and the partial;
// until then the kernel moves its bytes at the rate of a plain read of the same codes.
// OCC: workgroups per compute unit the kernel is compiled for (see launch_scan_gather_as).
// The grid is one workgroup per run (at 8 KV heads x 98304 keys: 768, exactly what is resident
// at once; workgroups that start late end last).  The keys of the static set T are dealt over
// the runs of their KV head (key j to run j mod runs) and join the gather batches there, so
// they cost neither workgroups nor batches nor partials of their own.
// One partial per (head, run); where two wavefronts share a head's keys (kScanParts) they join theirs in LDS.
// DBG: with the debug outputs (counts, candidate lists).
// ONE: a workgroup (grid layer z) serves one of the G heads (few keys, see launch_scan_gather_as).
// KT, WDT, LT: see scan_blocks; KT = 0: any K and L, WDT = the heads scan_block_any is laid out for.
// ET: element type of the caches (kBF16, kFP32, or kFP8 with bf16 queries).
template <int KT, int WDT, int LT, int ET, bool DBG, int OCC, bool ONE = false>
__global__ __launch_bounds__(256, OCC) void scan_gather_kernel(AttnArgs a) {
  constexpr bool FP32 = ET == kFP32;
  constexpr int kIt = FP32 ? (kFusedIters + 1) / 2 : kFusedIters;   // the same registers per batch
  constexpr int kSeg = kFusedWaveBlocks * kBlockKeys;      // most keys one wavefront can report for a head
  // seg[h][w]: the keys of the run that head h samples among the blocks of wavefront w, in key
  // order (position in the run, 11 bits); seg_n[h][w]: how many.  Written while the blocks are
  // compared, so that nothing but the row gather is left to do after the last block.
  constexpr int kHeads = ONE ? 1 : 8;
  __shared__ uint16_t seg[kHeads][4][kSeg];
  __shared__ int seg_n[kHeads][4];
  const Ctx c = resolve_context(a);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int unit = blockIdx.y, run = blockIdx.x;
  const int nruns = gridDim.x;                             // = f_nranges
  const int G = a.Hq / a.Hkv;
  const int64_t head0 = (int64_t)(unit / a.Hkv) * a.Hq + (int64_t)(unit % a.Hkv) * G;
  const int h0 = ONE ? blockIdx.z : 0, h1 = ONE ? h0 + 1 : G;   // heads of this workgroup
  const int64_t nblk = key_blocks(c.n);
  const int wave_blocks = a.f_wave_blocks;                 // 1 .. kFusedWaveBlocks key blocks per wavefront
  const int run_blocks = 4 * wave_blocks;
  const int64_t blk0 = (int64_t)run * run_blocks;
  int found = 0;                                           // lane h: keys of head h found so far by this wavefront
  uint64_t last_found = 0;                                 // keys of the wavefront's last block that some head samples
  AnyWords<KT == 0 ? WDT : 1> ahead;                       // (any K and L only)
  if constexpr (KT == 0)
    if (blk0 + wave * wave_blocks < nblk) request_any(a, unit, blk0 + wave * wave_blocks, lane, ahead);
#pragma unroll 1
  for (int j = 0; j < wave_blocks; ++j) {
    const int bi = wave * wave_blocks + j;
    if (blk0 + bi < nblk) {
      auto emit = [&](int h, int64_t, uint64_t m) {
        if (m) {                                           // (wave-uniform)
          const int at = __builtin_amdgcn_readlane(found, h - h0);
          const int below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
          if ((m >> lane) & 1) seg[h - h0][wave][at + below] = (uint16_t)(bi * kBlockKeys + lane);
          if (lane == h - h0) found = at + __popcll(m);
        }
        if (j == wave_blocks - 1) last_found |= m;
      };
      if constexpr (KT == 0) scan_block_any<WDT, DBG>(a, c, unit, blk0 + bi, lane, h0, h1 - h0, ahead, j + 1 < wave_blocks && blk0 + bi + 1 < nblk, emit);
      else scan_blocks<KT, WDT, LT, 1, DBG>(a, c, unit, blk0 + bi, lane, h0, h1, emit);
    }
  }
  if (lane < h1 - h0) seg_n[lane][wave] = found;
  // The gather reads its arguments from the kernel argument segment again, through a pointer the
  // compiler cannot trace back: otherwise it loads them all at the start of the kernel and keeps
  // them in scalar registers across the scan, whose query words then no longer fit (50 spills,
  // a reload on every third instruction of the compare loop).
  typedef const AttnArgs __attribute__((address_space(4))) * const_args_ptr;
  const_args_ptr kp = (const_args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(kp));
  const AttnArgs& ga = *(const AttnArgs*)kp;
  // ... and all of them here, in one batch of scalar loads that is back before the barrier opens
  // (requested where they are used they cost four dependent round trips at the end of the kernel)
  asm volatile("" ::"s"(ga.q), "s"(ga.Kc), "s"(ga.Vc), "s"(ga.mu), "s"(ga.partial), "s"(ga.Hq), "s"(ga.Hkv), "s"(ga.K), "s"(ga.L),
               "s"(ga.tau), "s"(ga.n_sink), "s"(ga.n_local), "s"(ga.ks_b), "s"(ga.ks_h), "s"(ga.ks_n), "s"(ga.vs_b), "s"(ga.vs_h),
               "s"(ga.vs_n), "s"(ga.f_nranges), "s"(ga.f_touch), "s"(ga.scale));
  asm volatile("" ::"s"(ga.head_ratio[0]), "s"(ga.head_ratio[1]), "s"(ga.head_ratio[2]), "s"(ga.head_ratio[3]), "s"(ga.tail_ratio[0]),
               "s"(ga.tail_ratio[1]), "s"(ga.tail_ratio[2]), "s"(ga.tail_ratio[3]), "s"(ga.tail_ratio[4]), "s"(ga.tail_ratio[5]),
               "s"(ga.tail_ratio[6]), "s"(ga.tail_ratio[7]), "s"(ga.tail_ratio[8]), "s"(ga.tail_ratio[9]), "s"(ga.tail_ratio[10]),
               "s"(ga.tail_ratio[11]), "s"(ga.tail_ratio[12]), "s"(ga.tail_ratio[13]), "s"(ga.tail_ratio[14]), "s"(ga.tail_ratio[15]));
  static_assert(kFastTau == 4 && kTailTerms == 16, "the list above names every ratio");
  // When the workgroups of a launch come in several rounds the memory system is busy whenever one
  // of them reaches its gather, and its rows then take as long as a block of codes.  The rows of
  // the keys found in the last block are requested last of all (block compared, barrier, candidate
  // positions, only then the request): a wavefront touches one word of each of their cache lines
  // here already, so that the gather finds them in, or on their way to, the L2 (measured at batch
  // 16 x 65536 keys: 284 -> 276 us; with all workgroups resident at once it costs half a
  // microsecond instead, and touching the rows of every block costs 10 %).  The touches are
  // loads with a destination, consumed at the end of the kernel; the barrier does not wait for them.
  constexpr int kLines = ET == kFP32 ? 4 : (ET == kFP8 ? 1 : 2);            // 128-byte lines per row
  uint32_t touched[2 * kLines];
#pragma unroll
  for (int l = 0; l < 2 * kLines; ++l) touched[l] = 0;
  if (ga.f_touch && ((last_found >> lane) & 1)) {
    const int64_t key = (blk0 + wave * wave_blocks + wave_blocks - 1) * kBlockKeys + lane;
    const int b = unit / ga.Hkv, g = unit % ga.Hkv;
    const char* kr = (const char*)ga.Kc + ((int64_t)b * ga.ks_b + (int64_t)g * ga.ks_h + key * ga.ks_n) * (kLines * 128 / kHeadDim);
    const char* vr = (const char*)ga.Vc + ((int64_t)b * ga.vs_b + (int64_t)g * ga.vs_h + key * ga.vs_n) * (kLines * 128 / kHeadDim);
#pragma unroll
    for (int l = 0; l < kLines; ++l) {
      touched[2 * l] = *reinterpret_cast<const uint32_t*>(kr + 128 * l);
      touched[2 * l + 1] = *reinterpret_cast<const uint32_t*>(vr + 128 * l);
    }
  }
  // (the barrier orders the LDS writes above: it waits for them, not for loads in flight)
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  constexpr int parts = ONE ? 1 : kScanParts<KT, WDT>;    // (ONE: the same sums as a workgroup for G heads)
  auto attend = [&](int h, int part) {                     // share `part` of the keys of head h
    HeadVectors<FP32> hv;
    request_head_vectors<FP32>(ga, unit, head0 + h, hv);
    // the four wavefronts' keys of head h, one after the other: candidate cc is entry cc - s_w of
    // the last wavefront w whose first candidate s_w is not beyond cc
    const int s1 = __builtin_amdgcn_readfirstlane(seg_n[h - h0][0]);
    const int s2 = s1 + __builtin_amdgcn_readfirstlane(seg_n[h - h0][1]);
    const int s3 = s2 + __builtin_amdgcn_readfirstlane(seg_n[h - h0][2]);
    const int total = s3 + __builtin_amdgcn_readfirstlane(seg_n[h - h0][3]);
    const uint16_t* segh = &seg[h - h0][0][0];
    // static keys run, run + nruns, ... ride along behind the sampled ones
    const int all = total + static_share(c, run, nruns);
    // this wavefront's share: candidates lo .. lo + mine - 1
    const int share = (all + parts - 1) / parts, lo = part * share;
    const int mine = parts == 1 ? all : (all - lo < share ? (all > lo ? all - lo : 0) : share);
    return gather_estimate_wave<ET, kIt>(ga, unit, mine, total - lo, hv, [&](int cl) {
      const int cc = cl + lo;
      if (cc >= total) return static_key(ga, c, run + (int64_t)(cc - total) * nruns);
      const int w = (cc >= s1) + (cc >= s2) + (cc >= s3);
      const int first = w == 0 ? 0 : (w == 1 ? s1 : (w == 2 ? s2 : s3));
      return blk0 * kBlockKeys + (int64_t)segh[w * kSeg + cc - first];
    });
  };
  auto place = [&](int h) { return ga.partial + ((head0 + h) * ga.f_nranges + run) * kPartialStride; };
  if constexpr (parts == 1) {
    for (int h = h0 + wave; h < h1; h += 4) store_partial(attend(h, 0), place(h));
  } else {                                                 // one head
    __shared__ float joined[kPartialStride];
    WavePartial wp;
    if (wave < parts) wp = attend(h0, wave);
    if (wave == 1) store_partial(wp, joined);
    __syncthreads();
    if (wave == 0) {
      join_partial(wp, joined);
      store_partial(wp, place(h0));
    }
  }
#pragma unroll
  for (int l = 0; l < 2 * kLines; ++l) asm volatile("" ::"v"(touched[l]));
}

// Merges the (max, sum, output) partials of one query head (NWAVES wavefronts: wavefront w takes
// every NWAVES-th group of partials, lane = two output elements).  Every load of a pass is
// issued before any is used - their addresses do not depend on the data - so a pass costs
// one memory round trip; LDS joins the wavefronts.
template <int NWAVES>
__global__ __launch_bounds__(64 * NWAVES) void merge_partials_kernel(AttnArgs a) {
  constexpr int kPer = 16;                    // partials per wavefront and pass
  __shared__ float sm[NWAVES], sl_[NWAVES], so[NWAVES][kHeadDim];
  const int64_t bh = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const float* hp = a.partial + bh * a.nranges * kPartialStride;
  float m = -INFINITY, l = 0.f, ox = 0.f, oy = 0.f;
  for (int r0 = wave * kPer; r0 < a.nranges; r0 += NWAVES * kPer) {
    float2 oc[kPer];
    float mr[kPer], lr[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const bool ok = r0 + j < a.nranges;
      const float* pp = hp + (int64_t)(ok ? r0 + j : r0) * kPartialStride;
      oc[j] = *reinterpret_cast<const float2*>(pp + 2 * lane);
      mr[j] = ok ? pp[128] : -INFINITY;
      lr[j] = pp[129];
    }
    float mn = m;
#pragma unroll
    for (int j = 0; j < kPer; ++j) mn = fmaxf(mn, mr[j]);
    if (mn > -INFINITY) {
      const float sa = expf(m - mn);
      ox *= sa; oy *= sa; l *= sa;
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const float sb = mr[j] > -INFINITY ? expf(mr[j] - mn) : 0.f;
        ox += sb * oc[j].x;
        oy += sb * oc[j].y;
        l += sb * lr[j];
      }
      m = mn;
    }
  }
  if (lane == 0) { sm[wave] = m; sl_[wave] = l; }
  so[wave][2 * lane] = ox;
  so[wave][2 * lane + 1] = oy;
  __syncthreads();
  if (threadIdx.x < kHeadDim) {
    float M = sm[0];
#pragma unroll
    for (int w = 1; w < NWAVES; ++w) M = fmaxf(M, sm[w]);
    float acc = 0.f, lt = 0.f;
    if (M > -INFINITY) {
#pragma unroll
      for (int w = 0; w < NWAVES; ++w) {
        if (sm[w] > -INFINITY) {
          const float s = expf(sm[w] - M);
          acc += s * so[w][threadIdx.x];
          lt += s * sl_[w];
        }
      }
    }
    a.out[bh * kHeadDim + threadIdx.x] = lt > 0.f ? acc / lt : 0.f;
  }
}

__global__ void zero_output_kernel(float* out, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) out[i] = 0.f;
}

// Ordinary launch, or - when events are given - a launch whose events carry the kernel's own
// begin / end timestamps (what a profiler reports), not the stream's dispatch times.
template <class F, class... Args>
static void launch_timed_lds(F kernel, dim3 grid, dim3 block, size_t lds, hipStream_t s, hipEvent_t start, hipEvent_t stop, Args... args) {
  if (start || stop) hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)lds, s, start, stop, 0, args...);
  else hipLaunchKernelGGL(kernel, grid, block, lds, s, args...);
}
template <class F, class... Args>
static void launch_timed(F kernel, dim3 grid, dim3 block, hipStream_t s, hipEvent_t start, hipEvent_t stop, Args... args) {
  launch_timed_lds(kernel, grid, block, 0, s, start, stop, args...);
}

static hipError_t launch_scan(const AttnArgs& a, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  constexpr int kBPW = MP_SCAN_BPW;
  const dim3 block(256);
  const int64_t nscanned = key_blocks(a.n) - a.blk_begin;   // > 0
  // Few blocks (the keys appended since the tables were built): a head per wavefront.  A wavefront that
  // takes all heads waits for the query words of one after the other (64 units x 8 blocks, eight heads:
  // 9.0 us against 6.6); with four wavefronts per SIMD those waits are hidden and the blocks are read once.
  const unsigned layers = nscanned * a.B * a.Hkv <= 4 * kNumCU ? (unsigned)(a.Hq / a.Hkv) : 1u;
  const dim3 grid_t((unsigned)((nscanned + 4 * kBPW - 1) / (4 * kBPW)), (unsigned)(a.B * a.Hkv), layers);
#define MP_TUNED(KT, LL)                                                                            \
  if (a.K == KT && a.L == LL) {                                                                     \
    launch_timed(collision_scan_kernel<KT, words_of(LL), tail_of(LL), kBPW>, grid_t, block, s, start, stop, a);  \
    return hipGetLastError();                                                                       \
  }
  MP_TUNED_TABLES(MP_TUNED)
#undef MP_TUNED
  const dim3 grid((unsigned)((nscanned + 3) / 4), (unsigned)(a.B * a.Hkv), layers);
  const int per = a.Hq / a.Hkv / (int)layers;            // heads of a wavefront
  if (per == 1) launch_timed(collision_scan_kernel<0, 1, 0, 1>, grid, block, s, start, stop, a);
  else if (per == 2) launch_timed(collision_scan_kernel<0, 2, 0, 1>, grid, block, s, start, stop, a);
  else if (per <= 4) launch_timed(collision_scan_kernel<0, 4, 0, 1>, grid, block, s, start, stop, a);
  else launch_timed(collision_scan_kernel<0, 8, 0, 1>, grid, block, s, start, stop, a);
  return hipGetLastError();
}

// a wavefront merges 16 partials per pass: enough wavefronts for one pass where that fits
static hipError_t launch_merge(const AttnArgs& a, int64_t heads, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  const dim3 grid((unsigned)heads);
  if (a.nranges <= 64) launch_timed(merge_partials_kernel<4>, grid, dim3(256), s, start, stop, a);
  else if (a.nranges <= 128) launch_timed(merge_partials_kernel<8>, grid, dim3(512), s, start, stop, a);
  else launch_timed(merge_partials_kernel<16>, grid, dim3(1024), s, start, stop, a);
  return hipGetLastError();
}

// Workgroups per compute unit the kernel is compiled for: three (up to 168 registers) when the
// whole grid is resident at once - there the fourth could not be used, and the looser register
// allocation measured 0.4 us faster at 32 heads x 98304 keys - and four (128 registers) when the
// workgroups come in several rounds (batch 16 x 65536 keys: 283 against 285 us, and 275 with the
// early touches, which only pay at that occupancy).
template <int KT, int WDT, int LT, int ET, bool DBG>
static void launch_scan_gather_as(const AttnArgs& a, dim3 grid, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  const dim3 block(256);
  // (any K and L: 95 to 128 registers, four workgroups fit either way.  Eight heads, bf16, spill two since the next block's
  // words are requested early; compiled for three workgroups, which spills none, or with six or seven groups in flight in
  // place of eight it measured the same within 1 % at ten shapes, 64 heads x 98304 keys, (10,300): 99.9 us, 99.5, 100.1, 100.3.)
  constexpr int kOcc = KT == 0 ? 4 : 3;
  const int G = a.Hq / a.Hkv;
  if (!DBG && G > 1 && (int64_t)grid.x * grid.y * G <= head_per_workgroup_limit(KT != 0, G))
    launch_timed(scan_gather_kernel<KT, KT == 0 ? 1 : WDT, LT, ET, false, kOcc, true>, dim3(grid.x, grid.y, (unsigned)G), block, s, start, stop, a);
  else if (KT == 0 || a.f_touch) launch_timed(scan_gather_kernel<KT, WDT, LT, ET, DBG, 4>, grid, block, s, start, stop, a);
  else launch_timed(scan_gather_kernel<KT, WDT, LT, ET, DBG, kOcc>, grid, block, s, start, stop, a);
}

template <int KT, int WDT, int LT>
static void launch_scan_gather_for(const AttnArgs& a, dim3 grid, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  constexpr int W = KT == 0 && kScanParts<KT, WDT> == 1 ? 8 : WDT;   // (debug outputs of any K and L: one form for all)
  const bool dbg = a.dbg_counts || a.dbg_cand;
  if (a.is_fp32) {
    if (dbg) launch_scan_gather_as<KT, W, LT, kFP32, true>(a, grid, s, start, stop);
    else launch_scan_gather_as<KT, WDT, LT, kFP32, false>(a, grid, s, start, stop);
  } else if (a.kv_fp8) {
    if (dbg) launch_scan_gather_as<KT, W, LT, kFP8, true>(a, grid, s, start, stop);
    else launch_scan_gather_as<KT, WDT, LT, kFP8, false>(a, grid, s, start, stop);
  } else {
    if (dbg) launch_scan_gather_as<KT, W, LT, kBF16, true>(a, grid, s, start, stop);
    else launch_scan_gather_as<KT, WDT, LT, kBF16, false>(a, grid, s, start, stop);
  }
}

static hipError_t launch_scan_gather(const AttnArgs& a, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  const dim3 grid((unsigned)a.f_nranges, (unsigned)(a.B * a.Hkv));
#define MP_TUNED(KT, LL) if (a.K == KT && a.L == LL) launch_scan_gather_for<KT, words_of(LL), tail_of(LL)>(a, grid, s, start, stop); else
  MP_TUNED_TABLES(MP_TUNED) {                              // any other: by the heads that share a KV head
    const int G = a.Hq / a.Hkv;
    if (G == 1) launch_scan_gather_for<0, 1, 0>(a, grid, s, start, stop);
    else if (G == 2) launch_scan_gather_for<0, 2, 0>(a, grid, s, start, stop);
    else if (G <= 4) launch_scan_gather_for<0, 4, 0>(a, grid, s, start, stop);
    else launch_scan_gather_for<0, 8, 0>(a, grid, s, start, stop);
  }
#undef MP_TUNED
  return hipGetLastError();
}

hipError_t launch_sampled_attention(const AttnArgs& a, const TableArgs* tables, hipStream_t s, hipEvent_t const* ev) {
  const int64_t heads = (int64_t)a.B * a.Hq;
  if (heads <= 0) return hipSuccess;
  if (a.nranges <= 0) {      // no keys: the output is defined as the zero vector
    hipLaunchKernelGGL(zero_output_kernel, dim3((unsigned)((heads * kHeadDim + 255) / 256)), dim3(256), 0, s,
                       a.out, heads * kHeadDim);
    return hipGetLastError();
  }
  hipError_t e;
  // retrieval: stream every key's code, or look the query's codes up in the hash tables and
  // stream only the codes of the keys appended since the tables were built
  if (tables) {
    AttnArgs b = a;
    b.blk_begin = key_blocks(tables->n);                 // tables->n is a.n or a multiple of the block size
    const bool lookup = tables->n > 0, scan = b.blk_begin < key_blocks(a.n);
    const int nslices = (int)((b.blk_begin + kLgSliceBlocks - 1) / kLgSliceBlocks);
    const int app_runs = (int)((key_blocks(a.n) - b.blk_begin + 15) / 16);
    // One launch for lookup, gather, the static set and the few keys appended since the build
    // pays while its workgroups (one per head and slice, one per compute unit at a time) are
    // resident all at once: it removes launches and round trips from a latency-bound step.  Beyond
    // that a second round of workgroups costs more than the launches saved (64 heads x 98304
    // keys: 42.9 against 37.9 us per step), and with many heads the step is throughput-bound:
    // separate lookup and gather launches, each filling the chip with its own kind of work,
    // measured 35-40 % faster (batch 16 x 65536 keys, batch 8 x 131072).
    const bool few = heads * nslices <= kNumCU;
    if (lookup && few && !a.dbg_counts && (a.tau == 1 || a.tau == 2) && app_runs <= nslices) {
      b.nranges = nslices * 16;
      if ((e = launch_lookup_gather(b, *tables, nslices, app_runs, s, ev ? ev[0] : nullptr, ev ? ev[1] : nullptr)) != hipSuccess)
        return e;
      if (ev && (e = hipEventRecord(ev[2], s)) != hipSuccess) return e;
      return launch_merge(b, heads, s, ev ? ev[4] : nullptr, ev ? ev[3] : nullptr);
    }
    if (lookup) {
      e = launch_table_lookup(a, *tables, s, ev ? ev[0] : nullptr, ev && !scan ? ev[1] : nullptr);
      if (e != hipSuccess) return e;
    }
    if (scan) {
      e = launch_scan(b, s, ev && !lookup ? ev[0] : nullptr, ev ? ev[1] : nullptr);
      if (e != hipSuccess) return e;
    }
  } else {
    // whole-context scan: scan and gather in one launch, then the merge over its partials
    if ((e = launch_scan_gather(a, s, ev ? ev[0] : nullptr, ev ? ev[1] : nullptr)) != hipSuccess) return e;
    if (ev && (e = hipEventRecord(ev[2], s)) != hipSuccess) return e;
    AttnArgs b = a;
    b.nranges = a.f_nranges;
    if ((e = launch_merge(b, heads, s, ev ? ev[4] : nullptr, ev ? ev[3] : nullptr)) != hipSuccess) return e;
    return hipGetLastError();
  }
  AttnArgs b = a;                                          // (no more partials than a.nranges, for which there is room)
  const int G = a.Hq / a.Hkv;
  const GatherPlan plan = plan_gather(a.B * a.Hkv, G, key_blocks(a.n), a.n_static, a.tau);
  b.g_run_blocks = plan.run_blocks;
  b.g_static_runs = plan.static_runs;
  b.g_static_keys = plan.static_keys;
  b.nranges = plan.runs + plan.static_runs;
  const dim3 grid((unsigned)b.nranges, (unsigned)(a.B * a.Hkv)), block(64 * G);
  auto gather = [&](auto kernel, int list) {
    launch_timed_lds(kernel, grid, block, (size_t)G * list * sizeof(uint16_t), s, nullptr, ev ? ev[2] : nullptr, b);
  };
  auto gather_as = [&](auto whole) {
    constexpr bool kFull = decltype(whole)::value;
    if (a.is_fp32) gather(gather_estimate_kernel<kFP32, kFull>, kGatherList<kFP32>);
    else if (a.kv_fp8) gather(gather_estimate_kernel<kFP8, kFull>, kGatherList<kFP8>);
    else gather(gather_estimate_kernel<kBF16, kFull>, kGatherList<kBF16>);
  };
  if (plan.full) gather_as(std::true_type{});
  else gather_as(std::false_type{});
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return launch_merge(b, heads, s, ev ? ev[4] : nullptr, ev ? ev[3] : nullptr);
}

}  // namespace mp
