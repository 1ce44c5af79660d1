// Rules by which the launchers choose a form from the sizes alone, host code without the HIP runtime.
#pragma once
#include <cstdint>

namespace mp {

constexpr int kNumCU = 256;           // MI355X
constexpr int kRangeBlocks = 16;      // key blocks whose ballots a gather wavefront expands at a time (1024 keys)

// The separate gather of the table form: every head is taken by `runs` wavefronts of `run_blocks` key blocks each, and
// its static keys are dealt over them (static_runs = 0), or over static_runs wavefronts of their own, static_keys
// neighbouring ones each.  full: the form that takes full batches of rows through code of their own.
struct GatherPlan { int run_blocks, runs, static_runs, static_keys; bool full; };

// Key blocks of a gather wavefront, in pieces of kRangeBlocks.  A wavefront that takes several pieces fills its
// batches of rows (a piece samples about 20 keys of a batch's 32 at 2 %), asks for the next piece's ballots early
// and leaves one partial: as many pieces as bring all wavefronts into one round, sixteen per compute unit.
// Measured (us per step through tables, pieces 1 | 2 | 3 | 4 | 8): 512 heads x 131072 keys, (10,170), - | 181 | - | 166.5 |
// 161.8 (16: 162.5); (10,150): 512 x 32768 62.9 | 59.6 | 59.3 | 58.2 | 58.0; 128 x 65536
// 43.6 | 42.4 | 42.5 | 43.1 | 47.4; 64 x 98304 42.4 | 40.6 | 39.2 | 40.6 | 48.6; 256 x 20000, (9,120), 46.0 | 45.6 | 45.5 | 49.5 |
// 60.8; 512 x 30000, (9,100), six pieces (five runs, 1.25 workgroups per compute unit) 86.6, four 78.0.
constexpr int64_t kGatherWaves = 16 * kNumCU;
constexpr int64_t kMaxGatherPieces = 8;
// Static keys.  Up to 16 of them, half a batch, join a run's last batch.  More cost it batches of their own, one after
// the other, so they go to wavefronts of their own while the chip has room: of 32 keys, and of 64 where that leaves the
// fullest SIMD fewer wavefronts, from four on.  Measured, us per step through tables, static keys dealt over the runs |
// own wavefronts of 32 | of 64 (all of 32 contiguous keys and no full batches: the form before runs had several pieces):
// (10,150), 512 heads, 1024 keys, 68 static 25.2 | 18.8 | 19.5 (18.7), 1004 static 119 | 42.3 | 40.0 (41.8); 2048, 68 22.8 |
// 21.4 | 19.9 (20.9); 16384, 4100 147 | 133 | 113 (129); 32 heads, three hits, 16384 keys, 4100 38.2 | 22.7 | 21.5 (22.6), 528
// 18.8 | 16.8 | 17.3 (16.1); 68 16.0 | 16.4 | 16.7 (15.9).
// Where the runs fill the chip by themselves, static keys dealt over them fill their batches, and wavefronts of
// their own only pay for more than two batches per piece: 512 heads, dealt | own of 64 | of 128: 8192 keys, 516 static 36.2 |
// 37.4 | 41.5; 16384, 2004 84.4 | 73.3 | 77.1; 32768, 1092 73.3 | 73.2 | 69.8; 65536, 1004 97.5 | 105.3 | 97.6; 2504
// 141 | 147 | 135; 6004 259 | 198 | 205; (8,75), float32, 32768, 1504 280 | 455 | 313; (9,120), e4m3, 65536, 2504 126 | 161 | 138.
// Full batches through code of their own cost a wavefront that has none 0.4 us (32 heads, 16384 keys, three hits 16.5 |
// 16.0): where one piece of a run samples most of a batch at most, the form without is taken, for any threshold above one hit.
inline GatherPlan plan_gather(int units, int G, int64_t nblk, int64_t n_static, int tau) {
  const int64_t heads = (int64_t)units * G;
  int64_t pieces = (heads * ((nblk + kRangeBlocks - 1) / kRangeBlocks) + kGatherWaves - 1) / kGatherWaves;
  pieces = pieces < 1 ? 1 : (pieces > kMaxGatherPieces ? kMaxGatherPieces : pieces);
  GatherPlan p;
  p.run_blocks = (int)pieces * kRangeBlocks;
  p.runs = (int)((nblk + p.run_blocks - 1) / p.run_blocks);
  p.full = pieces > 1 || tau == 1;
  p.static_runs = 0;
  p.static_keys = 32;
  auto wavefronts = [&](int64_t per_head) {                // of the fullest SIMD
    return (units * per_head + kNumCU - 1) / kNumCU * G / 4;
  };
  auto own = [&](int keys) { return (n_static + keys - 1) / keys; };
  const bool filled = pieces > 1 || wavefronts(p.runs) >= 4;
  if (n_static <= p.runs * (filled ? 64 * pieces : 16)) return p;
  if (filled) p.static_keys = pieces > 2 ? 128 : 64;
  else if (wavefronts(p.runs + own(32)) >= 4 && wavefronts(p.runs + own(64)) < wavefronts(p.runs + own(32))) p.static_keys = 64;
  p.full |= p.static_keys > 32;
  p.static_runs = (int)own(p.static_keys);
  return p;
}

// One-launch scan + gather: most workgroups of one head each for which a workgroup serves one of the G > 1 heads of a KV
// head.  Where few workgroups share the chip a wavefront then compares its blocks with one head's code, not with G one after
// the other, and gathers for one head (of five to eight heads a wavefront gathers for two); beyond that reading the
// codes G times costs more.  tuned: table sets with a scan of their own.  us of scan + gather and merge, G heads a
// workgroup | one (workgroups of one head): G = 2, 8 KV heads, (10,150): 4096 keys 10.5 | 9.9 (256), 6144 10.5 | 10.4 (384), 8192 10.5 | 10.9 (512);
// (9,110) 8192 13.5 | 13.5 (512).  G = 3: 4096 10.6 | 10.3 (384), (8,75), float32, 5400 12.8 | 12.0 (528); step, 10000 19.2 | 20.0 (960).
// G = 4: 2048 step 19.0 | 16.7 (256), 6144 11.1 | 11.1 (768), step 10000 19.8 | 21.1 (1280); any K and L: 4096 step 20.8 | 19.5 (512), 6144
// 13.0 | 13.8 (768).  G = 5: 4096 13.9 | 10.8 (640), 6400 13.9 | 12.5 (1000), (10,100) 16.5 | 15.1; G = 6: (9,120) 5400 15.3 | 12.3 (1056);
// G = 7, 4 KV heads: 9000 14.5 | 12.2 (1008); G = 8: 4000 14.9 | 12.1 (1024), (10,100) 16.8 | 15.0, step 8000 25.2 | 26.0 (2048).
inline int64_t head_per_workgroup_limit(bool tuned, int G) {
  if (G > 4) return 4 * kNumCU;
  return (G == 4 && tuned ? 3 : (G == 2 ? 1 : 2)) * kNumCU;
}

// Float32 key hashing: keys of a workgroup, 32 or 64 (in which a projector element serves two matrix instructions), by the
// workgroups of either kind that the fullest compute unit gets: one of 64 keys takes about 1.75 times one of 32.  Below
// five bits per table 32 throughout: a workgroup is K wavefronts, and many small ones hide each other's latencies.
// us of the kernel, workgroups of 32: 32 keys | 64 keys: 257 (4,32) 11.1 | 12.5; 512 (2,32) 11.4 | 13.6; 1000 (2,64) 12.5 | 18.2; 8192 (4,100)
// 114 | 121; 282 (5,75) 15.6 | 16.0, 1002 35.7 | 25.4; 320 (10,150) 24.9 | 20.9, 515 35.1 | 39.2, 770 46.3 | 39.7, 2560 115.9 | 97.5;
// 384 (8,75) 16.9 | 16.5, 768 24.2 | 27.3, 1536 44.5 | 40.1; 640 (9,100) 35.7 | 39.0, 1272 58.8 | 57.6; 258 (16,64) 29.8 | 26.1, 750 46.2 | 50.8.
inline int hash_f32_keys(int K, int64_t groups32, int64_t groups64) {
  auto fullest = [](int64_t groups) { return (groups + kNumCU - 1) / kNumCU; };
  return K >= 5 && 7 * fullest(groups64) < 4 * fullest(groups32) ? 64 : 32;
}

}  // namespace mp
