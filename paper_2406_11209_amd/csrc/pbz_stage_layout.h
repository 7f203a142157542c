// How the staged operations (pbz_ops_staged.hip) deal blocks to waves and a workgroup's LDS to its waves.  Plain integer
// arithmetic, for the host and the kernels, and for a CPU test that goes through every kept count.
#pragma once

#include <cstddef>
#include <cstdint>

#ifdef __HIPCC__
#define PBZ_HD __host__ __device__ inline
#else
#define PBZ_HD inline
#endif

namespace pbz {
namespace ops {

constexpr int kMaxWaves = 4;             // waves per workgroup, fewer when a wave's regions are large
constexpr int kTeamDwords = 12;          // a team is the fewest lanes with at most this many dwords each (64 at most) ...
constexpr int kFewDwords = 4;            // ... or, where the launch would have fewer waves than it should, this many
constexpr int kMaxBlocksPerWave = 256;
constexpr int kStageLds = 60 * 1024;     // of a workgroup (the reductions' final sums need some, too)

struct Stage {
  int kept;         // indices per block
  int bpb;          // bytes of F per block
  int dwords;       // dwords per block, the last one possibly partial
  int team_shift;   // log2 of the lanes per block
  int run;          // consecutive dwords of a block per lane, the last lanes possibly fewer or none
  int blocks;       // blocks per wave and tile, a multiple of the blocks per round (64 lanes over the team)
  int region;       // bytes of an LDS region: a span at any phase and one word more, a multiple of 16
  int numbers;      // bytes of an LDS region for N of the tile's blocks in FP64, a multiple of 16
};

// bytes of LDS of a wave with that many operands and results.  Every region of every wave is 16-byte aligned: spans move in 16-byte
// pieces.
PBZ_HD int wave_bytes(const Stage& st, int regions, int numbers) { return regions * st.region + numbers * st.numbers; }

// `target`: bytes of a span that a wave should have in flight per operand; `min_waves`: smaller spans are taken before
// the launch falls below that many waves
inline Stage make_stage(int kept, int index_bytes, int64_t n_blocks, int target, int64_t min_waves, int team_dwords = kTeamDwords) {
  Stage st;
  st.kept = kept;
  st.bpb = kept * index_bytes;
  st.dwords = (st.bpb + 3) / 4;
  st.team_shift = 0;
  const auto run_of = [&] { return ((st.dwords - 1) >> st.team_shift) + 1; };
  while (st.team_shift < 6 && run_of() > team_dwords) ++st.team_shift;
  while (st.team_shift < 6 && run_of() > kFewDwords && (n_blocks << st.team_shift) / 64 < min_waves) ++st.team_shift;
  st.run = run_of();
  // Lanes of a large block that start a multiple of sixteen banks apart wait for each other in LDS: one dword more then.  4095 dwords, 64
  // a lane, all on one bank: sum of 2500 blocks 156 -> 86 us, block-wise covariance 58 -> 24.  (Multiples of four gain 2 %
  // and can lose a wave per workgroup to the larger region: shift of 6000 blocks of 3300 dwords 65 and 87.)
  if (st.run > kTeamDwords && st.run % 16 == 0) ++st.run;
  const int per_round = 64 >> st.team_shift;
  int rounds = target / st.bpb / per_round;
  if (rounds * per_round > kMaxBlocksPerWave) rounds = kMaxBlocksPerWave / per_round;
  while (rounds > 1 && n_blocks / (int64_t(rounds) * per_round) < min_waves) rounds >>= 1;
  if (rounds < 1) rounds = 1;
  st.blocks = rounds * per_round;
  // the last dword is cut from two whole words; lanes whose run lies beyond the block's end read it all the same
  st.region = (15 + st.blocks * st.bpb + 8 + 4 * ((st.run << st.team_shift) - st.dwords) + 15) / 16 * 16;
  st.numbers = (8 * st.blocks + 15) / 16 * 16;
  return st;
}

// waves per workgroup, and the bytes of LDS they take.  A block has at most 4096 indices of 4 bytes: three regions and N are
// below kStageLds for one wave.
inline int waves_for(const Stage& st, int regions, int numbers, size_t* lds) {
  const size_t per_wave = size_t(wave_bytes(st, regions, numbers));
  int waves = kMaxWaves;
  while (waves > 1 && per_wave * size_t(waves) > size_t(kStageLds)) waves >>= 1;
  *lds = per_wave * size_t(waves);
  return waves;
}

}  // namespace ops
}  // namespace pbz
