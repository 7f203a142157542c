// Host check of the staged operations' layout (csrc/pbz_stage_layout.h) for every kept count and index size: teams, blocks per
// tile, LDS regions and their alignment for the kernels' operand counts.  Prints "ok <layouts>" or the first failure.
#include <cstdio>
#include <initializer_list>

#include "pbz_stage_layout.h"

using namespace pbz::ops;

int main() {
  // (regions, numbers): sum, shift, one or two operands; sums and shifts of held blocks, by types and phases
  const int uses[7][2] = {{3, 2}, {2, 1}, {1, 1}, {2, 2}, {1, 0}, {2, 0}, {3, 0}};
  long layouts = 0;
  for (int bytes = 1; bytes <= 4; bytes *= 2)
    for (int kept = 1; kept <= 4096; ++kept)
      for (int target : {2048, 4096})
        for (int64_t n_blocks : {int64_t(1), int64_t(77), int64_t(5000), int64_t(1) << 20})
          for (int64_t min_waves : {int64_t(0), int64_t(4), int64_t(4096)})
            for (int team_dwords : {5, 6, 10, 12}) {       // those of the sums and shifts, and what all others take
              const Stage st = make_stage(kept, bytes, n_blocks, target, min_waves, team_dwords);
              const int team = 1 << st.team_shift, per_round = 64 / team;
              const char* bad = nullptr;
              if (st.bpb != kept * bytes || st.dwords * 4 < st.bpb || st.dwords * 4 >= st.bpb + 4) bad = "dwords";
              if (team > 64 || (team < 64 && st.dwords > team_dwords * team)) bad = "team";
              if (st.run * team < st.dwords) bad = "lanes that do not reach the block's end";
              if (st.run > team_dwords && team < 64) bad = "run";
              // held blocks: the lane's first dword is its last one only where the block has no other, and no run is longer than the block
              if (st.run <= team_dwords && (st.run > st.dwords || (st.run == 1 && st.dwords > 1))) bad = "held run";
              if (st.blocks < per_round || st.blocks % per_round || st.blocks > kMaxBlocksPerWave) bad = "blocks";
              if (st.region % 16 || st.region < 15 + st.blocks * st.bpb + 8) bad = "region";      // any phase, and a word more
              // the last word that the last lane reads of the tile's last block, `run` after the one its share starts in
              if (4 * (((15 + (st.blocks - 1) * st.bpb + 4 * (team - 1) * st.run) >> 2) + st.run) + 3 >= st.region) bad = "a read past the region";
              if (st.numbers % 16 || st.numbers < 8 * st.blocks) bad = "numbers";
              for (const auto& u : uses) {
                size_t lds;
                const int waves = waves_for(st, u[0], u[1], &lds);
                if (waves < 1 || waves > kMaxWaves || lds != size_t(waves) * wave_bytes(st, u[0], u[1])) bad = "waves";
                if (lds > size_t(kStageLds)) bad = "too much LDS";
                for (int w = 0; w < waves; ++w)
                  if (w * wave_bytes(st, u[0], u[1]) % 16) bad = "a wave's regions are not 16-byte aligned";
              }
              if (bad) {
                std::printf("%s: kept %d of %d bytes, %lld blocks, target %d, %lld waves, teams of %d dwords\n", bad, kept, bytes,
                            (long long)n_blocks, target, (long long)min_waves, team_dwords);
                return 1;
              }
              ++layouts;
            }
  std::printf("ok %ld\n", layouts);
  return 0;
}
