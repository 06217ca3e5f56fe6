// The walk of a lane over a tile's output chunks (ChunkWalk), on the host: every chunk of the tile is where it should be, and
// no lane, past the tile's end or not, looks outside the period of the gather table.
#include <cstdio>

#include "thk_prune_device.h"

int main() {
  using namespace thk;
  for (int vec = 4; vec <= 8; vec += 4)   // elements of a 16-byte chunk: fp32, bf16
    for (int ld = 1; ld <= kD; ++ld)
      for (int c_lo = 0; c_lo <= 1; ++c_lo)
        for (int lane = 0; lane < kWave; ++lane) {
          const int cpp = 8 * ld / vec;
          ChunkWalk at(c_lo + lane, cpp);
          for (int i = 0; c_lo + i * kWave < 4 * cpp; ++i, at.next()) {
            const int c = c_lo + lane + i * kWave;
            const bool there = c < 4 * cpp ? at.block * cpp + at.entry == c : at.block > 3;
            if (at.entry < 0 || at.entry >= cpp || !there) {
              std::printf("%d elements a chunk, ld %d, lane %d, chunk %d: block %d, entry %d of %d\n", vec, ld, lane, c, at.block, at.entry, cpp);
              return 1;
            }
          }
        }
  std::puts("chunk walk ok");
  return 0;
}
