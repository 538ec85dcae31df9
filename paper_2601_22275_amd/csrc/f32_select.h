// Which float32 calls the matrix-core kernels of f32.hip take.  Plain C++, no HIP: the host test compiles it by itself.
#pragma once

namespace vm {

constexpr int kF32Tile = 32;   // query rows of a tile, keys of a tile
constexpr int kF32Waves = 4;   // waves (and, one wave to a query tile, query tiles) of a workgroup

// A launch counts its threads per dimension in 32 bits.
constexpr bool grid_fits(long long blocks, int threads) { return blocks >= 1 && blocks <= 0xffffffffLL / threads; }

// Query tiles of `problems` x `nq` rows, one wave each, dealt to the 8 XCDs: the largest grid of the blocked-softmax kernel.
constexpr bool f32_attend_fits(long long problems, long long nq) {
  const long long tiles = problems * ((nq + kF32Tile - 1) / kF32Tile);
  const long long groups = (tiles + kF32Waves - 1) / kF32Waves;
  return tiles <= 0x3fffffffLL && grid_fits((groups + 7) / 8 * 8, 64 * kF32Waves);
}

}  // namespace vm
