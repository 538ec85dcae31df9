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

// Whether a call has so few keys that the plain-ALU kernel, a wave per query row, is the faster one; with_v: the call
// multiplies values (its waves stage two tensors).  A tile of 32 x 32 costs the matrix kernel the same however empty it is:
//   - few keys and few rows: it takes 4.7 (d = 32, without values) .. 12.3 us (d = 128, with) as one tile's chain.  The plain-ALU
//     kernel starts at 4 .. 6 us, grows with the keys of a row's chain and, from about a thousand, with the rows.  The line is
//     drawn through where the two meet: d = 128, last update: 100 frames of 8 tokens 9.1 / 13.2 us, of 12 11.3 / 13.3, of 16 level,
//     600 of 4 10.7 / 13.0, of 6 level; d = 64, fitting: 100 frames of 4 5.6 / 6.4, of 8 6.3 / 6.6; d = 32, last: 4 of 6 5.1 / 5.6;
//   - frames of so few tokens that the tiles are nearly empty, however many there are: 8000 frames of 1 token, d = 128, last
//     update 20 / 90 us, of 3 59 / 94, of 4 82 / 94, of 5 level; d = 32, fitting, of 1 9 / 18, of 2 15 / 17, of 3 level.
constexpr bool f32_few_keys(int d, bool with_v, long long problems, long long nq, long long nk) {
  const int tokens = 2 + (with_v ? 1 : 0) + (d == 128 ? 1 : 0);
  if (nq <= tokens && nk <= tokens) return true;
  const long long keys = d == 128 ? (with_v ? 25 : 17) : d == 64 ? (with_v ? 20 : 13) : (with_v ? 9 : 6);
  const long long rows = with_v ? 3200 : 2304;
  return nk < keys && problems * nq < rows && nk * rows + problems * nq * keys < keys * rows;
}

}  // namespace vm
