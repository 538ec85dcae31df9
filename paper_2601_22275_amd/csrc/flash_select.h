// Which bf16 calls take which block sizes of the streaming kernels (flash2.hip, backward_mfma.hip) and the whole-frame kernel
// (frame.hip).  Plain C++, no HIP: the host test compiles it by itself.  `units`: the device's compute units.
#pragma once

namespace vm {

// Blocks of `rows` rows of `problems` problems of n rows each that the busiest compute unit gets.
constexpr long long blocks_per_unit(long long problems, long long n, int rows, int units) {
  return (problems * ((n + rows - 1) / rows) + units - 1) / units;
}

// The same as a fraction; a last block of r < rows rows counts 0.6 + 0.4 r / rows: it streams all keys for the waves that have rows.
constexpr double work_per_unit(long long problems, long long n, int rows, int units) {
  const double tail = n % rows == 0 ? 0.0 : 0.6 + 0.4 * (double)(n % rows) / rows;
  return (double)problems * ((double)(n / rows) + tail) / units;
}

// Query (owner) blocks of 128 rows, one 32-row tile per wave, or of 256, two?  The short ones hide each other's start and end
// and waste less on a ragged last block or round; the long ones read an operand from LDS for two products, which counts where the
// launch is long and the device's power is the limit.  A unit works through its blocks in groups as large as it holds, so the two
// launches' times follow from the blocks per unit, with a group's time measured against that of the long blocks' full group.  The
// constants are chosen for the least loss against the better of the two over 129 .. 470 launches a pass (8 .. 4000 problems x 129 .. 4000
// rows, random inputs with logits of deviation 3 and video-like ones).  The rule's mean loss is 0.0 .. 0.4 %, its largest 1 .. 10 %, where
// one or two blocks to a unit are near each other.
//
// A unit holds two short blocks or one long one.  A pair of short ones takes `a - b / n` of a long one's time, n the length of the loop (a
// block's start and end, which a pair shares, count less the longer the loop).  Short blocks follow the work, long ones partly go in rounds.
constexpr bool short_pairs_faster(long long problems, long long n, int units, double a, double b) {
  const double w1 = 0.5 * work_per_unit(problems, n, 128, units), w2 = work_per_unit(problems, n, 256, units);
  const double rounds = (double)blocks_per_unit(problems, n, 256, units);
  return (a - b / (double)n) * (w1 > 0.66 ? w1 : 0.66) < 0.4 * rounds + 0.6 * (w2 > 1.0 ? w2 : 1.0);
}
// A unit holds three short blocks or two long ones.  Three, two, one short ones take `three`, `two`, `one` of two long ones' time, a single
// long one 0.64.
constexpr bool short_triples_faster(long long problems, long long n, int units, double three, double two, double one) {
  const long long n1 = blocks_per_unit(problems, n, 128, units), n2 = blocks_per_unit(problems, n, 256, units);
  return three * (double)(n1 / 3) + (n1 % 3 == 2 ? two : n1 % 3 == 1 ? one : 0.0) < (double)(n2 / 2) + 0.64 * (double)(n2 % 2);
}

// R-updates of frames of b tokens.  Short / long, us: d = 64 without values 130 frames of 300 11.1 / 16.5, 252 of 2048 308 / 289; with values 16
// of 1000 20.3 / 29.3, 252 of 2048 474 / 450; d = 128 without values 130 of 300 15.0 / 29.5, 130 of 1456 158 / 176, 252 of 2048 532 / 509, with
// values 130 of 300 20.8 / 42.1, 130 of 1456 230 / 257, 252 of 2048 793 / 741.
constexpr bool update_short_blocks(int d, bool with_v, long long frames, int b, int units) {
  if (d == 64 && !with_v) return short_triples_faster(frames, b, units, 0.84, 0.6, 0.3);
  return d == 64 ? short_pairs_faster(frames, b, units, 1.07, 60.0) : short_pairs_faster(frames, b, units, 1.17, 140.0);
}

// Passes of the temporal factor over T frames.  Log-sum-exps: three short blocks to a unit or two long ones, at d = 128 level only in full
// groups; products: as many at d = 64, at d = 128 two or one.  There the last sweep's pass takes long blocks where the rows are long (short /
// long, us: 256 problems of 300 frames 29.3 / 36.7, 768 of 512 165 / 169, 512 of 2048 1343 / 1263, 400 of 3000 2150 / 1955), and the short
// ones win the fitting sweep's second pass (12 x 64 of 512 207 / 218 with the log-sum-exps, 8 x 100 of 300 110 / 150).
// (The one-tile kernel this pass ran on before took 158 and 1188 for 768 of 512 and 512 of 2048: up to 5 % less where rows fill blocks of 256
// exactly, 5 .. 30 % more elsewhere.)
constexpr bool temporal_lse_short_blocks(int d, long long problems, int T, int units) {
  return short_triples_faster(problems, T, units, d == 64 ? 0.92 : 1.04, 0.6, 0.4);
}
constexpr bool temporal_product_short_blocks(int d, bool last, long long problems, int T, int units) {
  if (d == 64) return short_triples_faster(problems, T, units, 0.92, 0.6, 0.4);
  return !last || short_pairs_faster(problems, T, units, 1.10, 80.0);
}

// The backward at d = 128, all gradients: a unit holds two short blocks or one long one, both go in rounds.  Short / long, us: 130 frames of 300
// 44 / 79, 32 of 1000 74 / 91, 130 of 1560 589 / 605, 252 of 1560 level, 252 of 2048 1807 / 1763.
constexpr bool backward_short_blocks(long long frames, int b, int units) {
  const long long n1 = blocks_per_unit(frames, b, 128, units), n2 = blocks_per_unit(frames, b, 256, units);
  return (1.02 - 20.0 / (double)b) * (double)(n1 / 2) + 0.66 * (double)(n1 % 2) < (double)n2;
}

// Key ranges for exact attention of `rows` query rows per head over n keys.  Counted in items of 256 rows, one to a compute unit: all take the
// same time, so the launch runs in ceil(items / units) rounds, and the count is the one that wastes least of the last round, after a
// charge of a few 64-key tiles' worth of time per item for its start-up and wind-down.
constexpr int exact_rows_ranges(long long heads, long long rows, long long n, int units) {
  const long long blocks = (rows + 255) / 256;
  const long long tiles = (n + 63) / 64;
  int best = 1;
  double best_score = -1.0;
  for (long long s = 1; s <= 64; ++s) {
    const long long per = (tiles + s - 1) / s;  // tiles per key range
    if (s > 1 && per < 8) break;
    if ((tiles + per - 1) / per != s) continue;  // would leave an empty range: the same as a smaller count
    const long long items = heads * blocks * s;
    const long long rounds = (items + units - 1) / units;
    const double score = (double)items / (double)(rounds * units) * (double)per / (double)(per + 6);
    if (score > best_score * 1.005) {  // prefer fewer ranges (less merge traffic) unless clearly better
      best_score = score;
      best = (int)s;
    }
  }
  return best;
}
constexpr long long exact_rows_range_keys(long long n, int ranges) { return ((n + 63) / 64 + ranges - 1) / ranges * 64; }
// Their query blocks have 128 rows instead of 256 where the items are small, for lack of keys or of rows to fill the units: their start
// and end count then, and the short blocks hide them from each other (short / long, us, ranges and partial results the same:
// d = 128: 4 heads x 400 rows x 8000 keys (16 ranges of 512) 29.9 / 36.6, 12 x 200 x 32,760 (21 of 1600) 67.2 / 67.0, 24 x 500 x 20,000
// (5 of 4032) 150.6 / 131.8; d = 64: 10 x 323 x 4199 (9 of 512) 22.2 / 23.9, 8 x 800 x 16,000 (8 of 2048) 48.8 / 48.2).
constexpr bool exact_rows_short_blocks(long long heads, long long rows, long long n, int units) {
  const int ranges = exact_rows_ranges(heads, rows, n, units);
  return exact_rows_range_keys(n, ranges) <= 1536 || 2 * heads * ((rows + 255) / 256) * ranges <= units;
}

// The longest frame that the kernel of a whole frame per workgroup takes, by sweeps of b = 32 .. 256 with 16 .. 6000 frames against the streaming
// kernel's blocks of 128 rows (us for 2000 frames, this kernel / that one).  d = 64 without values up to 160 tokens: 20.7 / 22.9 at 128, 34.2 /
// 40.4 at 160, 50.8 / 41.0 at 192; with values up to 224: 79 / 88 there, 101.6 / 96.9 at 256.  d = 128 without values up to 160: 33.2 / 38.8 at
// 128, 70.9 / 72.6 at 160, 94.5 / 81.0 at 192; with values up to 128: 63 / 72 there, 120.8 / 109.1 at 160, and up to 192 while every frame
// has a unit of its own (a seventh tile of logits spills): 130 frames of 192 13.1 / 15.1; one more frame than units costs this kernel a second
// round (192 tokens: 256 frames 17.2, 257 25.7 / 24.7, 384 29.5 / 26.4, 640 45.6 / 40.5, 2048 135 / 131).
constexpr int whole_frame_tokens(int d, bool with_v, long long frames, int units) {
  return !with_v ? 160 : d == 64 ? 224 : frames <= units ? 192 : 128;
}

}  // namespace vm
