// Which of two kernels a call takes, where that depends on sizes alone: plain
// host functions, so that the rules can be looked at without a GPU.
#pragma once

#include <cstdint>

namespace mgc {

constexpr int64_t route_ceil(int64_t a, int64_t b) { return (a + b - 1) / b; }

// 3-axis levels of fewer fine points use the tiled kernels: there are too few
// wavefronts of columns to fill the chip, each a serial chain of planes.
// Decomposition in FP64: 129^3 26 us (tiled 18), 75 x 100 x 125 with many escaped
// values 42 (32), 150 x 200 x 250 50 (69), 257^3 59 (94).  Restriction of
// coefficients: 129^3 22 us (18), 150 x 200 x 250 with many escaped values 167
// (87), 257^3 34 (55).
constexpr int64_t kDecColsMin = int64_t(1) << 22, kRecColsMin = int64_t(1) << 24;
constexpr int kColX = 62;                   // coarse columns of a wavefront along x
constexpr int kColY = 4, kDecColY = 2;      // its coarse rows: restriction, decomposition

// Decomposition of a 3-axis level by columns of wavefronts (else tiled).  A
// wavefront takes 62 columns whatever the contiguous axis holds, a tile 16 (FP32
// input) or 8 (FP64), so an axis of few values leaves the wavefront's lanes idle.
// Over 55 sizes a type, 5 to 513 values along x and 4 to 36 million points,
// columns take about 1.1 ns a step (62 columns x 2 rows of one coarse plane) and
// 10 us to get going, tiles about 18 ns (FP32) and 7 to 8 ns (FP64) each.  Columns against
// tiles, us: 513 x 513 x 17 63 / 52 and FP64 65 / 45; 1025 x 1025 x 17 163 / 165
// and 174 / 148; 513 x 513 x 33 61 / 91 and 66 / 64; 1449 x 1449 x 5 289 / 309
// and 311 / 141; 509 x 509 x 65 51 / 122 and 59 / 95.  The rule takes the faster
// one but for at most 1 % (FP32) and 7 % (FP64).  (The restriction's columns have
// no such side: 2897 x 2897 x 3 591 / 616, 1025 x 1025 x 17 105 / 167.)
constexpr bool dec_takes_columns(const int64_t (&nf)[3], const int64_t (&nc)[3], bool f32) {
  if (nf[0] * nf[1] * nf[2] < kDecColsMin) return false;
  const int64_t steps = route_ceil(nc[2], kColX) * route_ceil(nc[1], kDecColY) * nc[0];
  const int64_t tiles = route_ceil(nc[0], 4) * route_ceil(nc[1], 8) * route_ceil(nc[2], f32 ? 16 : 8);
  return f32 ? steps + 9000 <= 17 * tiles : steps + 6000 <= 6 * tiles;
}

// 2-axis levels streamed along the rows (else tiled).  With fewer fine points a
// streamed column's steps are a serial chain (decomposition of 2049^2 26 us
// streamed, 24 tiled; 4097^2 53 and 78; the restriction of recomposition 18 and
// 23 us, 33 and 78).  A block takes 254 columns whatever the contiguous axis
// holds, a tile 32, so a row needs four tiles (decomposition) or two (restriction)
// to keep enough of them busy.  Streamed against tiled, us: decomposition of
// 130,000 x 65 95 / 66, 66,000 x 129 57 / 51, 33,000 x 257 36 / 45, 16,384 x 513
// 40 / 41; restriction of 123,362 x 34 51 / 40, 64,000 x 40 31 / 24, 64,528 x 65
// 32 / 42, 65,027 x 129 34 / 59.
constexpr int64_t kStream2MinPoints = int64_t(1) << 23, kRecStream2MinPoints = int64_t(1) << 22;
constexpr bool dec_streams_rows(const int64_t (&nf)[3], const int64_t (&nc)[3]) {
  return nf[1] * nf[2] >= kStream2MinPoints && nc[2] > 3 * 32;
}
constexpr bool rec_streams_rows(const int64_t (&nf)[3], const int64_t (&nc)[3]) {
  return nf[1] * nf[2] >= kRecStream2MinPoints && nc[2] > 32;
}

// Codebooks of a batch with their leaf sorts and canonical codes on many blocks
// (else one workgroup an array for everything).  One workgroup each takes as long
// as the largest codebook, however many there are; the many blocks take that out
// but cost 1.8 to 2.5 us an array.  How many arrays that is worth grows with the
// codes there can be, known here by the largest array's values.  Many blocks
// against one each, us, for smooth / rough fields: 64 arrays of 17^3 177 / 178
// against 69 / 69, 24 of 33^3 145 / 150 against 138 / 169, 48 of 65^3 229 / 249
// against 199 / 289, 64 of 129^3 315 / 367 against 248 / 473, 64 of 257^3 397 /
// 441 against 460 / 642; 48 arrays of 33^3 to 257^3 350 against 540.
constexpr int kSpreadBatchMax = 96;
constexpr bool batch_spreads_codebooks(int arrays, int64_t most_values) {
  int bits = -1;  // floor(log2(most_values))
  for (int64_t v = most_values; v > 0; v >>= 1) ++bits;
  const int limit = 8 * (bits - 12);
  return arrays <= (limit < kSpreadBatchMax ? limit : kSpreadBatchMax);
}

}  // namespace mgc
