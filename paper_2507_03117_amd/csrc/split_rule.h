// Which single products take k_spmm_split (kern_split.h), and in which form.  Plain C++: no device code.
#pragma once
#include <cmath>
#include <cstdint>

namespace blast_dev {

// Workgroup ids between the token tiles of a unit (64 output rows); the ids go round the XCDs.  Eight: a unit's tiles are
// all on one XCD, whose L2 serves its weights to them.  With fewer than eight units, or a few more, that leaves most of the chip
// idle (one unit: 32 CUs for all tiles), so there the tiles of a unit follow each other, over all XCDs, each of which reads what
// little weight there is - where an XCD would have more tiles than CUs.  Eight waves, eight apart / one, microseconds: b = 64, 2 rows
// of 8 blocks, 4894 tokens 15.7 / 6.4 (streaming kernel 7.6), 3 rows of 8, 2672 tokens 11.3 / 6.1 (7.5), 11 rows of 20, 1031 tokens
// 15.4 / 11.0 (13.3); b = 128, one row of 8, 5421 tokens 21.3 / 9.1 (15.0).  Fewer tiles only read more (b = 64, 7 rows of 20, 269
// tokens 8.3 / 9.2; b = 128, 5 rows of 8, 823 tokens 8.4 / 9.0).  Eight units are spread as they are (b = 64, 8 rows of 8, 3210
// tokens 12.0 / 12.6), and from 12 on what the weights cost more is no longer always less than what was idle (equal rows, time with one
// over time with eight apart: 12 units 0.90 on average, but up to 1.15; 16, 24, 32 units 1.07, 1.11, 1.15).
constexpr int split_stride_log2(int64_t units, int64_t groups, int64_t cus) {
  return units < 12 && units != 8 && (units + 7) / 8 * 8 * groups > cus ? 0 : 3;
}

// Workgroups of a launch, those without a tile included.
constexpr int64_t split_workgroups(int64_t units, int64_t groups, int64_t cus) {
  const int64_t stride = (int64_t)1 << split_stride_log2(units, groups, cus);
  return (units + stride - 1) / stride * stride * groups;
}

// Unit (at or beyond the last: none) and token tile of workgroup `id`.
struct SplitTile {
  int unit, group;
};
constexpr SplitTile split_tile(int id, int stride_log2, int groups) {
  const int span = groups << stride_log2, turn = id / span, rem = id - turn * span;
  return SplitTile{(turn << stride_log2) + (rem & ((1 << stride_log2) - 1)), rem >> stride_log2};
}

// Waves to a tile, eight or four (the sums are the same): by the stages of the fullest row and of a row on average, and the
// workgroups per CU.  A CU takes one workgroup of eight or two of four.  Time with four over time with eight, 7200 products of 33
// to 32000 tokens, b = 64 / 128:
//   up to one per CU: fullest row of up to 4 stages 1.03 / 1.04, 5 to 12 1.07 / 1.09, 13 to 20 1.03 / 1.06, 21 to 40 0.97 / 0.98, more
//     0.91 / 0.91: eight waves are the shorter chain, until copies and not trips are what takes the time.
//   from there to 1.5: 0.67 / 0.71 at 2 stages, 0.78 / 0.79 at 8, 0.87 / 0.90 at 20, 0.95 / 0.97 at 40, 1.02 / 1.04 beyond; beyond 1.5:
//     0.69 / 0.73, 0.77 / 0.79, 0.85 / 0.87, 0.89 / 0.90, 0.93 / 0.95: eight waves leave half of the CUs a second round.
//   rows of which the fullest has 2.5 times the average, 1 to 1.5 per CU: 13 to 20 stages 1.02, 21 to 40 1.07, more 0.97; 1.5 to 2:
//     0.90, 1.01, 0.99: that row's tiles are a round of their own.
// (32 rows of 34 128-wide blocks, 257 tokens, 320 tiles: the two-matrix MLP it belongs to 62.0 us with eight, 65.8 with four.)
// Of 3400 products that are better off here than on another kernel, 118 (3 %) take more than 4 % longer than with the other form.
inline int split_form(double most, double average, double per_cu) {
  if (per_cu <= 1.0) return most <= 20.0 ? 8 : 4;
  const bool long_chain = (per_cu <= 1.75 && (most > 48.0 || (most >= 14.0 && most > 4.0 * average))) ||
                          (per_cu <= 1.5 && most >= 24.0 && most > 1.5 * average);
  return long_chain ? 8 : 4;
}

// The waves (4 or 8) of k_spmm_split (64 x 64 tiles, a row's stages dealt to the waves) for a single product that is better
// off there than on the kernel that would take it otherwise; 0 where it is not.  Microseconds, uniform masks unless said
// otherwise, bf16 output, graph replay:
//   streaming / split (the former walks a row in sequence, in one chain of sums, and leaves CUs idle while its tiles are few):
//     b = 64, 25 rows of 20 blocks, 384 tokens 17.0 / 10.6; 32 rows of 3, 512 tokens 6.6 / 5.2.  b = 128, 16 rows of 6.4, 384 / 1024
//     tokens 17.6 / 9.4, 17.9 / 15.0.  So up to 1.25 tiles per CU with 64-wide blocks (one where no wave has a whole stage), two
//     with 128-wide ones, always.  Rows that vary, as a uniform mask's do (the fullest 1.3 times the average), further, under at
//     most 1024 tokens: two per CU, three with 128-wide blocks (of 330 uniform masks none more than 4 % slower: b = 64, 32 rows of 3.2,
//     fullest 7, 700 tokens 7.1 / 6.0; 64 rows of 1, fullest 4, 450 tokens 5.1 / 4.7; b = 128, 32 rows of 3.2, 500 tokens 13.2 / 9.5;
//     but a two-matrix MLP of 1024 and 4096 features at 90 %, b = 64, whose second product has 16 rows of 6.4, 1500 tokens 17.9 / 20.2).
//     Beyond that by two estimates, fitted to 5600 products of 33 to 32000 tokens on one to six tiles per
//     CU (off by less than 3 % in the median, by 20 % at the fifth and the 95th percentile).  Equal rows are sooner better off on the
//     streaming kernel: b = 64, 56 rows of 2, 498 tokens, 448 tiles 4.5 / 4.8; 33 rows of 4.3, 841 tokens, 462 tiles 7.5 / 9.7; 74 rows
//     of 7, 323 tokens, 444 tiles 8.5 / 8.6; 82 rows of 13, 278 tokens, 410 tiles 11.2 / 11.0; b = 128, 52 rows of 5.7, 326 tokens, 624
//     tiles 12.9 / 15.3; 52 rows of 22, 261 tokens, 520 tiles 34.6 / 29.2.  A row much fuller than the others is a chain there, and
//     here one of four or eight waves: b = 64, 42 rows of 10, fullest 100, 1185 tokens, 798 tiles 53 / 25; b = 128, 47 rows of 12.8,
//     fullest 64, 332 tokens, 564 tiles 88 / 30.  Where there is no such row split has to be a tenth faster, and a fifth on narrow
//     outputs, whose tiles share no weights in an L2.  Over 6400 products, against the line by tiles alone: equal and uniform rows 2.6 %
//     less time on average, 0.8 % of them more than 4 % slower; uneven rows 16 %, 1.5 % (up to two or three tiles per CU always: 0.9 %,
//     7.7 %; 14 %, 9.1 %).
//   decode (33 to 256 tokens; it reads the matrix once per 32 tokens, in many small workgroups) / split: b = 64, 100 rows of 5, 64 /
//     100 / 160 / 256 tokens 5.2 / 5.4, 7.7 / 5.5, 9.4 / 7.6, 13.6 / 8.8; 32 rows of 13, 128 / 256 tokens 7.3 / 7.4, 10.0 / 8.4;
//     32 rows of 26, 192 tokens 9.5 / 11.3.  b = 128, 32 rows of 3.2, 64 / 100 / 256 tokens 4.1 / 5.9, 7.0 / 6.1, 13.0 / 7.7.
//     A full row among the others is dealt to four waves of each 16 of its rows by decode: b = 128, 32 rows of 4.1, one of
//     32, 64 / 160 / 256 tokens 6.8 / 14.9, 9.3 / 15.6, 12.0 / 16.1.  The two estimates were fitted to 1400 such
//     calls (uniform rows, Zipf rows, one or four full rows; 33 to 256 tokens) for the choice between them, with eight
//     waves: of the calls that they send here, none with 128-wide blocks and four with 64-wide ones are more than 5 %
//     slower than on decode.
// b: block width; nbr: block rows of the output; nnz: stored blocks, fullest: of the fullest row (0: not known); decode: whether
// the decode kernel would take it; cus: compute units.
inline int split_waves(int b, int64_t nbr, int64_t tokens, int64_t nnz, int64_t fullest, bool decode, int64_t cus) {
  if (b != 64 && b != 128) return 0;
  const int64_t units = nbr * (b / 64), groups = (tokens + 63) / 64, tiles = units * groups;
  const int64_t launched = split_workgroups(units, groups, cus);
  const bool spread = split_stride_log2(units, groups, cus) == 0;
  const double mean = (double)nnz / nbr;
  const double row = fullest > 0 ? (double)fullest : mean + 2.0 * std::sqrt(mean);  // (rows of a uniform mask vary by that)
  // stages of the fullest row, of a row on average; workgroups per CU; stages of a wave in the fullest row, of a CU
  const double most = row * (b / 64), average = mean * (b / 64), per_cu = (double)launched / cus;
  const double chain4 = std::ceil(most / 4.0), chain8 = std::ceil(most / 8.0), load = average * tiles / cus;
  const int waves = split_form(most, average, per_cu);
  if (decode) {
    if (tiles > 2 * cus) return 0;
    const double groups32 = (double)((tokens + 31) / 32), mbytes = nnz * 1e-6 * b * b * 2 * groups32;
    const double decode_units = nbr * (b / 16) * groups32 * 1e-3;
    double decode_us, split_us;
    if (b == 64) {
      decode_us = 3.30 + 0.162 * mbytes + 1.68 * decode_units + 0.149 * row / 4;
      split_us = (tiles > cus ? 3.06 : 3.68) + 1.65 * chain8 + 0.77 * load / 8;
    } else {
      decode_us = 3.33 + 0.128 * mbytes + 2.03 * decode_units + 0.291 * row / 4;
      split_us = (tiles > cus ? 5.44 : 3.86) + 1.39 * chain8 + 0.89 * load / 8;
    }
    return decode_us > split_us + 0.3 ? waves : 0;
  }
  if (tiles * 4 <= (b == 128 ? 8 : row < 8.0 ? 4 : 5) * cus) return waves;
  if (units >= 12 && tokens <= 1024 && most >= 1.3 * average && per_cu <= (b == 128 && average >= 2.0 ? 3.0 : 2.0)) return waves;
  if (per_cu > 6.0) return 0;
  const bool wide = (tokens + 255) / 256 * nbr >= 2 * cus;  // the streaming kernel's tiles, see launch_stream_c
  if (b == 128 && wide) return 0;
  const int64_t ntt = wide ? (tokens + 255) / 256 : (tokens + 127) / 128;
  const double blocks = (double)nnz * ntt / cus, items = (double)nbr * ntt / cus;
  const double stream_us = b == 128 ? 3.21 + 1.185 * row + 0.50 * blocks + 1.87 * items
                           : wide   ? 4.14 + 0.71 * row + 0.365 * blocks + 0.20 * items
                                    : 2.53 + 0.396 * row + 0.27 * blocks + 1.17 * items;
  // stages of a CU of the XCD with the fullest row, where that row's tiles are on one
  const double others = units > b / 64 ? (average * units - most * (b / 64)) / (units - b / 64) : 0.0;
  const double of_xcd = spread ? load : groups * (most + ((units + 7) / 8 - 1) * others) * 8.0 / cus;
  const double beyond = of_xcd > load ? of_xcd - load : 0.0;
  const double split_us = b == 64 ? 2.62 + 0.327 * chain4 + 0.261 * load + 0.113 * beyond + 1.21 * per_cu
                                  : 3.37 + 0.254 * chain4 + 0.269 * load + 0.127 * beyond + 1.08 * per_cu;
  const bool uneven = row > mean + 3.0 * std::sqrt(mean) + 1.0;  // (more than a uniform mask's fullest row)
  const double margin = spread ? 1.2 : uneven ? 1.0 : 1.1;
  return split_us * margin < stream_us ? waves : 0;
}

}  // namespace blast_dev
