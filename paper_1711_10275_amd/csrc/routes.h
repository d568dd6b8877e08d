// Which of two kernels takes a call: rules on sizes and numbers of pairs alone
// (host code without HIP, so that a test can hold them against measured times).
#pragma once

#include <cstdint>

namespace sscn {

// Pooling: the table kernel (k_pool) or the walk over the pairs (k_pool_walk).
// pieces: pieces of a row (16 bytes, or one channel); 2^pb of them per
// workgroup, so that a thread takes 2^pb / 4 of the tile's 64 rows.
//
// The table kernel's threads look up all K offsets of each of their rows,
// whether the row has a pair there or not, and every column group of a tile
// writes the table again.  The walk takes K steps with a barrier after each, of
// one pair per wavefront at a time.  So the table wins while a row has a pair
// at a good part of the offsets and a thread has few rows; the measure is its
// lookups per pair and thread, with the lanes that have no piece counted in;
// many tiles hide more of them.
// Measured us, table against walk (voxelised surfaces):
//   K  pairs/row  channels          table   walk   lookups
//   8     3.9     64 fp32, 100k       9.9   38.2       4    average
//   27    1       16 fp32, 100k      10.6   18.6      27    its gradient
//   27    1       36 fp32, 100k      24.1   19.1      96    two column groups
//   27    1       13 bf16, 20k       13.7   14.3     133
//   64    1       64 fp32, 1M         297    264     128
//   64    1       13 fp32, 2k        23.8   18.9     315
//   64    1        5 fp32, 1M         136    253     205
//   125   1       64 fp32, 100k      98.2   59.1     250
//   216   1       64 fp32, 100k       359   92.2     432
//   512   1       64 fp32, 100k      1528    196    1024
//   512   61      64 fp32, 100k       177    647      17    average
//   256   5        8 bf16, 400k       230    173      51    average, 4-d
// Threads of 8 rows and more (single channels of rows of 17 and more) lose to
// the walk where few tiles leave their chain of rows bare (27 offsets, 100 bf16
// channels, 2k sites: average 48.6 against 31.4); beyond 512 workgroups (1024 of
// few offsets), with several pairs a row and one per 5 offsets, the chip is full
// and they win (27 offsets, 33 fp32 channels, 500k: 61 against 129; 4 offsets,
// one pair, 33 bf16, 100k: 15.6 against 12.5).
inline bool pool_takes_table(int K, int64_t n_pairs, int64_t n_out, int64_t tiles, int pieces, int pb) {
  const int64_t groups = (pieces + (1 << pb) - 1) >> pb;
  const double pairs = n_out > 0 ? (double)n_pairs / (double)n_out : 0.0;  // of a row
  if (pairs >= 3 && K <= 5 * pairs && tiles * groups >= (K < 16 ? 1024 : 512)) return true;
  if (pb > (K <= 27 ? 5 : 4)) return false;
  const double rows = pb > 2 ? (double)(1 << pb) / 4 : 1.0, idle = (double)(groups << pb) / pieces;
  const double lookups = K * rows * idle;
  const int most = K > 128 ? 30 : groups > 1 ? 64 : pb > 4 || K > 64 ? 90 : tiles >= 2048 ? 270 : K <= 27 ? 140 : 90;
  return lookups <= most * pairs;
}

// Per-site layers (SSC, filter size 1) of kdim channels in and ncols out: the
// per-site kernel (k_conv_point) or what runs other layers.  rows: the row-block
// kernel takes the layer.
//
// A lane walks one row, its neighbours' rows lie kdim elements apart, and each
// row is read once per 4 columns: long rows of few columns leave the loads
// scattered, which the general kernels' staged rows are not.  So: at most 1024
// weights, and rows as long as these us, per-site kernel against the other, allow:
//   fp32, 4-channel pieces  36 -> 28   500k    34   54    44 -> 4   1.96M  134  102
//                           44 -> 20   1.96M  145  179    60 -> 16  1.96M  178  132
//   single channels         33 -> 31   500k    60  101    50 -> 4   1.96M  402  198
//                           50 -> 20   1.96M  363  409    70 -> 4   500k   146   84
//                           70 -> 12   500k    63   93    33 -> 8   1.96M  175  163
//   bf16, row-block         40 -> 20   500k    25   31    80 -> 4   500k    29   28
//                           64 -> 12   500k    25   27    200 -> 4  500k    64   47
// bf16 layers of the row-block kernel also count the columns that fill a group
// of four (32 -> 25: 32 against 30 us).
// fp32 rows that the row-block kernel takes as bf16 parts (16 channels, 32 and
// more) stay there whatever their time: a multiply-add chain rounds differently
// (1e-7 of the sum), and a network's later steps amplify that where a sum close
// to zero changes its sign.  So do rows of 24 (24 -> 40: 51 us at 500k there, 75
// here in the row-block kernel's order).
inline bool point_is_faster(int elem_bytes, bool rows, int kdim, int ncols) {
  const int groups = (ncols + 3) / 4;
  if ((int64_t)kdim * ncols > 1024) return false;
  if (elem_bytes == 2 && rows) return kdim <= 64 && (int64_t)kdim * groups * 4 <= 800;
  if (elem_bytes == 4 && rows) return kdim == 8;
  if (elem_bytes == 4 && kdim % 4 == 0) return kdim <= (groups >= 5 ? 44 : 40);
  return kdim <= (groups >= 3 ? 24 : 16) * groups;
}

// Layers of kdim < 8 channels in and ncols out, K offsets: the narrow kernel
// (k_conv_narrow) or what runs other layers, within 48 KB of LDS for the weights
// and the tile's table (three workgroups a CU).
//
// The narrow kernel stages all weights for every 64 rows, whatever pairs the rows
// have; the others pay per pair, in column groups of 64.  So the weights staged
// (columns in whole fours) may be many where rows have many pairs, some where
// rows have few, and more than that only in fp32, whose matrix products are the
// dearer, when enough tiles hide the staging.  Measured us, narrow kernel against
// the other:
//   3x3x3, 11 pairs/row     4 -> 96 fp32   100k 144  285    7 -> 48 fp32  20k    48  189
//   3x3x3, 1.1 pairs/row    6 -> 64 bf16   100k 102   64    6 -> 32 bf16  20k    23   57
//     rows in random order  7 -> 48 bf16   500k 1144  694    7 -> 48 fp32  500k  555  776
//   2x2x2 down              6 -> 96 bf16   20k   38   74    1 -> 512 bf16 20k    59   41
//                           4 -> 192 fp32  20k   36   32    4 -> 192 fp32 100k   44   67
//   2x2x2 up                7 -> 128 bf16  100k  74   46    5 -> 96 fp32  100k   36   63
//   3x3x3x3, 4.6 pairs/row  4 -> 16 fp32   500k 315  158    4 -> 16 fp32  100k   79  104
inline bool narrow_is_faster(int elem_bytes, int K, int kdim, int ncols, int64_t n_pairs, int64_t n_out) {
  const int64_t weights = (int64_t)K * kdim * ((ncols + 3) / 4 * 4);
  if (kdim >= 8 || 4 * weights + 256 * (int64_t)K > 48 * 1024) return false;
  const double pairs = n_out > 0 ? (double)n_pairs / (double)n_out : 0.0;  // of a row
  const int64_t tiles = (n_out + 63) / 64;
  if (weights <= (K > 27 ? 400 : elem_bytes == 4 ? 1000 : 600) * pairs) return true;
  if (K > 27) return weights <= 6000 && tiles <= 2048;
  if (weights <= (elem_bytes == 2 && kdim == 7 ? 2000 : 3500)) return ncols <= 192 || tiles >= 400;
  if (ncols <= 96 && weights <= 5400) return elem_bytes == 4 || kdim <= 6;
  return elem_bytes == 4 && K <= 8 && tiles >= 400;
}

}  // namespace sscn
