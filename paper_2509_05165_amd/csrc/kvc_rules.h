// Rules by which kvc_score chooses between the forms of its passes.  Plain C++, so that the host can
// check them too.
#pragma once

#include <stdint.h>

namespace kvc {

constexpr int MF_RCHUNK = 256;         // query rows of a workgroup of the query-stationary passes
constexpr int EK_KEYS = 256;           // keys of a workgroup of the key-stationary emit pass
constexpr int EK_MAX_CHUNKS = 32;      // row chunks of a head that it takes at most (a bit each)

// The K loads carry the streaming hint (which keeps a pass's partial results in L2 instead) where a
// launch reads each key once and its K is well beyond the 256 MB memory-side cache: 3/8 GiB and more.
// Below that the emit pass still finds part of what the statistics pass read, and plain loads
// are better.  Whole passes of 32 layers in us, plain / hint, by K: 32/8 heads 0.25 GiB 243 / 252,
// 0.31 347 / 348, 0.38 361 / 354, 0.5 444 / 439, 1 857 / 838, 2 1593 / 1562, 8 6371 / 6314; 16/8
// heads 0.18 GiB 163 / 183, 0.31 279 / 282, 0.38 316 / 306, 0.5 383 / 365, 2 1354 / 1251; 8/8 heads
// 0.31 GiB 258 / 262, 0.5 371 / 347.  Row chunks of a head share the reads, where plain loads
// are better at any size: 80 layers x 64k (four) 21250 / 22250, 16k per head (four) 4792 / 4856,
// ragged 4k (two) 1684 / 1708.
constexpr int64_t MF_STREAM_BYTES = int64_t(3) << 27;

// Heads of more than one row chunk take the key-stationary emit pass (bit for bit the same scores): K is
// read once, no wave works on rows that are not there, and the row chunks need no partials.  Score stage
// in us, query- / key-stationary: 28 layers 28/4 heads M = 64 (448 rows) 1 x 1500 tokens 65 / 61, 1 x 8192
// 246 / 226, 8 x 4096 946 / 919; 40/8 heads M = 128 (640) 1 x 8192 954 / 897, 8 x 4096 3662 / 3421; 80
// layers 64/8 M = 128 (1024) 8192 2551 / 2465; 32/8 M = 1024 (4096) 8192 3715 / 3586.  Two full row chunks
// have nothing to gain but the partials, and lose where K comes from memory, because a workgroup waits
// for its keys before it works on them: 32/8 M = 128 4 x 1500 500 / 486, 1 x 8192 (0.5 GiB of K) 631 / 608,
// 8 x 4096 (2 GiB) 2070 / 2142; 64/8 M = 64 80 layers 8192 (1.25 GiB) 1376 / 1370, 8 x 4096 5108 / 5292.
// One row chunk: 32/8 heads 128k tokens 2124 / 2371 (emit pass alone), 8 x 4096 M = 64 1177 / 1269.
//
// Where the launch leaves compute units idle it is the length of one workgroup that counts: all rows of
// a head, 64 at a time, by 256 keys, against at most 256 rows, 128 of the sequence's keys at a time, and the
// finish that joins the partials of hkv * row_chunks rows.  One layer: 8/1 heads M = 256 (2048 rows) 100
// tokens 24.3 / 49.0, 600 36.6 / 57.0, 1500 61.3 / 70.1, 4096 75.7 / 77.6; 28/4 M = 256 (1792) 300 33.4 / 49.2, 1500 66.7 / 66.6;
// 64/8 M = 128 (1024) 300 33.8 / 37.2, 600 42.1 / 41.5; 40/8 M = 64 (320, a short last row chunk) 100 25.4 /
// 22.3.  With a workgroup for most of the compute units the
// order is as above: 2048 rows 200 tokens 32/8 heads M = 512 16 layers (128 workgroups) 75.6 / 71.2, 28 layers 100
// tokens 86.9 / 77.5; but 16 layers 100 tokens 60.1 / 64.1.  More than 2048 rows: 28/4 heads M = 1024 (7168 rows) 28 layers x
// 300 tokens (224 workgroups) 226 / 245.  Over 2892 shapes of 257..8192 rows, 1..80 layers, 1..16 KV heads, 40..8192 tokens
// the choice costs 0.2 % on average against the better pass of each, where the first alone costs 7.9 %, the second 7.4 %.
//
// Heads of one row chunk take it where sequences are short, so that the workgroups of the other have next to
// nothing to do (32 layers 32/8 heads M = 32 1 x 200 tokens 28.5 / 24.0, 64 x 100 701 / 562, 1 x 512 34.8 / 32.4; but
// 16 x 300 at M = 64 309 / 335), and where their rows leave waves without work (5 to 7 blocks of 32) as long as K
// comes out of the cache (28/4 heads M = 32 1 x 1500 66 / 54, 1 x 9000 179 / 165, 4 x 20000 1158 / 1197; 40/8 1 x 2500
// 182 / 148).
//
// workgroups: of the key-stationary pass, over all sequences, heads and layers.
inline bool emit_by_keys(int rows_head, int hkv, int64_t k_bytes, int64_t workgroups, int64_t max_seqlen) {
  if (rows_head <= MF_RCHUNK) {
    const int blocks = rows_head / 32;
    return max_seqlen <= EK_KEYS || (max_seqlen <= 2 * EK_KEYS && workgroups <= 1536) ||
           (blocks > 4 && blocks < 8 && k_bytes < MF_STREAM_BYTES);
  }
  if (rows_head > MF_RCHUNK * EK_MAX_CHUNKS) return false;
  if (rows_head > 8 * MF_RCHUNK) return workgroups >= 512;
  if (rows_head == 2 * MF_RCHUNK && k_bytes >= int64_t(5) << 27) return false;
  const int left = rows_head % MF_RCHUNK, full = rows_head / MF_RCHUNK, joined = full - (left == 0);
  // in keys: what the partials cost that are joined, and the workgroups of a short last row chunk
  const int64_t saved = 16 * (int64_t(hkv) * joined + (hkv < 8 ? hkv : 8)) - 32 + (left > 0 && left <= 128 ? 128 : 0);
  return max_seqlen + saved >= rows_head ||
         workgroups >= (max_seqlen > EK_KEYS / 2 && max_seqlen <= EK_KEYS ? 128 : 192);
}

// Sequences of unequal lengths: the longest workgroups first, whatever their sequence, so that
// long ones are neither left over at the end nor paired with short ones.  Score stage in us, sequence by
// sequence / longest first: 16 x 150..4096 tokens 32/8 heads M = 32 1055 / 900, M = 64 1553 / 1303, M = 128
// 2856 / 2469, 28/4 heads M = 64 1152 / 1041, 40/8 heads 2491 / 2194; 32 x 100..1500 M = 64 1299 / 1054;
// 2 x 1000..3000 191 / 153.  Where most workgroups have a whole chunk the row chunks of a slice of
// K no longer run side by side, which costs more than the order gives: 3 x 5000..20000 M = 128 32/8 heads
// 2752 / 2854, 40/8 4238 / 4302; with one row chunk there is nothing to lose (M = 64 1499 / 1448, 8 x 4096..
// 32768 5288 / 5243).
//
// The order costs a workgroup some 0.5 us before its first load.  That is lost where every workgroup has a
// compute unit to itself, and where they are equally long: 6/2 heads M = 32 130 + 597 tokens 25.5 / 27.5, 16 layers of
// 16/8 42 + 136 14.4 / 15.4, 8/8 M = 256 46..70 (one tile each) 22.7 / 25.2, 28 layers of 28/4 M = 512 26..66 169 / 181.
// Equally long ones still gain in batches of many sequences, because no workgroup looks for its own: 16 short
// sequences, 8/1 heads M = 512 32768 workgroups 1250 / 1161, M = 64 1024 45.5 / 42.3.  Over 924 ragged batches of 2..16
// sequences the choice costs 0.3 % on average against the better order of each, where the order always costs 2.0 %, never 5.6 %.
//
// whole: whole chunks of the batch, last: sequences that end in a shorter one; longest, shortest: workgroups in
// tiles of keys.
inline bool longest_first(int64_t workgroups, int row_chunks, int whole, int last, int longest, int shortest) {
  if (last == 0 || workgroups <= 256 || workgroups >= int64_t(1) << 31) return false;
  if (longest == shortest && last < 12) return false;
  return whole == 0 || row_chunks == 1 || whole <= last;
}

}  // namespace kvc
