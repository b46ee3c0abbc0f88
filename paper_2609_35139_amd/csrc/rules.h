// Choices between kernels that depend on sizes alone (host code, no HIP).
#pragma once
#include <stdint.h>

namespace cr {

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

inline int64_t grid_tiles(int64_t M, int64_t N, int bm, int bn) {
  return ceil_div(M, bm) * ceil_div(N, bn);
}

// Output add (bf16): 256x256 tiles, one workgroup per CU, or the tiles of
// launch(), 128x128 ones of which two share a CU.  Compared by the time of
// their rounds over the chip, so that rows of padding count: a round of 256
// wide tiles covers what two rounds of 512 small ones do, and takes less time
// the deeper the product (its epilogue, in which nothing overlaps, costs as
// much as the loop over some 700 k, the small tiles' as much as 265).  The last
// round of many small ones overlaps the one before it, so it counts for less
// when it is ragged.  Below K = 512 the small tiles are always as fast.  Over 16
// to 8,192 rows, 15,360 to 65,536 columns and K from 128 to 2,048 the tiles not
// taken are at most 5% faster; us on 128- and 256-column ones:
//   equal rounds, 3,200 x 18,432: K = 256: 74 and 76, 512: 101 and 97,
//     1,024: 160 and 148, 2,048: 271 and 236;
//   1,920 x 18,432 (5 rounds and 3): K = 512: 63 and 70, 1,024: 108 and 107,
//     1,536: 141 and 140;  2,690 rows (7 and 4): 512: 86 and 94, 2,048: 248 and
//     230;  3,600 rows (9, ragged, and 5): 512: 110 and 117;  4,096 rows (9,
//     full, and 5): 512: 133 and 129, 1,024: 201 and 189;
//   65,536 columns, K = 1,024: 128 rows (1 and 1) 33 and 40, 320 rows (3 and 2)
//     71 and 75, 600 rows (5 and 3) 115 and 112.
inline bool expand_on_256(int64_t M, int64_t N, int K) {
  if (K < 512) return false;
  // (a grid of at most 256 small tiles runs one to a CU, on twice the waves)
  const int64_t t128 = grid_tiles(M, N, 128, 128);
  const double full = (double)t128 / 512.0;
  const double ragged = full + 0.5 + 0.5 / full, whole = (double)ceil_div(t128, 512);
  const double small = ragged < whole ? ragged : whole;
  const double wide = (double)ceil_div(grid_tiles(M, N, 256, 256), 256);
  return 2.0 * wide <= (1.01 + K / 4880.0) * small;
}

// Weights that the attention's launch brings into the last-level cache ahead
// of the products that stream them: `range` bytes of a repairer of `total`.
// Only where a repairer is larger than that cache (256 MB), since otherwise its
// weights stay there from call to call (162 MB, 57 tokens: 176 us without and
// 181 with; 82 MB: 131 and 134), and only ranges whose reading takes no longer
// than the attention leaves the chip idle: 26 MB a block pay (267 MB, 57
// tokens: 385 -> 347; 256: 445 -> 420; 1,500: 962 -> 898); 100 MB are read in
// 17 us beside an attention of 5 (57 tokens: 322 and 328, 1,200: 993 and
// 1,013), 164 MB in 28 (57: 333 and 356) and 292 MB, which the cache no longer
// holds, twice (57: 474 and 580, 1,500: 1,893 and 2,015).  Part of such a range
// gains nothing (32 of 100 MB: 57 tokens 324, 1,200 997), and ranges below 8 MB
// less than the workgroups cost (57 tokens, d_b = 512: 149 and 152).
inline bool prefetch_pays(int64_t range, int64_t total) {
  return range >= (int64_t)8 << 20 && range <= (int64_t)32 << 20 && total > (int64_t)256 << 20;
}

// ... and where the last round of the attention's workgroups (one per CU)
// leaves CUs idle, a quarter of them beside the short walks of 32-query tiles
// and one in sixteen else: there it costs the attention little or nothing
// (8 blocks of 26 MB, 200 tokens of an 8B cache 496 -> 480 us, 384 631 -> 587,
// 850 tokens, 224 workgroups, 705 -> 677, 1,177 ragged ones 898 -> 870, 10 x 512
// 3,298 -> 3,265; at worst 288 tokens, 144 workgroups of 32 queries: 482 and
// 488; 400, 208 workgroups: 520 and 527).  After a full round it is a tail of
// its own (8 x 512, 512 workgroups: attention +6 us, FFN2 -4), and over more
// than five rounds the products no longer gain (8,900 tokens, 1,120
// workgroups: 6,409 -> 6,371; 10,500, 1,328: 7,494 and 7,531; 15,000, 1,888:
// 8,302 and 8,350).
inline bool prefetch_fits(int64_t workgroups, int queries) {
  const int64_t last = workgroups % 256;
  return last > 0 && last <= (queries == 32 ? 192 : 240) && workgroups <= 1280;
}

// Attention: queries per workgroup (128 with two groups of waves splitting the
// keys, 64 or 32 with four).  A grid that leaves CUs idle, or has them all wait
// for the few workgroups of the last chunks, is bound by one workgroup's walk
// over its key tiles, so it takes shorter tiles and more key groups (16 heads
// of 64 unless said; us):
//   bf16, 32 queries while their grid fits the 256 CUs (200 tokens 6.1 -> 5.5,
//     57 tokens x 8 heads 5.1 -> 4.9 and 4 x 256 x 8 heads 9.1 -> 8.1 against
//     64-query tiles);
//   bf16, 64 queries while their grid fits the CUs (one workgroup each with
//     heads of 64, two with heads of 32: 1,024 tokens 9.4 against 12.5), and
//     until the 128-query grid does if a row has more than 512 keys (1,177
//     ragged tokens 21.9 -> 14.8, 2,500 tokens x 8 heads 24.7 -> 17.6, 4,000 37.1
//     -> 32.3; 2,000 tokens x 16 heads 21.1 -> 20.6).  Shorter walks do not repay the
//     second workgroup on a CU (2,500 tokens x 8 heads in requests of 512: 12.6
//     and 9.4, of 256: 10.5 and 7.0, of 100: 11.4 and 10.4; only unaligned
//     requests of 300 to 400 whose grid hardly exceeds the CUs would: 13.7 and
//     16.7 at 1,283 tokens);
//   fp32, 32 queries and 32-key tiles (two-slot rings of 32 KB per group) below
//     two 128-query workgroups per CU (2 x 256 tokens x 8 heads 37 -> 13.5,
//     2,048 x 8 heads 130 -> 54; at 512 workgroups, 4,096 tokens, 360 and 302).
//     From 384 on it depends on the chunks: 3,000 tokens in 512-token chunks of
//     one request 212 against 193, in two requests of one chunk 193 against 221.
inline int attention_queries(int64_t N, int n_heads, int d_head, bool fp32, int64_t max_keys) {
  const int64_t wg128 = ceil_div(N, 128) * n_heads;
  if (fp32) return wg128 < 512 ? 32 : 128;
  if (ceil_div(N, 32) * n_heads <= 256) return 32;
  if (ceil_div(N, 64) * n_heads <= (d_head == 32 ? 512 : 256)) return 64;
  return wg128 <= 256 && max_keys > 512 ? 64 : 128;
}

}  // namespace cr
