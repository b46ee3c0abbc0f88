// Choices between kernels that depend on sizes alone (host code, no HIP).
#pragma once
#include <stdint.h>

#include <algorithm>

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

// Key interval [lo, hi) of every attention row, as schedule_kernel derives it
// from the chunk and request offsets (mask: values of CR_MASK_*).
struct KeyIntervals {
  const int32_t* off;
  int32_t n_chunks;
  const int32_t* req;   // null: one request
  int32_t n_req;
  int mask;
  int chunk_of(int64_t t) const {
    return (int)(std::upper_bound(off, off + n_chunks + 1, t) - off) - 1;
  }
  int request_of(int chunk) const {
    return (int)(std::upper_bound(req, req + n_req + 1, chunk) - req) - 1;
  }
  int64_t lo(int64_t t) const {
    const int c = chunk_of(t);
    if (mask == 3) return off[c];
    return req ? off[req[request_of(c)]] : off[0];
  }
  int64_t hi(int64_t t) const {
    if (mask == 1) return t + 1;
    const int c = chunk_of(t);
    if (mask == 2) return req ? off[req[request_of(c) + 1]] : off[n_chunks];
    return off[c + 1];
  }
};

// Iterations that the workgroup of query tile qt spends on its 64-key tiles,
// which its `groups` groups of waves share.
inline int attention_iterations(const KeyIntervals& rows, int64_t N, int64_t qt, int queries,
                                int groups) {
  const int64_t q0 = qt * queries, q1 = (q0 + queries < N ? q0 + queries : N) - 1;
  const int64_t keys = rows.hi(q1) - rows.lo(q0) / 64 * 64;
  return (int)ceil_div(ceil_div(keys, 64), groups);
}

// Iterations of the busiest of 256 CUs over the workgroups of 64-query tiles,
// at most 512, dealt in launch order (latest tiles first, every head of a tile
// in turn): the first 256 go to a CU each, the others to the CUs that are
// done first.  A workgroup costs one iteration more than its keys.
inline int attention_chain_64(const KeyIntervals& rows, int64_t N, int n_heads) {
  int first[256], n = 0, second[256], m = 0, longest = 0;
  for (int64_t qt = ceil_div(N, 64) - 1; qt >= 0; --qt) {
    const int it = 1 + attention_iterations(rows, N, qt, 64, 4);
    for (int h = 0; h < n_heads; ++h) {
      if (n < 256) first[n++] = it;
      else if (m < 256) second[m++] = it;
    }
  }
  std::sort(first, first + n);
  for (int j = 0; j < n; ++j) longest = std::max(longest, first[j] + (j < m ? second[j] : 0));
  return longest;
}

// Attention: queries per workgroup (128 with two groups of waves splitting the
// keys, 64 or 32 with four).  A grid that leaves CUs idle, or has them all wait
// for the few workgroups of the last chunks, is bound by one workgroup's walk
// over its key tiles, so it takes shorter tiles and more key groups (16 heads
// of 64 unless said; us):
//   bf16, 32 queries while their grid fits the 256 CUs (200 tokens 6.1 -> 5.5,
//     57 tokens x 8 heads 5.1 -> 4.9 and 4 x 256 x 8 heads 9.1 -> 8.1 against
//     64-query tiles);
//   bf16, 64 queries while their grid fits the CUs (1,024 tokens 9.4 against
//     12.5);
//   bf16, 64 queries while the 128-query grid fits them, if the busiest CU then
//     has fewer iterations, counted one more per workgroup (with heads of 32,
//     where two workgroups share a CU and hide that, one more or as many): in
//     288 batches of one to six requests under every topology the tiles taken
//     are 0.4% slower than the better ones on average, 14% at worst (64-query
//     ones throughout 9%, 128-query ones throughout 12%).  On 64 and 128: 2,500
//     tokens x 8 heads in 512-token chunks of one request 17.6 and 24.7, in
//     requests of one chunk of 800 16.5 and 24.4, of 512 12.6 and 9.4, of 100
//     11.4 and 10.4; 3,374 in one request, bidirectional, 37.8 and 32.5;
//   fp32, 32 queries and 32-key tiles (two-slot rings of 32 KB per group) below
//     two 128-query workgroups per CU (2 x 256 tokens x 8 heads 37 -> 13.5,
//     2,048 x 8 heads 130 -> 54; at 512 workgroups, 4,096 tokens, 360 and 302).
//     From 384 on it depends on the chunks: 3,000 tokens in 512-token chunks of
//     one request 212 against 193, in two requests of one chunk 193 against 221.
inline int attention_queries(const KeyIntervals& rows, int64_t N, int n_heads, int d_head,
                             bool fp32) {
  const int64_t wg128 = ceil_div(N, 128) * n_heads;
  if (fp32) return wg128 < 512 ? 32 : 128;
  if (wg128 > 256) return 128;
  if (ceil_div(N, 32) * n_heads <= 256) return 32;
  if (ceil_div(N, 64) * n_heads <= 256) return 64;
  int longest = 0;
  for (int64_t qt = ceil_div(N, 128) - 1; qt >= 0; --qt)
    longest = std::max(longest, attention_iterations(rows, N, qt, 128, 2));
  return attention_chain_64(rows, N, n_heads) <= longest + (d_head == 32 ? 1 : 0) ? 64 : 128;
}

}  // namespace cr
