// How launches are divided, from sizes alone: rules without a device, so that they can be looked at on the CPU.
#pragma once

#include <algorithm>
#include <cstdint>

namespace kvs {

// Splits of K (at most `most`) of a streamed GEMM of one row block (up to 32 rows) over `col_tiles` column tiles and `steps`
// steps of 16 of K.  The split with the least
//     workgroups of the busiest CU * (its rows of K + 500) + workgroups, if their products are added later
// in rows of K (some 6 ns each where a CU has one): what counts is a chip whose CUs hold equally many, one each or
// two, and not how many workgroups there are.  Fitted to splits 1..8 of the four launches of 36 layers (d_model 1024 to
// 12288, d_ff 2816 to 28672, 16 and 32 rows, weights from memory): a launch loses 0.2 us on average to its fastest split;
// as many splits as make 512 workgroups, or 640, whichever is better at the size, lose 1.5.  A layer of 16 rows in us (640
// wanted / 512 / this rule):
//   d_model 2048, d_ff 7168              72.3 /  69.1 /  65.0
//   d_model 4096, d_ff 11008            122.9 / 117.2 / 111.8     (32 rows 138.0 / 131.1 / 125.3)
//   d_model 4096, 8 kv heads, 16896     137.6 / 149.1 / 133.7     (gate | up 264 column tiles: one split leaves
//   d_model 4096, 8 kv heads, 20480     146.3 / 156.6 / 142.1      eight CUs with two workgroups, the others with one)
//   d_model 5120, 8 kv heads, 13824     157.5 / 157.2 / 138.2
//   d_model 12288, d_ff 24576           575.5 / 585.6 / 552.1
inline int64_t stream_splits(int64_t col_tiles, int64_t steps, int64_t most) {
    most = std::min<int64_t>({most, 8, steps / 16});
    int64_t best = 1, least = 0;
    for (int64_t s = 1; s <= std::max<int64_t>(most, 1); ++s) {
        const int64_t each = (steps + s - 1) / s, groups = col_tiles * ((steps + each - 1) / each);
        const int64_t cost = (groups + 255) / 256 * (each * 16 + 500) + (s > 1 ? groups : 0);
        if (s == 1 || cost < least) {
            least = cost;
            best = s;
        }
    }
    return best;
}

// Recompute attention: one or two (row block, query head) pairs per kv head go to the kernel whose wavefronts share a pair:
// a layer of 32 rows 93.2 -> 92.1 us (32 heads, d_model 4096, d_ff 512, cache from memory), 64 rows 106.1 -> 104.2; two
// query heads on each of 16 kv heads, 16 rows 73.4 -> 71.7, 32 rows 85.1 -> 83.4; on each of 8 over 32768 tokens, 32 rows
// 101.7 -> 82.8.  With three pairs reading the keys three times costs more than the idle wavefront (32 heads, 96 rows 114.7 -> 120.2).
inline bool few_pairs(int64_t pairs) { return pairs <= 2; }

// With few recomputed rows the attention kernel has too few workgroups to fill 256 CUs: the key ranges are then
// divided (at least four key tiles per share over the whole cache), as far as there is room for the shares (`most`), until
// some 512 workgroups exist (two per CU; 768 cost more in partial results than they gain: 512 rows, 32 heads, 356
// against 344 us per layer).  More than eight shares only where eight do not make 256 workgroups: 128 rows, 32 heads
// 182 us with 8, 188 with 16, 190 with 4; 4 kv heads, 16 rows 52 us with 16, 53 with 8.
// Where the wavefronts of a workgroup share a pair, 256 workgroups do (512: the same at one pair, 3 us more at two), of at
// least eight tiles, or four until 128 exist (8 heads over 1024 tokens, 32 rows: 49.5 us of four tiles, 50.2 of eight; 32
// heads over 768 80.4 and 79.7).  Up to 640 tokens dividing costs more than it gains, a launch that merges the shares: 512
// tokens, 16 heads, 16 rows 51.2 us undivided, 53.4 divided in two, 52.9 in the other kernel; two heads on each of 4 kv
// heads 42.0, 43.8, 41.9; 640 tokens, 32 heads of 64 on 16, 32 rows 50.5, 52.9, 53.7.  At 768 they are even.
inline int64_t attention_shares(int64_t pairs, int64_t n_kv_heads, int64_t tiles, int64_t most, int waves, int max_shares) {
    const bool few = few_pairs(pairs);
    const int64_t base = (few ? pairs : (pairs + waves - 1) / waves) * n_kv_heads;
    int64_t shares = (few ? 256 : 512) / base;
    if (shares > 8) shares = std::max<int64_t>(8, std::min<int64_t>(max_shares, 256 / base));
    const int64_t in_few = tiles <= 20 ? 1 : std::max<int64_t>(tiles / 8, std::min<int64_t>(tiles / 4, 128 / base));
    shares = std::min<int64_t>({shares, few ? in_few : tiles / 4, most});
    return std::max<int64_t>(shares, 1);
}

}  // namespace kvs
