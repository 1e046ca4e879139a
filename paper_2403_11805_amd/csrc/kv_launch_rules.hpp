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

}  // namespace kvs
