// The launch rules of libkvswitch behind C names, for tests/test_launch_rules.py.
#include "kv_launch_rules.hpp"

extern "C" int64_t stream_splits(int64_t col_tiles, int64_t steps, int64_t most) {
    return kvs::stream_splits(col_tiles, steps, most);
}

extern "C" int64_t attention_shares(int64_t pairs, int64_t n_kv_heads, int64_t tiles, int64_t most) {
    return kvs::attention_shares(pairs, n_kv_heads, tiles, most, 4, 16);
}
