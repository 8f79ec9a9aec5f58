// Key ranges of a bf16 attention launch: host code without any dependency, so
// that tests can compile it by itself.
#pragma once

#include <stdint.h>

namespace acid {

// Short sequences, whose workgroups would leave CUs idle, split the keys over
// the waves: d = 64 in four ranges (64 queries a workgroup) or two (128), d =
// 128 in two (128), the most that gives at most one workgroup per CU.  In one
// round it runs 1.3-1.8 times as fast (12 heads of 128: 1024 tokens 31.5 ->
// 21.4 us, 1560 44.5 -> 30.3, 2340 60.8 -> 45.1; 16 heads of 64, 1024 tokens:
// 20.6 -> 12.8); with two rounds it loses (3000 tokens 74.0 -> 98.1 us; 16
// heads of 64, 4096 tokens 86.8 -> 124.9), since a split workgroup fills its
// CU's LDS or registers alone and streams K and V for fewer queries.  Below two
// whole tiles of 64 keys there is too little to split for the merge of the
// ranges (16 heads of 64 / 128, us: 17 tokens 3.6 -> 4.8 / 5.3 -> 6.2, 64 tokens
// 3.7 -> 5.0 / 5.8 -> 6.6, 100 tokens 5.5 -> 5.8 / 8.4 -> 8.5, 128 tokens 5.6 ->
// 5.2 / 8.5 -> 8.7, 200 tokens 8.4 -> 5.9 / 13.3 -> 10.9).
inline int attn_key_ranges(int d, int64_t n_heads, int64_t L, int64_t cus) {
  auto one_round = [&](int queries) { return (L + queries - 1) / queries * n_heads <= cus; };
  if (L < 128) return 1;
  if (d == 64 && one_round(64)) return 4;
  return one_round(128) ? 2 : 1;
}

}  // namespace acid
