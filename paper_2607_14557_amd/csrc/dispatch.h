// Which form a launch takes, from the sizes that the host knows.  Plain C++: no
// device code, so that the rules can be held to measured times on any machine.
#pragma once

namespace seer {

// ---- bf16 attention ---------------------------------------------------------

// The most tiles of `qt` rows that `rows` rows in `batch` sequences can make.
inline int max_row_tiles(int rows, int batch, int qt) {
  return rows >= batch ? (rows - batch) / qt + batch : rows;
}

// Queries of a workgroup of the split-key form.
constexpr int kFewQueries = 32;

// Whether the attention splits the keys over the waves of 32-query workgroups
// (attn_few_bf16_kernel) instead of walking them in 128-query ones.  Its
// workgroups hold 128 KiB of LDS, one a CU, and load K and V four times as often:
// it pays while one round holds them all, whatever the lengths (8 heads, 3700
// cached keys: 49 against 78 us at 1024 rows in two sequences; 64 against 56 at
// 2048, where they need two rounds), and while there are keys to split (4
// sequences of 64 rows and 100 cached keys, 32 heads: 12.0 against 10.2).
inline bool few_attention(int rows_ub, int batch, int heads, int kv_rows_ub, int cus) {
  const long long groups = (long long)max_row_tiles(rows_ub, batch, kFewQueries) * heads;
  const long long keys = ((long long)rows_ub + kv_rows_ub) / batch;     // of a sequence, on average
  return groups <= cus && keys >= 320;
}

}  // namespace seer
