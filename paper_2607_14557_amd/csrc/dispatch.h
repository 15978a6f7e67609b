// Which form a launch takes, from the sizes that the host knows.  Plain C++: no
// device code, so that the rules can be held to measured times on any machine.
#pragma once

#include <stddef.h>

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

// ---- bf16 GEMM of few tiles -------------------------------------------------

// The forms of a launch whose 256x256 tiles (of the rows bound) fill at most one
// round of the CUs:
//   FEW_NARROW, FEW_WIDE  128x64 and 128x128 tiles, K split over the waves of a
//                         workgroup and over few_k_splits workgroups (few_tile)
//   FEW_PARTS             256x256 tiles, K split over workgroups that leave fp32
//                         sums, added by a second launch
//   FEW_WHOLE             256x256 tiles and halves
enum FewShape { FEW_WHOLE, FEW_NARROW, FEW_WIDE, FEW_PARTS };

// The tiles that run whole in full rounds; the others are the last round's, K split.
constexpr int few_full(int units, int tiles) { return tiles > units ? tiles / units * units : 0; }

// K splits of a tile so that `tiles` tiles of 64-wide K tiles fill one round.
constexpr int few_k_splits(int units, int tiles, int ktiles) {
  if (tiles == 0) return 1;
  int s = units / tiles;
  s = s < ktiles / 8 ? s : ktiles / 8;
  return s < 1 ? 1 : (s > 16 ? 16 : s);
}

// The form by the number of 128-row tiles, which the kernel reads on the device:
// up to the first run's end its shape, and so on, FEW_WHOLE past the last.  A run
// is one word, so that the kernel has the rule with one scalar load.
constexpr int kFewRuns = 8;
struct FewRuns {
  unsigned run[kFewRuns];            // end << 16 | k_split << 12 | parts << 4 | shape
};
constexpr int few_end(unsigned run) { return (int)(run >> 16); }
constexpr int few_form(unsigned run) { return (int)(run & 15); }
constexpr int few_run_parts(unsigned run) { return (int)(run >> 4 & 255); }     // FEW_PARTS: K splits of a tile
constexpr bool few_run_splits(unsigned run) { return (run >> 12 & 1) != 0; }    // whether few_k_splits applies

struct FewRule {
  FewRuns runs;
  int n_runs;
  int grid;              // the most workgroups that any row count up to the bound has
  int parts_rows;        // rows that the second launch has to cover, 0 for none
};

struct FewLaunch {
  int m_ub, N, K;
  int units;             // workgroups that run at once
  bool k_split;          // scratch and counters for few_k_splits
  bool parts;            // the epilogue has a second launch
  size_t scratch;        // bytes for its sums
};

// K splits of FEW_PARTS: the most whose units fit one round and their sums (of
// whole 128-row tiles) the scratch, each of an even number of 64-wide K tiles
// (the loop's unroll); 0 for fewer than three, where two gain nothing over halves,
// and for a K below 8192, where the second launch costs more than the parts save
// (K = 5632, N = 2048, 1280 rows: 48.9 against 41.9 us in 128x128 tiles; K = 12288,
// N = 4096, 640 rows: 84.5 against 101).
inline int few_parts(const FewLaunch& g, int row_tiles) {
  if (!g.parts || g.K < 8192) return 0;
  const int ktiles = g.K / 64;
  int s = g.units / ((row_tiles + 1) / 2 * (g.N / 256));
  s = s < 16 ? s : 16;
  while (s > 2 && (ktiles % (2 * s) != 0 || (size_t)s * row_tiles * 128 * g.N * 4 > g.scratch)) --s;
  return s > 2 ? s : 0;
}

// Expected us of a form at `row_tiles` row tiles, below 0 where it doesn't apply:
// fits to the measured times of each form alone, 97 to 12,000 rows, d_model 512 to
// 4096 (rms 10, 11, 16 and 6%).  128x64 tiles are left to one round and 128x128
// ones to two: more never paid (2048 rows at N = K = 2048: 28 us in one round of
// 128x128 tiles, 32 in two of 128x64 ones, 29 whole).
inline double few_us(const FewLaunch& g, int shape, int row_tiles) {
  const double k = g.K / 4096.0, weights = 2.0 * g.N * g.K;
  if (shape == FEW_NARROW || shape == FEW_WIDE) {
    const bool wide = shape == FEW_WIDE;
    const int tiles = row_tiles * (g.N / (wide ? 128 : 64));
    // the 128x128 loop takes two K tiles a wave
    if (tiles > (wide ? 2 : 1) * g.units || (wide && g.K % 512 != 0)) return -1.0;
    const int full = few_full(g.units, tiles), rem = tiles - full;
    const int s = g.k_split ? few_k_splits(g.units, rem, g.K / 64) : 1;
    const double round = (wide ? 29.3 : 20.8) * k;
    double us = rem > 0 ? round : 0.0;
    if (rem > 0 && s > 1) us = round / s + (wide ? 9.9 + 0.66 * s : 5.2 + 0.16 * s);
    if (full > 0) us = 1.1 * (us + round * (full / g.units));
    return (wide ? 9.4 : 6.0) + (us > weights / 5.0e6 ? us : weights / 5.0e6);
  }
  if (shape == FEW_PARTS) {
    const int s = few_parts(g, row_tiles);
    if (s == 0) return -1.0;
    return 10.0 + 88.6 * k / s + 0.16 * s * (128.0 * row_tiles) * g.N * 8e-6;
  }
  const int tn = g.N / 256;
  const int full = row_tiles / 2 * tn, half = row_tiles % 2 ? tn : 0;   // tiles; half tiles of a short last row
  const bool halves = 2 * full + half <= g.units;
  const double us = halves ? 47.3 * k : 89.1 * k * ((full + g.units - 1) / g.units);
  return 5.8 + (us > weights / 4.0e6 ? us : weights / 4.0e6);
}

inline FewRule few_rule(const FewLaunch& g) {
  FewRule r{};
  const int tn = g.N / 256;
  const int last = (g.m_ub + 127) / 128;
  // past two rounds of 128x128 tiles only whole tiles are left
  int lim = g.units / tn + 1;
  lim = lim < last ? lim : last;
  auto best = [&](int t, bool parts) {
    int shape = FEW_WHOLE;
    double us = few_us(g, FEW_WHOLE, t);
    for (int f = FEW_NARROW; f <= FEW_PARTS; ++f) {
      const double v = f == FEW_PARTS && !parts ? -1.0 : few_us(g, f, t);
      if (v >= 0.0 && v < us) { us = v; shape = f; }
    }
    return shape;
  };
  // Every row count waits for the second launch, in vain where its form has none
  // (5 us), so parts are for a bound that takes them itself and row counts within
  // two row tiles of it.
  const bool parts = best(last, true) == FEW_PARTS;
  // whole tiles: tiles of 128 rows while they fit as halves, else of 256
  const int whole = (last + 1) / 2 * tn;
  int most = last * tn <= g.units ? last * tn : (g.units / tn) * tn;
  most = most > whole ? most : whole;
  int used = 0, prev = -1;
  for (int t = 1; t <= lim; ++t) {
    const int shape = best(t, parts && t >= last - 1);
    int p = 0, u = 0;
    if (shape == FEW_PARTS) {
      p = few_parts(g, t);
      u = (t + 1) / 2 * tn * p;
      r.parts_rows = 128 * t;
    } else if (shape != FEW_WHOLE) {
      const int tiles = t * (g.N / (shape == FEW_WIDE ? 128 : 64)), full = few_full(g.units, tiles);
      u = full + (tiles - full) * (g.k_split ? few_k_splits(g.units, tiles - full, g.K / 64) : 1);
    }
    const int key = p << 4 | shape;
    if (key != prev) {
      if (used == kFewRuns) break;                   // the rest runs whole
      ++used;
      prev = key;
    }
    r.runs.run[used - 1] = (unsigned)t << 16 | (g.k_split ? 1u : 0u) << 12 | (unsigned)key;
    if (shape != FEW_WHOLE) r.n_runs = used;         // whole runs at the end need no word
    most = u > most ? u : most;
  }
  // Asking on the device costs whole tiles 1 to 1.5 us (1068 rows, d 4096, QKV: 93.8
  // against 95.4): not where only rows below a quarter of the bound gain by it.
  if (r.n_runs > 0 && last > 4 * few_end(r.runs.run[r.n_runs - 1])) r.n_runs = 0;
  for (int i = r.n_runs; i < kFewRuns; ++i) r.runs.run[i] = 0;
  r.grid = most;
  return r;
}

}  // namespace seer
