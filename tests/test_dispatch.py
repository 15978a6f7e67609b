"""The launch rules against measured times (MI355X, 256 CUs): dispatch.h is
compiled for the host and asked which form each size takes."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2607_14557_amd", "csrc")
CXX = shutil.which("g++") or shutil.which("c++")
pytestmark = pytest.mark.skipif(CXX is None, reason="no host C++ compiler")


def _ask(tmp_path, body, rows):
    """Compile `body` (a function int answer(const long long* v)) with the rules and run it over rows of integers."""
    src = tmp_path / "ask.cpp"
    src.write_text('#include <cstdio>\n#include "dispatch.h"\nusing namespace seer;\n' + body + """
int main() {
  long long v[8];
  int n;
  while (scanf("%d", &n) == 1) {
    for (int i = 0; i < n; ++i) if (scanf("%lld", v + i) != 1) return 1;
    printf("%d\\n", answer(v));
  }
}
""")
    exe = tmp_path / "ask"
    subprocess.run([CXX, "-std=c++17", "-O1", "-Wall", "-Werror", "-I" + CSRC, str(src), "-o", str(exe)], check=True)
    text = "\n".join("%d %s" % (len(r), " ".join(str(int(x)) for x in r)) for r in rows)
    out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout.split()
    assert len(out) == len(rows)
    return [int(o) for o in out]


# heads, sequences (of equal length), rows, cached prefix of each; us with 128 queries a workgroup, with split keys
ATTENTION = [
    (32, 1, 32, 200, 9.6, 11.1), (32, 1, 128, 100, 11.8, 10.0), (32, 1, 128, 400, 17.1, 13.9),
    (32, 1, 128, 800, 23.5, 15.4), (32, 1, 256, 800, 26.7, 18.8), (32, 1, 256, 3700, 77.1, 49.5),
    (32, 4, 256, 3700, 83.1, 62.8), (32, 16, 256, 100, 11.4, 18.6), (32, 1, 320, 800, 26.4, 31.8),
    (32, 4, 384, 3700, 83.9, 105.1), (32, 8, 512, 100, 12.4, 20.2), (16, 4, 256, 400, 15.0, 12.8),
    (16, 2, 512, 100, 14.0, 13.1), (16, 1, 512, 800, 29.8, 19.5), (16, 1, 640, 3700, 79.1, 91.1),
    (16, 8, 1024, 800, 23.8, 31.3), (8, 1, 512, 200, 20.4, 15.2), (8, 3, 1024, 400, 20.6, 27.4),
    (8, 2, 1024, 3700, 78.3, 49.2), (8, 4, 1100, 100, 13.8, 20.0), (8, 1, 2048, 800, 55.9, 64.0),
    (4, 3, 1280, 1, 16.2, 14.3), (4, 1, 1536, 100, 35.9, 24.7), (4, 4, 2048, 800, 30.8, 37.2),
    (4, 1, 2048, 3700, 105.1, 61.5), (4, 4, 4096, 100, 27.3, 53.2), (4, 8, 2200, 3700, 76.8, 89.3),
]


def test_attention_form(tmp_path):
    """Splitting the keys is never the slower form, and is taken where one round of its workgroups is sure to hold
    every tile and it gains a quarter."""
    few = _ask(tmp_path, "int answer(const long long* v) { return few_attention(v[2], v[1], v[0], v[1] * v[3], 256); }",
               [r[:4] for r in ATTENTION])
    for f, (heads, batch, rows, prefix, many_us, few_us) in zip(few, ATTENTION):
        assert not f or few_us <= 1.05 * many_us, (heads, batch, rows, prefix)
        if few_us < 0.75 * many_us and heads * (rows // 32 + batch - 1) <= 256:
            assert f, (heads, batch, rows, prefix)


def test_row_tiles(tmp_path):
    """The bound on row tiles holds for every split of the rows and is reached."""
    rows = [(r, b, q) for r in (1, 2, 31, 32, 33, 64, 97, 255, 256, 1000) for b in (1, 2, 3, 7, 40) for q in (32, 128)]
    got = _ask(tmp_path, "int answer(const long long* v) { return max_row_tiles(v[0], v[1], v[2]); }", rows)
    for (r, b, q), g in zip(rows, got):
        most = min(b, r)                     # one row each, the rest in whole tiles of one sequence
        assert g == most + (r - most) // q


# N, K, rows, whether a second launch can add parts; us whole, in 128x64 tiles, in 128x128 tiles, in parts (bound:
# the rows rounded up to 256)
GEMM = [
    (12288, 4096, 97, 0, 56.0, 32.0, 35.0, None), (4096, 4096, 97, 0, 56.4, 18.7, 27.6, None),
    (24576, 4096, 97, 0, 60.9, 55.0, 50.7, None), (4096, 12288, 97, 1, 152.8, 33.7, 40.0, 43.1),
    (12288, 4096, 256, 0, 60.4, 51.3, 47.1, None), (4096, 4096, 256, 0, 59.5, 23.7, 30.1, None),
    (24576, 4096, 256, 0, 69.0, 87.5, 78.2, None), (4096, 12288, 256, 1, 157.9, 49.2, 48.0, 55.0),
    (12288, 4096, 320, 0, 56.4, 65.5, 61.0, None), (4096, 4096, 320, 0, 55.4, 28.2, 33.2, None),
    (24576, 4096, 320, 0, 75.9, 118.0, 98.3, None), (4096, 12288, 320, 1, 143.9, 67.8, 61.2, 58.2),
    (12288, 4096, 512, 0, 69.8, 81.4, 71.3, None), (4096, 4096, 512, 0, 62.4, 31.5, 37.7, None),
    (24576, 4096, 512, 0, 86.7, 156.3, 118.4, None), (4096, 12288, 512, 1, 159.7, 74.1, 64.9, 65.7),
    (12288, 4096, 640, 0, 74.7, 106.5, 82.7, None), (4096, 4096, 640, 0, 62.7, 46.4, 42.6, None),
    (4096, 12288, 640, 1, 161.4, 100.9, 101.4, 84.5), (12288, 4096, 768, 0, 81.8, 127.4, 104.2, None),
    (4096, 4096, 768, 0, 64.3, 48.9, 43.4, None), (4096, 12288, 768, 1, 161.0, 108.9, 99.7, 86.2),
    (12288, 4096, 890, 0, 84.5, 146.2, 110.8, None), (4096, 4096, 890, 0, 64.7, 52.6, 43.6, None),
    (4096, 12288, 890, 1, 163.3, 148.0, 102.6, 102.0), (12288, 4096, 1024, 0, 86.9, 154.2, 114.5, None),
    (4096, 4096, 1024, 0, 66.4, 59.5, 44.8, None), (4096, 12288, 1024, 1, 165.2, 139.3, 102.7, 108.7),
    (12288, 4096, 1137, 0, 94.7, 173.6, 141.2, None), (4096, 4096, 1137, 0, 65.2, 72.6, 71.0, None),
    (4096, 12288, 1137, 1, 164.8, 163.3, 138.6, 121.3), (12288, 4096, 1280, 0, 104.5, 189.0, 152.2, None),
    (4096, 4096, 1280, 0, 66.0, 74.6, 69.6, None), (4096, 12288, 1280, 1, 166.3, 177.1, 147.3, 124.1),
    (6144, 2048, 97, 0, 20.8, 14.9, 19.2, None), (2048, 2048, 97, 0, 23.6, 14.8, 20.4, None),
    (11264, 2048, 97, 0, 21.0, 14.4, 19.0, None), (2048, 5632, 97, 1, 50.0, 17.4, 23.8, None),
    (6144, 2048, 256, 0, 22.0, 15.2, 20.4, None), (2048, 2048, 256, 0, 24.4, 14.8, 21.2, None),
    (11264, 2048, 256, 0, 24.9, 26.8, 20.8, None), (2048, 5632, 256, 1, 51.0, 18.4, 32.6, None),
    (6144, 2048, 512, 0, 24.2, 28.4, 22.6, None), (2048, 2048, 512, 0, 25.2, 17.4, 21.7, None),
    (11264, 2048, 512, 0, 30.3, 39.7, 40.0, None), (2048, 5632, 512, 1, 52.1, 23.2, 30.3, None),
    (6144, 2048, 890, 0, 31.9, 40.1, 41.8, None), (2048, 2048, 890, 0, 25.8, 16.3, 22.8, None),
    (11264, 2048, 890, 0, 43.2, 64.3, 60.7, None), (2048, 5632, 890, 1, 54.2, 29.0, 36.4, None),
    (6144, 2048, 1280, 0, 34.6, 53.8, 45.5, None), (2048, 2048, 1280, 0, 27.0, 29.8, 23.9, None),
    (11264, 2048, 1280, 0, 50.6, 91.6, 81.6, None), (2048, 5632, 1280, 1, 55.1, 45.6, 41.9, None),
    (6144, 2048, 2048, 0, 47.9, 82.4, 68.6, None), (2048, 2048, 2048, 0, 29.3, 31.6, 27.8, None),
    (2048, 5632, 2048, 1, 58.5, 59.4, 49.1, None), (6144, 2048, 2560, 0, 54.7, 112.5, 87.6, None),
    (2048, 2048, 2560, 0, 30.4, 47.0, 44.6, None), (2048, 5632, 2560, 1, 61.6, 83.2, 76.4, None),
    (3072, 1024, 256, 0, 13.5, 10.7, 15.2, None), (1024, 1024, 256, 0, 16.2, 11.6, 16.5, None),
    (5632, 1024, 256, 0, 13.5, 10.5, 14.5, None), (1024, 2816, 256, 1, 29.9, 13.6, None, None),
    (3072, 1024, 1137, 0, 15.7, 19.0, 17.0, None), (1024, 1024, 1137, 0, 17.3, 11.6, 16.6, None),
    (5632, 1024, 1137, 0, 18.8, 34.0, 28.4, None), (1024, 2816, 1137, 1, 30.9, 18.0, None, None),
    (3072, 1024, 2560, 0, 21.5, 35.6, 31.9, None), (1024, 1024, 2560, 0, 18.5, 20.3, 18.5, None),
    (5632, 1024, 2560, 0, 30.0, 59.2, 56.3, None), (1024, 2816, 2560, 1, 32.6, 31.6, None, None),
    (3072, 1024, 3600, 0, 29.5, 52.8, 46.9, None), (1024, 1024, 3600, 0, 19.6, 21.5, 19.6, None),
    (1024, 2816, 3600, 1, 34.0, 36.3, None, None), (1536, 512, 97, 0, 9.6, 7.7, 12.0, None),
    (512, 512, 97, 0, 12.0, 8.1, 12.0, None), (2048, 512, 97, 0, 9.2, 7.8, 10.8, None),
    (512, 1024, 97, 1, 15.6, 8.8, 14.6, None), (1536, 512, 1137, 0, 10.2, 11.1, 14.0, None),
    (512, 512, 1137, 0, 12.6, 10.0, 14.1, None), (2048, 512, 1137, 0, 10.3, 14.9, 13.2, None),
    (512, 1024, 1137, 1, 16.7, 10.1, 16.3, None), (1536, 512, 3500, 0, 12.0, 21.9, 24.4, None),
    (512, 512, 3500, 0, 13.7, 10.4, 15.0, None), (2048, 512, 3500, 0, 11.8, 27.4, 22.7, None),
    (512, 1024, 3500, 1, 17.5, 11.4, 17.0, None), (1536, 512, 8000, 0, 20.3, 40.7, 35.9, None),
    (512, 512, 8000, 0, 15.3, 17.6, 17.4, None), (2048, 512, 8000, 0, 22.0, 50.9, 43.8, None),
    (512, 1024, 8000, 1, 19.2, 21.0, 19.4, None),
]
LAUNCH = "FewLaunch{(int)v[0], (int)v[1], (int)v[2], 256, true, v[3] != 0, ((size_t)64 << 20) - 4096}"
FORM = """
struct Form { int shape, parts; };
static Form form(const FewRule& r, int t) {
  for (unsigned run : r.runs.run) if (t <= few_end(run)) return {few_form(run), few_run_parts(run)};
  return {FEW_WHOLE, 0};
}
"""


def test_gemm_form(tmp_path):
    """The form taken is within 10% of the fastest measured one (kernels of 10 to 300 us that differ by 2% from run
    to run), and within 1% on average."""
    import math
    got = _ask(tmp_path, FORM + "int answer(const long long* v) { return form(few_rule(" + LAUNCH + "), (v[4] + 127) / 128).shape; }",
               [(-(-m // 256) * 256, n, k, second, m) for n, k, m, second, *_ in GEMM])
    regret = []
    for shape, (n, k, m, second, *us) in zip(got, GEMM):
        assert us[shape] is not None, (n, k, m)
        regret.append(us[shape] / min(u for u in us if u is not None))
        assert regret[-1] <= 1.10, (n, k, m, shape, us)
    assert math.exp(sum(map(math.log, regret)) / len(regret)) <= 1.01


def test_gemm_grid(tmp_path):
    """Every row count up to the bound has its units inside the grid, its sums inside the scratch, and the
    second launch covers the rows that need it."""
    body = FORM + """
int answer(const long long* v) {
  const FewLaunch g = LAUNCH;
  const FewRule r = few_rule(g);
  const int tn = g.N / 256;
  for (int m = 1; m <= g.m_ub; m += m % 128 == 0 ? 1 : (m % 128 == 1 ? 126 : 1)) {
    const int t = (m + 127) / 128;
    const Form f = form(r, t);
    long long units;
    if (f.shape == FEW_PARTS) {
      units = (long long)(m + 255) / 256 * tn * f.parts;
      if (g.K / 64 % (2 * f.parts) != 0 || (size_t)f.parts * t * 128 * g.N * 4 > g.scratch || m > r.parts_rows) return 2;
    } else if (f.shape == FEW_WHOLE) {
      units = (long long)t * tn <= g.units ? (long long)t * tn : (long long)(m + 255) / 256 * tn;
    } else {
      const int tiles = t * (g.N / (f.shape == FEW_WIDE ? 128 : 64)), full = few_full(g.units, tiles), rem = tiles - full;
      const int s = few_k_splits(g.units, rem, g.K / 64);
      units = full + (long long)rem * s;
      if (rem * s > g.units || (s > 1 && rem > 128) || (f.shape == FEW_WIDE && g.K % 512 != 0)) return 3;
    }
    if (r.n_runs > 0 && units > r.grid) return 4;
  }
  return 0;
}""".replace("LAUNCH", LAUNCH)
    rows = [(ub, n, k, s) for n, ks in ((256, (256, 512, 8192)), (512, (512, 1024, 65536)), (1024, (1024, 2816)),
                                        (4096, (4096, 8192, 12288, 16384)), (12288, (4096,)), (24576, (4096,)))
            for k in ks for s in (0, 1) for ub in (1, 97, 128, 129, 256, 640, 1024, 1280, 1500, 2304, 4096, 9000)
            if -(-ub // 256) * (n // 256) <= 256]
    for r, a in zip(rows, _ask(tmp_path, body, rows)):
        assert a == 0, (r, a)
