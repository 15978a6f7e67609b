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
    src.write_text('#include <cstdio>\n#include "dispatch.h"\nusing namespace seer;\n%s\n'
                   "int main() { long long v[8]; int n;\n"
                   '  while (scanf("%%d", &n) == 1) { for (int i = 0; i < n; ++i) if (scanf("%%lld", v + i) != 1) return 1;\n'
                   '    printf("%%d\\n", answer(v)); } return 0; }\n' % body)
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
