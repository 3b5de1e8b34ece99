"""CPU-only check of the rules that choose the backward kernels (csrc/bwd_forms.hpp), compiled with g++."""
import os
import subprocess

import pytest

from test_gpu_split import RECTANGLES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER_DIR = os.path.join(ROOT, "paper_2510_04212_amd", "csrc")

MAIN = r"""
#include "bwd_forms.hpp"
#include <cstdio>
#include <cstdlib>
// stdin: lines "kernel(0 dq, 1 dkdv) d causal grouped heads nq nk" -> form, whether that form exists
int main() {
  int k, d, c, g, h, nq, nk;
  while (scanf("%d %d %d %d %d %d %d", &k, &d, &c, &g, &h, &nq, &nk) == 7) {
    const int f = k ? dkdv_form(d, c != 0, g != 0, h, nk) : dq_form(d, c != 0, h, nq, nk);
    printf("%d %d\n", f, k ? dkdv_has_form(d, c != 0, g != 0, f) : dq_has_form(d, f));
  }
  for (k = 0; k < 2; ++k)
    for (int dd : {32, 64, 96, 128, 256})
      for (c = 0; c < 2; ++c)
        for (g = 0; g <= k; ++g)
          for (int f : {1, 2, 4, kNarrow, kHalf, kDense, 8})
            if (k ? dkdv_has_form(dd, c != 0, g != 0, f) : dq_has_form(dd, f)) printf("has %d %d %d %d %d\n", k, dd, c, g, f);
  return 0;
}
"""
NARROW, HALF, DENSE = 5, 6, 7


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("forms")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", HEADER_DIR, str(d / "main.cpp"), "-o", str(d / "main")], check=True)

    def run(cases):
        out = subprocess.run([str(d / "main")], input="\n".join(" ".join(map(str, c)) for c in cases), check=True,
                             capture_output=True, text=True).stdout.splitlines()
        return [tuple(map(int, l.split())) for l in out if not l.startswith("has")], {tuple(map(int, l.split()[1:])) for l in out if l.startswith("has")}
    return run


def test_every_compiled_form_is_used_and_every_used_one_compiled(ask):
    cases = [(k, d, c, g, h, nq, nk) for k in (0, 1) for d in (32, 64, 96, 128, 256) for c in (0, 1) for g in range(k + 1)
             for h in (1, 2, 3, 5, 8, 11, 12, 16, 24, 31, 32, 40, 48, 64, 72, 96, 128, 512) for nk in (64, 511, 512, 640, 1000, 1024, 1500, 2048, 2816, 4096)
             for nq in ({nk, 64} if k == 0 else {nk})]
    got, has = ask(cases)
    assert all(ok for _, ok in got)
    assert {c[:4] + (f,) for c, (f, _) in zip(cases, got)} == has
    # blocks of 32 rows: never more work-groups than compute units (pairs of mirrored blocks count once)
    for (k, d, c, g, h, nq, nk), (f, _) in zip(cases, got):
        if f in (8, NARROW):
            blocks = h * ((((nk if k else nq) + 127) // 128) * 4)
            assert blocks <= 256 * (2 if k and c and h % 8 else 1)


@pytest.mark.parametrize("kernel,d,causal,heads,n,form", [
    # measured: the form that stands here against the one that an earlier rule took (us)
    (0, 96, 0, 58, 640, 1), (0, 96, 0, 53, 768, 1), (0, 64, 0, 58, 640, 1),          # 23.6 : 28.3 (two groups), 27.4 : 30.8, 17.5 : 18.4
    (0, 96, 0, 54, 576, 2), (0, 96, 0, 64, 640, 2), (0, 96, 0, 18, 2048, 2),         # and where two groups stay: 50.0 : 53.2
    (0, 32, 1, 24, 1000, 4), (0, 32, 1, 26, 1000, 2), (0, 32, 1, 17, 2048, 2),       # 9.4 : 10.1; 11.2 : 11.7, 21.6 : 27.7
    (0, 128, 1, 80, 512, 1), (0, 128, 1, 20, 2048, 2),                               # 18.6 : 19.6; 47.5 : 56.8
    (0, 128, 0, 3, 3000, 4), (0, 128, 0, 8, 1024, NARROW), (0, 128, 0, 9, 1024, 2),  # 35.1 : 36.5
    (0, 96, 1, 59, 768, 1), (0, 96, 1, 48, 768, 2),                                  # 24.5 : 26.5; 16.1 : 18.5
    (1, 64, 1, 10, 640, HALF), (1, 64, 1, 22, 640, HALF), (1, 64, 1, 11, 768, 8),    # 14.4 : 16.4 (eight groups), 15.2 : 17.4; 15.6 : 16.7
    (1, 96, 0, 11, 3000, 1), (1, 96, 0, 70, 640, 1), (1, 96, 0, 17, 2048, HALF),     # 97.6 : 106.3, 30.8 : 34.7; 65.8 : 71.1
    (1, 96, 1, 18, 2688, 2), (1, 96, 1, 24, 1536, HALF), (1, 32, 1, 24, 768, 4),     # 61.2 : 66.1; 28.9 : 35.1; 9.87 : 10.22
    (1, 128, 1, 16, 1000, 4), (1, 64, 0, 400, 200, DENSE)])
def test_the_faster_form_is_taken(ask, kernel, d, causal, heads, n, form):
    assert ask([(kernel, d, causal, 0, heads, n, n)])[0][0][0] == form


def test_the_rectangles_reach_the_forms_they_name(ask):
    """The GPU test of these sizes says which kernels it is about."""
    cases = [(k, d, int(c), 0, H, nq, nk) for H, nq, nk, d, c, _, _ in RECTANGLES for k in (0, 1)]
    assert [f for f, _ in ask(cases)[0]] == [f for r in RECTANGLES for f in r[5:]]
