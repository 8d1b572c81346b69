"""The host rules of the convolution launches (csrc/conv_rules.h), compiled with the host compiler and checked without a GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def compiled(tmp_path, body):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text('#include "conv_rules.h"\n#include <cstdio>\n#include <cstdlib>\nusing namespace cd;\n' + body)
    subprocess.run(["g++", "-std=c++17", "-O0", "-Wall", "-I", os.path.join(ROOT, "paper_2010_02838_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    return lambda *args: subprocess.run([str(exe)] + [str(a) for a in args], check=True, capture_output=True, text=True).stdout


@pytest.fixture(scope="module")
def split_rows(tmp_path_factory):
    """(splits, end of the rows the splits take one after the other, whether each is a whole number of 64-row steps)"""
    run = compiled(tmp_path_factory.mktemp("splits"), """
int main(int, char** v) {
  const long long M = atoll(v[1]);
  const GenericWgradPlan p = generic_wgrad_plan(M, atoi(v[2]), atoi(v[3]), atoi(v[4]) != 0, (size_t)atoll(v[5]));
  long long at = 0;
  for (long long s = 0; s < p.splits; s++) {   // the kernel's 32-bit arithmetic
    const int mbeg = (int)s * p.m_per_split, mend = generic_split_end((int)M, mbeg, p.m_per_split);
    if (mbeg != at || mend <= mbeg) break;
    at = mend;
  }
  printf("%lld %lld %d", p.splits, at, p.m_per_split % 64 == 0);
}
""")
    return lambda *a: tuple(int(t) for t in run(*a).split())


@pytest.mark.parametrize("M", [1, 63, 64, 65, 127, 128, 129, 4097, 98304, 2 ** 24 + 1, 2 ** 30 - 63, 2147475456, 2 ** 31 - 49151, 2 ** 31 - 257])
@pytest.mark.parametrize("N,K,v4", [(1, 9, 0), (1, 27, 0), (16, 144, 1), (33, 45, 0), (320, 180, 1), (4100, 1025, 0)])
@pytest.mark.parametrize("scratch", [128 << 20, 1 << 10])
def test_generic_weight_gradient_splits_take_every_row_once(split_rows, M, N, K, v4, scratch):
    splits, end, whole = split_rows(M, N, K, v4, scratch)
    assert end == M and whole
    assert splits == 1 or splits * N * K * 4 <= scratch
