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


@pytest.mark.parametrize("M", [1, 63, 64, 65, 127, 128, 129, 256, 257, 4097, 98304, 2 ** 24 + 1, 2 ** 30 - 63, 2147475456, 2 ** 31 - 49151, 2 ** 31 - 257])
@pytest.mark.parametrize("N,K,v4", [(1, 9, 0), (1, 27, 0), (16, 144, 1), (33, 45, 0), (320, 180, 1), (4100, 1025, 0)])
@pytest.mark.parametrize("scratch", [128 << 20, 1 << 10])
def test_generic_weight_gradient_splits_take_every_row_once(split_rows, M, N, K, v4, scratch):
    splits, end, whole = split_rows(M, N, K, v4, scratch)
    assert end == M and whole
    assert splits == 1 or (M > 256 and splits * N * K * 4 <= scratch)


@pytest.fixture(scope="module")
def generic_fits(tmp_path_factory):
    """whether conv_generic.hip takes a convolution, and the threads along x and blocks along y its launches would have at most"""
    run = compiled(tmp_path_factory.mktemp("fits"), """
int main(int, char** v) {
  long long a[11];
  for (int i = 0; i < 11; i++) a[i] = atoll(v[1 + i]);
  const long long M = a[0] * a[4] * a[5], Min = a[0] * a[1] * a[2], K = a[7] * a[8] * a[3];
  const bool ok = generic_conv_fits(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10]);
  long long x = ((M > Min ? M : Min) + 63) / 64, y = ((a[3] > a[6] ? a[3] : a[6]) + 63) / 64;
  if (ok) {
    const GenericWgradPlan p = generic_wgrad_plan(M, (int)a[6], (int)K, false, 128u << 20);
    if (p.tiles * p.splits > x) x = p.tiles * p.splits;
  }
  printf("%d %lld %lld", (int)ok, x * 256, y);
}
""")
    return lambda *a: tuple(int(t) for t in run(*a).split())


@pytest.mark.parametrize("geom,fits", [
    ((32, 32, 32, 16, 32, 32, 16, 3, 3, 1, 1), True),
    ((256, 2048, 2047, 1, 2048, 2047, 1, 3, 3, 1, 1), True),         # 1073217536 pixels
    ((1073741760, 1, 1, 1, 1, 1, 1, 1, 1, 1, 0), True),              # the most
    ((1073741761, 1, 1, 1, 1, 1, 1, 1, 1, 1, 0), False),
    ((133, 4096, 3942, 1, 4096, 3942, 1, 3, 3, 1, 1), False),        # 2147475456 pixels: 2^33 threads of 64-pixel tiles
    ((133, 4096, 3942, 1, 2048, 1971, 1, 3, 3, 2, 1), False),        # the same number in the data gradient alone
    ((1, 1, 1, 1, 1, 1, 4194240, 1, 1, 1, 0), True),
    ((1, 1, 1, 1, 1, 1, 4194241, 1, 1, 1, 0), False),                # 65536 column tiles
    ((1, 1, 1, 4194240, 1, 1, 1, 7, 7, 1, 3), True),
    ((2, 8, 8, 4000000, 8, 8, 1, 13, 13, 1, 6), False),              # 21 M tiles of the weight gradient
])
def test_generic_convolutions_stay_within_the_launch_limits(generic_fits, geom, fits):
    ok, threads, blocks_y = generic_fits(*geom)
    assert ok == fits
    if ok:
        assert threads < 2 ** 32 and blocks_y <= 65535
