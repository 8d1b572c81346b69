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


def test_division_by_a_launch_constant(tmp_path):
    """Quotients below, at and above multiples, at the largest dividend, for small, odd, two's-power and very large divisors."""
    assert compiled(tmp_path, """
int main() {
  auto div = [](unsigned n, FastDiv f) { return (unsigned)(((unsigned long long)(n << 1) * f.mul) >> 32) >> f.shift; };
  for (unsigned d = 1; d < 4000; d++) {
    const FastDiv f = fast_div(d);
    for (unsigned k : {0u, 1u, 2u, 7u, 1000u, 2147483647u / d - 1, 2147483647u / d})
      for (int e = -1; e <= 1; e++) {
        const long long n = (long long)k * d + e;
        if (n >= 0 && n < (1ll << 31) && div((unsigned)n, f) != (unsigned)n / d) { printf("%u %lld", d, n); return 0; }
      }
    if (div(2147483647u, f) != 2147483647u / d) { printf("%u", d); return 0; }
  }
  for (unsigned d : {65535u, 65536u, 65537u, 1000003u, 1073741823u, 1073741824u, 1073741825u, 2147483647u, 2147483648u})
    for (unsigned n : {0u, 1u, d - 1, d, 2147483647u, 1073741824u})
      if (n < (1u << 31) && div(n, fast_div(d)) != n / d) { printf("%u %u", d, n); return 0; }
  printf("ok");
}
""")() == "ok"


SQUARE, TALL, WIDE, NARROW, SMALL = range(5)


@pytest.fixture(scope="module")
def tile(tmp_path_factory):
    run = compiled(tmp_path_factory.mktemp("tile"),
                   "int main(int, char** v) { printf(\"%d\", conv_tile_rule(atoll(v[1]), atoi(v[2]), atoi(v[3]), atoi(v[4]) != 0, atoi(v[5]) != 0)); }")
    return lambda *a: int(run(*a))


@pytest.fixture(scope="module")
def generic_tile(tmp_path_factory):
    run = compiled(tmp_path_factory.mktemp("generic"),
                   "int main(int, char** v) { const int n = atoi(v[2]); printf(\"%d %d\", generic_column_tiles(n), "
                   "(int)generic_tall_tiles(atoll(v[1]), n, atoi(v[3]) != 0)); }")
    return lambda *a: tuple(int(x) for x in run(*a).split())


@pytest.mark.parametrize("shape,want", [
    # (rows, columns, contraction, 64 channels or more per tap, column sums): the launches that test_gpu_conv_tiles.py is for
    ((2800, 72, 648, 1, 1), SMALL), ((700, 200, 648, 1, 1), SMALL), ((700, 200, 1800, 1, 1), SMALL),   # "small"
    ((25600, 128, 1152, 1, 1), SQUARE), ((25600, 128, 64, 1, 1), NARROW),                              # "alone"
    ((38400, 128, 1152, 1, 1), SQUARE),                                                                # "two_stages"
    ((24576, 320, 2880, 1, 1), NARROW),                                                                # "uneven_columns"
    ((66560, 128, 1152, 1, 1), SQUARE),                                                                # "rows_per_sum"
    ((66759, 128, 1152, 1, 0), TALL),                                                                  # tall tiles, no sums
    ((2100, 2048, 512, 1, 0), WIDE), ((2100, 512, 2048, 1, 0), SMALL),                                 # dense layers
    ((70, 200, 72, 1, 0), SMALL), ((8200, 128, 64, 1, 0), SMALL), ((8200, 4104, 128, 1, 0), SQUARE),
    ((10240, 512, 64, 1, 1), TALL), ((10240, 512, 128, 1, 1), TALL), ((10240, 512, 64, 1, 0), WIDE), ((10240, 512, 128, 1, 0), WIDE),  # timer classes
    # and of ResNet-50 at batch 256, with the sums
    ((802816, 256, 64, 1, 1), WIDE), ((200704, 512, 128, 1, 1), TALL), ((200704, 512, 256, 1, 1), WIDE), ((50176, 256, 1024, 1, 1), WIDE),
    ((50176, 256, 2304, 1, 1), TALL),
])
def test_tile_of_a_convolution(tile, shape, want):
    assert tile(*shape) == want


TILE_256, WIDE8 = 6, 7


@pytest.mark.parametrize("shape,want", [
    # (rows, columns, contraction, 64 channels or more per tap): either side of each line
    ((10240, 512, 2048, 1), WIDE8), ((8192, 512, 2048, 1), 0), ((9153, 512, 2048, 1), WIDE8), ((9088, 512, 2048, 1), 0), ((16384, 512, 2048, 1), WIDE8),
    ((16385, 512, 2048, 1), 0), ((18176, 512, 2048, 1), 0), ((18177, 512, 2048, 1), TILE_256), ((8192, 2048, 512, 1), TILE_256),
    ((8193, 2048, 512, 1), 0), ((12288, 2048, 512, 1), 0), ((14336, 2048, 512, 1), TILE_256), ((16384, 2048, 512, 1), TILE_256),
    ((16385, 2048, 512, 1), 0), ((8192, 2048, 256, 1), TILE_256), ((8192, 2048, 192, 1), 0), ((8192, 2048, 512, 0), 0), ((8192, 2176, 512, 1), 0),
    # the launches of test_gpu_conv_tiles.py: "eight_waves_tall", "eight_waves_256", "eight_waves_128", dense layers
    ((50286, 256, 2304, 1), TILE_256), ((9537, 1024, 256, 1), TILE_256), ((4624, 1024, 256, 1), WIDE8), ((4700, 2304, 256, 1), TILE_256),
    ((4700, 1024, 256, 1), WIDE8),
])
def test_tiles_of_eight_waves(tmp_path_factory, shape, want):
    run = compiled(tmp_path_factory.mktemp("eight"),
                   "int main(int, char** v) { printf(\"%d\", conv_eight_waves_rule(atoll(v[1]), atoi(v[2]), atoi(v[3]), atoi(v[4]) != 0)); }")
    assert int(run(*shape)) == want


def test_partial_sums_of_the_tiles_that_256_rows_take_the_place_of(tile):
    """256x256 tiles leave one partial sum for their rows where 256x128 tiles would, two elsewhere."""
    assert tile(50286, 256, 2304, 1, 1) == TALL and tile(9537, 1024, 256, 1, 1) == WIDE


@pytest.mark.parametrize("shape,want", [
    # (rows, columns, contraction, 64 channels or more per tap): either side of each line, and widths that 160 does not divide
    ((98304, 160, 1440, 1), 1), ((98304, 160, 1440, 0), 0), ((32768, 160, 1440, 1), 1), ((16384, 160, 1440, 1), 0), ((24576, 320, 2880, 1), 1),
    ((12288, 320, 2880, 1), 0), ((20480, 320, 2880, 1), 0), ((6144, 640, 5760, 1), 0), ((65536, 480, 480, 1), 1), ((8192, 480, 480, 1), 0),
    ((98304, 128, 1440, 1), 0), ((98304, 168, 1440, 1), 0),
    ((26010, 160, 1440, 1), 1), ((26010, 320, 1440, 1), 1), ((26010, 320, 64, 1), 1),   # the launches of test_gpu_conv_tiles.py, "columns_160" and "columns_320"
])
def test_columns_in_tiles_of_160(tmp_path_factory, shape, want):
    run = compiled(tmp_path_factory.mktemp("cols160"),
                   "int main(int, char** v) { printf(\"%d\", (int)conv_cols160_rule(atoll(v[1]), atoi(v[2]), atoi(v[3]), atoi(v[4]) != 0)); }")
    assert int(run(*shape)) == want


@pytest.fixture(scope="module")
def rows_rule(tmp_path_factory):
    """rows of a tile, and whether the sums it leaves are at most as many as the check for their room counts and 64 KB"""
    run = compiled(tmp_path_factory.mktemp("rows"), """
int main(int, char** v) {
  const long long M = atoll(v[1]);
  const int N = atoi(v[2]), sums = atoi(v[3]), rows = conv_rows_rule(M, N, atoi(v[4]), sums != 0);
  const long long tiles = (M + rows - 1) / rows;
  printf("%d %d", rows, (int)(tiles <= conv_stat_chunks_max(M) && (rows == 256 || tiles * N * 8 <= kSumBytes)));
}
""")
    return lambda *a: tuple(int(t) for t in run(*a).split())


@pytest.mark.parametrize("M,N,sums,rows", [(1, 64, 1, 64), (8192, 64, 1, 64), (8193, 64, 1, 128), (16384, 33, 1, 128), (16385, 64, 1, 256),
                                           (16384, 64, 0, 64), (16385, 64, 0, 128), (32769, 64, 0, 256), (1, 32, 1, 128), (32768, 32, 1, 128),
                                           (32769, 32, 1, 256), (32768, 8, 0, 128), (32769, 8, 0, 256)])
def test_rows_of_a_narrow_tile(rows_rule, M, N, sums, rows):
    got, room = rows_rule(M, N, sums, 129)
    assert got == rows and (room or not sums)
    assert rows_rule(M, N, sums, 128)[0] == 256


@pytest.mark.parametrize("rows,cols,vec4,want", [
    (66309, 12, 1, (1, 1)), (66309, 20, 1, (2, 1)), (66309, 36, 1, (4, 1)), (33635, 68, 1, (4, 1)),   # test_gpu_generic_conv.py
    (17664, 20, 1, (2, 0)), (66309, 12, 0, (1, 0)), (65408, 16, 1, (1, 0)), (65409, 16, 1, (1, 1)),
])
def test_tile_of_a_generic_convolution(generic_tile, rows, cols, vec4, want):
    assert generic_tile(rows, cols, vec4) == want
    if want[1] and rows > 66000:
        assert rows % 128


def test_partial_sums_fit_where_the_check_says_so(tmp_path):
    """Over row, column and contraction counts: the row tiles of a launch with column sums are at most conv_stat_chunks_max, and an
    area of exactly that many rows and the 32 fold rows is accepted, a float less is not."""
    run = compiled(tmp_path, """
int main() {
  const long long Ms[] = {1, 63, 64, 65, 128, 129, 2450, 8192, 12544, 16320, 16384, 16385, 24576, 32704, 32767, 32768, 32769, 32832, 50176, 65536, 200704, 802816, 3211264};
  const int Ns[] = {65, 72, 128, 129, 256, 320, 512, 640, 1024, 2048, 4096}, Ks[] = {64, 128, 256, 576, 1024, 2304, 4608, 36864}, rows[] = {128, 256, 128, 128, 64};
  long long worst = 0;
  for (long long M : Ms)
    for (int N : Ns) {
      const long long pitch = 2 * N + 64;
      const size_t need = (size_t)(conv_stat_chunks_max(M) + 32) * pitch * 4;
      if (!conv_sums_fit(M, pitch, need) || conv_sums_fit(M, pitch, need - 4)) { printf("check %lld %d", M, N); return 0; }
      for (int K : Ks)
        for (int w64 = 0; w64 < 2; w64++) {
          const int r = rows[conv_tile_rule(M, N, K, w64 != 0, true)];
          const long long chunks = (M + r - 1) / r;
          if (chunks > conv_stat_chunks_max(M)) { printf("%lld %d %d: %lld chunks", M, N, K, chunks); return 0; }
          if (chunks - (M / 128 + 1) > worst) worst = chunks - (M / 128 + 1);
        }
    }
  printf("ok %lld", worst);
}
""")
    out = run().split()
    assert out[0] == "ok"
    assert int(out[1]) > 32     # more than 128-row tiles and the fold rows' room would have held


@pytest.mark.parametrize("F,C", [(1, 1), (63, 5), (64, 1000), (2048, 1000), (192, 1 << 24), (254, 1 << 24), (16000, 1 << 18)])
def test_dense_weight_gradient_stays_within_the_launch_limits(tmp_path, F, C):
    """The most classes that a model takes (2^24) and inputs for which a thread per weight is a launch of fewer than 2^32 threads."""
    x, y = (int(v) for v in compiled(tmp_path, "int main(int, char** v) { const LinearDwGrid g = linear_dw_grid(atoi(v[1]), atoi(v[2])); "
                                     "printf(\"%lld %lld\", (long long)g.x, (long long)g.y); }")(F, C).split())
    tiles, groups = -(-(F + 1) // 64), -(-C // 4)
    assert x * 256 < 2 ** 32 and y <= 65535 and x % tiles == 0
    assert (y - 1) * (x // tiles) < groups <= y * (x // tiles)    # the last row of blocks is wanted, and the last class has a block


@pytest.fixture(scope="module")
def wgrad_splits(tmp_path_factory):
    """per layer: splits, where the rows that the splits take one after the other end, whether each is whole 32-row steps; then the
    launch's workgroups and the bytes of its partial sums.  arguments: scratch bytes, then M N K pointwise bias per layer"""
    run = compiled(tmp_path_factory.mktemp("wgrad"), """
int main(int c, char** v) {
  const int n = (c - 2) / 5;
  WgradShape s[16]; WgradSplit r[16];
  for (int k = 0; k < n; k++) {
    char** a = v + 2 + 5 * k;
    s[k].M = atoll(a[0]); s[k].N = atoi(a[1]); s[k].K = atoi(a[2]); s[k].pointwise = atoi(a[3]); s[k].bias = atoi(a[4]);
    s[k].taps = s[k].pointwise ? 1 : 9; s[k].slices = 1;
  }
  wgrad_plan(s, n, (size_t)atoll(v[1]), 0, r);
  long long blocks = 0, bytes = 0;
  for (int k = 0; k < n; k++) {
    long long at = 0, i;
    for (i = 0; i < r[k].splits; i++) {   // the kernel's 32-bit arithmetic
      const int M = (int)s[k].M, mbeg = (int)i * (int)r[k].m_per_split;
      const int mend = M - mbeg > (int)r[k].m_per_split ? mbeg + (int)r[k].m_per_split : M;
      if (mbeg != at || mend <= mbeg) break;
      at = mend;
    }
    printf("%lld %lld %d ", (long long)r[k].splits, at, r[k].m_per_split % 32 == 0);
    blocks += s[k].tiles() * r[k].splits; bytes += s[k].partials(r[k].splits);
  }
  printf("%lld %lld", blocks, bytes);
}
""")
    return lambda *a: [int(t) for t in run(*a).split()]


@pytest.mark.parametrize("scratch", [128 << 20, 1 << 20])
@pytest.mark.parametrize("layers", [[(1, 8, 8, 1, 0)], [(134217727, 8, 8, 1, 0)], [(8192, 512, 512, 1, 1)], [(8192, 32768, 512, 1, 0)], [(802816, 64, 576, 0, 0)],
                                    [(8192, 512, 512, 1, 1), (8192, 1536, 512, 1, 1), (8192, 2048, 512, 1, 1), (8192, 512, 2048, 1, 1)],
                                    [(31, 128, 1152, 0, 0)] * 16, [(75, 72, 648, 0, 0), (27, 80, 720, 0, 0), (50176, 256, 2304, 0, 0)],
                                    [(12544, 512, 4608, 0, 0)] * 5])
def test_weight_gradient_splits_take_every_row_once(wgrad_splits, layers, scratch):
    got = wgrad_splits(scratch, *[v for l in layers for v in l])
    blocks, bytes_ = got[-2:]
    splits = got[0:-2:3]
    for k, l in enumerate(layers):
        assert got[3 * k + 1] == l[0] and got[3 * k + 2] == 1
    assert bytes_ <= scratch
    if len(layers) > 1:   # a launch of several layers stays within two workgroups a compute unit where it splits at all
        assert blocks <= 512 or all(s == 1 for s in splits)


def test_weight_gradient_shape_starts_from_defined_values(tmp_path):
    """Every field, also in memory that held something else: the decisions below are made from shapes that the caller fills in part."""
    out = compiled(tmp_path, """
#include <cstring>
#include <new>
int main() {
  for (int fill = 0; fill < 256; fill += 255) {
    alignas(WgradShape) unsigned char mem[sizeof(WgradShape)];
    memset(mem, fill, sizeof mem);
    const WgradShape* s = new (mem) WgradShape;
    unsigned char bools[2];
    memcpy(bools, &s->pointwise, 1);
    memcpy(bools + 1, &s->bias, 1);
    printf("%lld %d %d %d %d %d %d ", (long long)s->M, s->N, s->K, s->taps, s->slices, bools[0], bools[1]);
  }
}
""")().split()
    assert out == ["0"] * 14


@pytest.mark.parametrize("M,N,K,with_bias,without", [
    (8192, 2048, 32, 0, 1), (65536, 32, 32, 0, 1),      # the bias sums of the splits are what tips them
    (8192, 512, 512, 0, 0), (8192, 32768, 512, 1, 1), (802816, 64, 64, 1, 1)])
def test_weight_gradient_by_itself(tmp_path, M, N, K, with_bias, without):
    """Pointwise layers whose partial sums, with those of the bias gradient, are a quarter of what the operands move or less go by themselves."""
    run = compiled(tmp_path, """
int main(int, char** v) {
  WgradShape s;
  s.M = atoll(v[1]); s.N = atoi(v[2]); s.K = atoi(v[3]); s.pointwise = true; s.taps = s.slices = 1; s.bias = atoi(v[4]) != 0;
  printf("%d", (int)wgrad_alone(s, 2 * s.M * ((int64_t)s.N + s.K)));
}
""")
    assert (int(run(M, N, K, 1)), int(run(M, N, K, 0))) == (with_bias, without)
