"""The tile shapes and step widths the matrix-core convolutions choose between, each at a size that selects it (which one is
asserted on the host, test_conv_rules_host.py), layer by layer against the oracle: ragged rows and columns, contractions that are no multiple of a step, forward, data gradient (with the
BatchNorm sums in the epilogue, and in parity classes for stride 2), bias and ReLU epilogues."""
import numpy as np
import pytest
import torch

from oracle import nets
from paper_2010_02838_amd.runner import pack_flat, to_device

from gpu_util import Case, rel
from test_gpu_step import check_layers
from test_gpu_transformer_head import head_case

pytestmark = pytest.mark.gpu

SHAPES = {
    # 64x64 tiles: 2800 and 700 rows, 72 and 200 columns, contractions of 648 and 1800; stride 2 in between
    "small": (dict(kind=1, widths=[72, 200], blocks=[1, 1], stem_width=72), lambda: nets.resnet20(widths=(72, 200), blocks=(1, 1)), 7, 20),
    # 200 tiles of 128x128: 64-wide steps in four stages (3x3), 128x64 tiles (1x1 into 128 columns)
    "alone": (dict(kind=2, widths=[128], blocks=[1], stem_width=64),
              lambda: nets.resnet50(classes=10, widths=(128,), blocks=(1,), stem=64), 100, 64),
    # 300 tiles of 128x128, a contraction of 1152: 64-wide steps in two stages
    "two_stages": (dict(kind=1, widths=[128], blocks=[1], stem_width=128), lambda: nets.resnet20(widths=(128,), blocks=(1,)), 150, 16),
    # 320 columns: five 128x64 tiles instead of three of 128x128
    "uneven_columns": (dict(kind=1, widths=[320], blocks=[1], stem_width=320), lambda: nets.resnet20(widths=(320,), blocks=(1,)), 96, 16),
    # 537 tiles of 256x32, the last one ragged: two stages; three and five steps of 8 and 16 channels, nine of 32
    "narrow_16": (dict(kind=1, widths=[16], blocks=[1], stem_width=16), lambda: nets.resnet20(widths=(16,), blocks=(1,)), 143, 31),
    "narrow_32": (dict(kind=1, widths=[32], blocks=[1], stem_width=32), lambda: nets.resnet20(widths=(32,), blocks=(1,)), 143, 31),
    # weight gradients of several layers in a launch: 21 of one tile class (more than a launch takes), 75 and 27 pixels (no whole steps)
    "many_layers": (dict(kind=1, widths=[72, 80], blocks=[5, 5], stem_width=72), lambda: nets.resnet20(widths=(72, 80), blocks=(5, 5)), 3, 5),
    # 16 and 4 pixels: less than a step; 64-column and 64-row tiles beside 128 (bottleneck: 1x1 and 3x3, stride 2, a shortcut each)
    "few_pixels": (dict(kind=2, widths=[24, 72], blocks=[2, 2], stem_width=64),
                   lambda: nets.resnet50(classes=10, widths=(24, 72), blocks=(2, 2), stem=64), 1, 16),
    # at most 64 columns over few rows: 63 tiles of 128x32, 32 of 64x64 (the last ones ragged), stride 2 between them
    "rows_32_64": (dict(kind=1, widths=[32, 64], blocks=[2, 1], stem_width=32), lambda: nets.resnet20(widths=(32, 64), blocks=(2, 1)), 20, 20),
    # 12493 rows of 64 columns: 128x64 with column sums, 64x64 without; 16 channels gathered for 64
    "rows_16_64": (dict(kind=1, widths=[16, 64], blocks=[1, 2], stem_width=16), lambda: nets.resnet20(widths=(16, 64), blocks=(1, 2)), 13, 62),
    # 8410 and 2250 rows of 40 columns, 40 channels: 32-wide steps
    "columns_40": (dict(kind=1, widths=[40, 40], blocks=[1, 1], stem_width=40), lambda: nets.resnet20(widths=(40, 40), blocks=(1, 1)), 10, 29),
    # tiles of eight waves: 256x256 with one partial sum for their 256 rows (50286 rows, 197 tiles, the last one 110 rows), with two (9537 rows
    # onto 1024 columns, the last tile 65 rows: one of its two), 128x256 (4624 rows onto 1024 columns)
    "eight_waves_tall": (dict(kind=1, widths=[256], blocks=[1], stem_width=256), lambda: nets.resnet20(widths=(256,), blocks=(1,)), 174, 17),
    "eight_waves_256": (dict(kind=2, widths=[256], blocks=[1], stem_width=64), lambda: nets.resnet50(classes=10, widths=(256,), blocks=(1,), stem=64), 33, 68),
    "eight_waves_128": (dict(kind=2, widths=[256], blocks=[1], stem_width=64), lambda: nets.resnet50(classes=10, widths=(256,), blocks=(1,), stem=64), 16, 68),
    # 128x160 tiles, the last row tile ragged: 104040 rows of 160 columns, the parity classes of a stride-2 data gradient onto 160 (26010
    # rows), and two columns of tiles (320) over 26010 rows
    "columns_160": (dict(kind=1, widths=[160, 64], blocks=[1, 1], stem_width=160), lambda: nets.resnet20(widths=(160, 64), blocks=(1, 1)), 90, 34),
    "columns_320": (dict(kind=1, widths=[320], blocks=[1], stem_width=320), lambda: nets.resnet20(widths=(320,), blocks=(1,)), 90, 17),
    # 520 tiles with column sums: 128x128 still (without the sums 256x128: the test below)
    "rows_per_sum": (dict(kind=1, widths=[128], blocks=[1], stem_width=128), lambda: nets.resnet20(widths=(128,), blocks=(1,)), 260, 16),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_tile_shapes_bf16_layers(name):
    kw, mk, batch, res = SHAPES[name]
    c = Case(kw, mk(), "bf16", batch, res, 10)
    check_layers(c, c.gpu())


def test_tall_tiles_without_column_sums(monkeypatch):
    """66759 rows (522 tiles of 128 rows, 261 of 256, the last one ragged) onto 128 columns: launches that take no column sums run
    on 256x128 tiles.  Data gradients (layer by layer, the reduction pass of BatchNorm kept apart), and the forward pass in
    evaluation mode against the same pass on the plain kernels (which round the same fp32 sums to bf16: a last place now and
    then, behind three convolutions; the bound is four times 2^-9)."""
    monkeypatch.setenv("CODISTILL_SEPARATE_BN_REDUCTION", "1")
    c = Case(dict(kind=1, widths=[128], blocks=[1], stem_width=128), nets.resnet20(widths=(128,), blocks=(1,)), "bf16", 231, 17, 10)
    check_layers(c, c.gpu())
    B, m, dev = c.B, c.model, "cuda:0"
    rng = np.random.default_rng(7)
    run = torch.from_numpy(np.concatenate([np.concatenate([rng.normal(0, 0.5, 128), rng.uniform(0.5, 2, 128)]) for _ in range(3)]).astype(np.float32)).to(dev)
    params, x = to_device(pack_flat(m, c.th), m.torch_dtype), to_device(c.x, m.torch_dtype)
    ws = torch.empty(m.workspace_bytes(c.batch, False), dtype=torch.uint8, device=dev)
    z = [torch.empty(c.batch, 10, device=dev) for _ in range(2)]
    B.codistill_forward(m, params, x, ws, z[0], False, B.CD_BN_RUNNING, run)
    monkeypatch.setenv("CODISTILL_FORCE_SIMPLE", "1")
    B.codistill_forward(m, params, x, ws, z[1], False, B.CD_BN_RUNNING, run)
    torch.cuda.synchronize()
    assert rel(z[0].cpu().numpy(), z[1].cpu().numpy()) <= 4 * 2.0 ** -9


@pytest.mark.parametrize("shape", [(2100, 512, 2048, 264),    # 128x256 tiles with bias and ReLU, 64x64 with bias
                                   (70, 72, 200, 1000),       # few rows: 64x64 tiles, fp32 logits too
                                   (300, 520, 72, 4104),      # logits of a filter beyond 4 MiB: grouped tile order, 64-wide steps
                                   (4700, 256, 2304, 264),    # 256x256 tiles, 18 row tiles and a ragged one; bias and ReLU, data gradient
                                   (4700, 256, 1024, 264),    # 128x256 tiles of eight waves
                                   (8200, 64, 128, 4104)])    # 64-wide steps with a single step; ragged logits
def test_dense_layer_tiles_bf16_layers(shape):
    c = head_case("bf16", *shape)
    check_layers(c, c.gpu())


def _timer_classes(m, batch, res, evaluation):
    """launches per class of the built-in timer in one forward pass"""
    from paper_2010_02838_amd import binding as B
    dev = "cuda:0"
    x = torch.randn(batch, res, res, 3, device=dev).to(m.torch_dtype)
    run = torch.ones(m.bn_running_elements(), device=dev)
    B.profile_reset()
    B.profile_enable(True)
    try:
        B.codistill_forward(m, torch.zeros(m.n_elements, dtype=m.torch_dtype, device=dev), x,
                            torch.empty(m.workspace_bytes(batch, False), dtype=torch.uint8, device=dev), torch.empty(batch, 10, device=dev), False,
                            B.CD_BN_RUNNING if evaluation else B.CD_BN_BATCH_STATS, run)
        torch.cuda.synchronize()
        return {k: v["launches"] for k, v in B.profile_collect().items()}
    finally:
        B.profile_enable(False)
        B.profile_reset()


def test_timer_class_of_a_convolution_is_that_of_its_tiles():
    """10240 rows: the 1x1 convolutions onto 512 columns (contractions of 64 and 128) take 256x128 tiles with the column sums and
    128x256 ones without; every other convolution has 64 or 128 columns."""
    from paper_2010_02838_amd import binding as B
    m = B.Model(B.arch_preset(2, in_h=64, in_w=64, classes=10, widths=[128], blocks=[1], stem_width=64), B.CD_BF16)
    assert _timer_classes(m, 40, 64, evaluation=False)["conv_fprop_wide"] == 0
    assert _timer_classes(m, 40, 64, evaluation=True)["conv_fprop_wide"] == 2


def test_timer_counts_only_launches_that_are_made():
    """Evaluation: one normalisation pass per BatchNorm, none in front of it; the one that also computes the max-pool has two
    (statistics, then both in one pass)."""
    from paper_2010_02838_amd import binding as B
    m = B.Model(B.arch_preset(2, in_h=64, in_w=64, classes=10, widths=[128], blocks=[1], stem_width=64), B.CD_BF16)
    bn = [o for o in m.graph(4)[0] if o["kind"] == "bn"]
    n = _timer_classes(m, 4, 64, evaluation=True)
    assert n["bn_apply"] == len(bn) - 1 and sum(o["fused_pool"] for o in bn) == 1
    assert n["norm"] == 2


@pytest.mark.parametrize("name,dtype", [("groups_of_channels", "bf16"), ("groups_of_channels", "f32"), ("one_group", "bf16"), ("one_group", "f32"),
                                        ("sums_in_a_kernel", "bf16")])
def test_batchnorm_column_sums(name, dtype):
    """The elementwise passes that add up their channels' partial sums themselves, and the ones behind a kernel that does: 136
    and 200 channels (three groups of 48 at the most, four of 56 and a last one of 32), 8 (one vector a row), 24; rows that end inside a trip; 30 MB
    of 40 channels, whose sums are folded."""
    kw, mk, batch, res = {
        "groups_of_channels": (dict(kind=1, widths=[136, 200], blocks=[1, 1], stem_width=136), lambda: nets.resnet20(widths=(136, 200), blocks=(1, 1)), 3, 11),
        "one_group": (dict(kind=1, widths=[8, 24], blocks=[1, 1], stem_width=8), lambda: nets.resnet20(widths=(8, 24), blocks=(1, 1)), 5, 19),
        "sums_in_a_kernel": (dict(kind=1, widths=[40], blocks=[1], stem_width=40), lambda: nets.resnet20(widths=(40,), blocks=(1,)), 90, 64),
    }[name]
    c = Case(kw, mk(), dtype, batch, res, 10)
    check_layers(c, c.gpu())


EVAL_SHAPES = {   # architecture, batch, resolution: the tiles, column counts and dtypes an evaluation-mode convolution can take
    "small_tiles": (dict(kind=2, widths=[72], blocks=[2], stem_width=64), "bf16", 3, 40),            # 288 columns, 300 rows
    "narrow_columns": (dict(kind=1, widths=[16, 40], blocks=[1, 1], stem_width=16), "bf16", 143, 31),  # 32- and 64-column tiles
    "wide_and_tall": (dict(kind=2, widths=[128], blocks=[1], stem_width=64), "bf16", 130, 65),         # 128x256; odd image: no fused pool
    "columns_160": (dict(kind=1, widths=[160], blocks=[1], stem_width=160), "bf16", 90, 17),           # 128x160
    "eight_waves_256": (dict(kind=2, widths=[256], blocks=[2], stem_width=64), "bf16", 33, 68),        # 256x256, with a residual
    "eight_waves_128": (dict(kind=2, widths=[256], blocks=[1], stem_width=64), "bf16", 16, 68),        # 128x256 of eight waves
    "tall": (dict(kind=1, widths=[128], blocks=[1], stem_width=128), "bf16", 231, 17),                 # 256x128
    "grouped": (dict(kind=5, widths=[128, 256], out_widths=[128, 256], blocks=[2, 1], stem_width=64, groups=32), "bf16", 5, 48),
    "odd_channels": (dict(kind=1, widths=[18, 22], blocks=[1, 1], stem_width=18), "bf16", 7, 13),
    "f32": (dict(kind=1, widths=[16, 33], blocks=[1, 1], stem_width=16), "f32", 5, 15),
    "few_rows": (dict(kind=1, widths=[8, 8, 8, 8], blocks=[1, 1, 1, 1], stem_width=8), "bf16", 1, 8),
}
for _c in (12, 20, 36):   # 66309 rows: the 128-row tiles of the fp32 matrix instruction, the last one ragged, with one, two and four column tiles
    for _t in ("bf16", "f32"):
        EVAL_SHAPES["generic_tall_%d_%s" % (_c, _t)] = (dict(kind=1, widths=[_c], blocks=[1], stem_width=_c), _t, 69, 31)


def _same(a, b):
    return bool(((a == b) | (a.isnan() & b.isnan())).all())


@pytest.mark.parametrize("name,odd", [(n, False) for n in EVAL_SHAPES] + [(n, True) for n in (
    "small_tiles", "odd_channels", "f32", "generic_tall_20_bf16", "generic_tall_36_f32")])
def test_evaluation_norm_inside_the_convolution(name, odd):
    """Evaluation applies a BatchNorm as the convolution in front of it stores; with the per-launch timer on it is a pass of its
    own.  Same arithmetic on the same rounded values: every normalised tensor and the logits agree bit for bit.  odd: an image with an
    infinite pixel and one with a NaN (elements that the kernel of the fp32 matrix instruction computes again from their definition)."""
    from paper_2010_02838_amd import binding as B
    kw, dtype, batch, res = EVAL_SHAPES[name]
    m = B.Model(B.arch_preset(kw["kind"], in_h=res, in_w=res, classes=10, **{k: v for k, v in kw.items() if k != "kind"}),
                B.CD_F32 if dtype == "f32" else B.CD_BF16)
    g = torch.Generator().manual_seed(3)
    params = (torch.randn(m.n_elements, generator=g) * 0.1).to("cuda:0", m.torch_dtype)
    x = torch.randn(batch, res, res, 3, generator=g).to("cuda:0", m.torch_dtype)
    if odd:
        x[0, res // 2, 3, 1], x[-1, 2, res // 2, 0] = float("inf"), float("nan")
    run = (torch.rand(m.bn_running_elements(), generator=g) + 0.5).to("cuda:0")
    z = [torch.empty(batch, 10, device="cuda:0") for _ in range(2)]
    ops, ts = m.graph(batch)

    def forward(out):
        ws = torch.zeros(m.workspace_bytes(batch, False), dtype=torch.uint8, device="cuda:0")
        B.codistill_forward(m, params, x, ws, out, False, B.CD_BN_RUNNING, run)
        torch.cuda.synchronize()
        return ws

    fused = forward(z[0])
    B.profile_reset()
    B.profile_enable(True)
    try:
        apart = forward(z[1])
        assert B.profile_collect()["bn_apply"]["launches"] > 0
    finally:
        B.profile_enable(False)
        B.profile_reset()
    assert odd or bool(torch.isfinite(z[0]).all()) and float(z[0].std()) > 0
    seen = 0
    for o in ops:   # (the activations lie in the same places whether a pass keeps them or not)
        if o["kind"] == "bn" and not o["fused_pool"]:
            t = ts[o["y"]]
            n = batch * t["h"] * t["w"] * t["c"] * m.torch_dtype.itemsize
            a, b = (w[t["act_offset"]:t["act_offset"] + n].view(m.torch_dtype) for w in (fused, apart))
            assert float(a.nan_to_num(0, 0, 0).float().std()) > 0 and _same(a, b), "op on %d channels" % t["c"]
            seen += 1
    assert seen > 0 and _same(*z)
