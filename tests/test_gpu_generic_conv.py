"""Convolutions on the fp32 matrix instruction (any channel count, fp32 and bf16 storage), layer by layer against the oracle."""
import numpy as np
import pytest
import torch

from oracle import nets
from paper_2010_02838_amd import synth
from paper_2010_02838_amd.runner import pack_flat, to_device

from gpu_util import Case, rel
from test_gpu_step import check_layers

pytestmark = pytest.mark.gpu

SHAPES = {
    # four channels per load; 66309 rows: 519 tiles of 128 rows, the last one ragged; 12 columns (one tile of 16), and 20 behind
    # the stride, on 64-row tiles
    "vec4_tall": (dict(kind=1, widths=[12, 20], blocks=[1, 1], stem_width=12), lambda: nets.resnet20(widths=(12, 20), blocks=(1, 1)),
                  69, 31),
    # the same 128-row tiles with two and with four 16-column tiles side by side, and with two such blocks of columns (33635 rows)
    "vec4_tall_20": (dict(kind=1, widths=[20], blocks=[1], stem_width=20), lambda: nets.resnet20(widths=(20,), blocks=(1,)), 69, 31),
    "vec4_tall_36": (dict(kind=1, widths=[36], blocks=[1], stem_width=36), lambda: nets.resnet20(widths=(36,), blocks=(1,)), 69, 31),
    "vec4_tall_68": (dict(kind=1, widths=[68], blocks=[1], stem_width=68), lambda: nets.resnet20(widths=(68,), blocks=(1,)), 35, 31),
    # one channel per load: odd channel counts, ragged tiles in every dimension
    "scalar": (dict(kind=1, widths=[5, 33], blocks=[1, 1], stem_width=5), lambda: nets.resnet20(widths=(5, 33), blocks=(1, 1)), 3, 13),
    # the same over more pixels (2197): few weights leave the plain weight gradient for the tiled one
    "scalar_rows": (dict(kind=1, widths=[5, 33], blocks=[1, 1], stem_width=5), lambda: nets.resnet20(widths=(5, 33), blocks=(1, 1)), 13, 13),
    # more than 64 columns and a contraction of many taps; fewer pixels than one step of the weight gradient
    "columns": (dict(kind=1, widths=[68, 132], blocks=[1, 1], stem_width=68), lambda: nets.resnet20(widths=(68, 132), blocks=(1, 1)),
                1, 7),
    # 7x7 stride-2 stem on odd images, 1x1 filters with and without stride
    "bottleneck": (dict(kind=2, widths=[6, 12], blocks=[1, 1], stem_width=20),
                   lambda: nets.resnet50(classes=10, widths=(6, 12), blocks=(1, 1), stem=20), 5, 37),
    # 4100 channels into the average pool: more vectors than one block takes
    "many_channels": (dict(kind=2, widths=[1025], blocks=[1], stem_width=4),
                      lambda: nets.resnet50(classes=10, widths=(1025,), blocks=(1,), stem=4), 2, 16),
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", list(SHAPES))
def test_generic_convolutions_layers(name, dtype):
    kw, mk, batch, res = SHAPES[name]
    c = Case(kw, mk(), dtype, batch, res, 10)
    check_layers(c, c.gpu())


def _both_forms(monkeypatch, run):
    """run() on the fp32 matrix instruction and on the plain kernels, which leave out what lies outside the image"""
    a = run()
    monkeypatch.setenv("CODISTILL_FORCE_SIMPLE", "1")
    b = run()
    monkeypatch.delenv("CODISTILL_FORCE_SIMPLE")
    return zip(a, b)


def _same(got, want, tol, what):
    """NaN and infinities at the same places, the finite values alike; there are finite and infinite or NaN ones at all"""
    finite = np.isfinite(want)
    assert finite.any() and not finite.all(), what
    assert np.array_equal(np.isnan(got), np.isnan(want)), (what, int(np.isnan(got).sum()), int(np.isnan(want).sum()))
    assert np.array_equal(got[~finite & ~np.isnan(want)], want[~finite & ~np.isnan(want)]), what
    assert rel(got[finite], want[finite]) <= tol, (what, rel(got[finite], want[finite]))


class _Net:
    """A network, its inputs and its finite parameters; pass_() runs forward and, given dz, backward with other parameters."""

    def __init__(self, dtype, batch, h, w, **kw):
        import torch
        from paper_2010_02838_amd import binding as B
        self.B, self.batch = B, batch
        self.m = B.Model(B.arch_preset(kw.pop("kind"), in_h=h, in_w=w, classes=10, **kw), B.CD_BF16 if dtype == "bf16" else B.CD_F32)
        self.flat = pack_flat(self.m, synth.he_init(self.m.param_table(), 1, 0.1))
        self.x = to_device(synth.images(batch, h, w, 3, seed=0), self.m.torch_dtype)
        self.ops, self.tensors = self.m.graph(batch)
        self.ws = torch.zeros(self.m.workspace_bytes(batch, True), dtype=torch.uint8, device="cuda:0")

    def param(self, flat, idx):
        q = self.m.params[idx]
        return flat[q["offset"]:q["offset"] + q["size"]].reshape(q["shape"])

    def pass_(self, forward, backward=None, dz=None):
        import torch
        dev = lambda a: to_device(a, self.m.torch_dtype)  # noqa: E731
        self.B.codistill_forward(self.m, dev(forward), self.x, self.ws, torch.empty(self.batch, 10, device="cuda:0"), True)
        if dz is None:
            return None
        grads = torch.zeros(self.m.n_elements, device="cuda:0")
        self.B.codistill_backward(self.m, dev(forward if backward is None else backward), self.x, self.ws, torch.from_numpy(dz).to("cuda:0"), grads)
        return grads.cpu().numpy()

    def read(self, t, key):
        import torch
        t = self.tensors[t]
        n, at = self.batch * t["h"] * t["w"] * t["c"], t[key]
        size = 2 if self.m.torch_dtype == torch.bfloat16 else 4
        return self.ws[at:at + size * n].view(self.m.torch_dtype).double().cpu().numpy().reshape(self.batch, t["h"], t["w"], t["c"])


@pytest.mark.parametrize("dtype,tol", [("f32", 1e-6), ("bf16", 1e-2)])
@pytest.mark.parametrize("widths", [(4, 8), (5, 3), (20, 68)])
def test_infinite_filter_elements_do_not_reach_past_the_border(monkeypatch, dtype, tol, widths):
    """Forward: where the tap of an infinite filter element lies outside the image the output stays finite."""
    c = _Net(dtype, 3, 9, 9, kind=0, widths=list(widths))
    first, second = [o for o in c.ops if o["kind"] == "conv"]
    w = c.flat.copy()
    c.param(w, first["param_w"])[0, 2, 2, 1] = np.inf    # the tap below and to the right
    c.param(w, second["param_w"])[1, 0, 1, 0] = -np.inf  # the tap above, on a channel that is infinite itself

    def run():
        c.pass_(w)
        return [c.read(first["y"], "act_offset"), c.read(second["y"], "act_offset")]
    for k, (a, b) in enumerate(_both_forms(monkeypatch, run)):
        if k == 0:
            assert np.isfinite(b[:, -1]).all() and np.isfinite(b[:, :, -1]).all() and not np.isfinite(b[:, :-1, :-1, 0]).all()
        _same(a, b, tol, "activation %d" % k)


@pytest.mark.parametrize("dtype,tol", [("f32", 1e-5), ("bf16", 1e-2)])
@pytest.mark.parametrize("hw", [(1, 1), (2, 1), (1, 5)])
def test_infinite_gradients_stay_with_the_taps_that_see_them(monkeypatch, dtype, tol, hw):
    """Weight gradients: taps that lie outside the image at every pixel keep their zero however large dy is."""
    c = _Net(dtype, 2100, hw[0], hw[1], kind=0, widths=[5, 12])
    dz = np.random.default_rng(2).standard_normal((2100, 10)).astype(np.float32)
    dz[7, 3] = np.inf
    for a, b in _both_forms(monkeypatch, lambda: [c.param(c.pass_(c.flat, dz=dz), o["param_w"]) for o in c.ops if o["kind"] == "conv"]):
        for r, s in ((0, 0), (0, 2), (2, 0), (2, 2)):    # the corner taps see no image of one row or one column
            assert np.all(b[:, r, s] == 0)
        _same(a, b, tol, "weight gradient")


@pytest.mark.parametrize("dtype,tol", [("f32", 1e-5), ("bf16", 2e-2)])
@pytest.mark.parametrize("widths", [(4, 12), (5, 33)])
def test_infinite_filter_elements_in_a_strided_data_gradient(monkeypatch, dtype, tol, widths):
    """Data gradient of a stride-2 3x3 convolution and of the stride-2 1x1 convolution beside it (accumulated): pixels
    between the strides do not see an infinite filter element, and what was there already stays."""
    c = _Net(dtype, 3, 9, 9, kind=1, widths=list(widths), blocks=[1, 1], stem_width=widths[0])
    dz = np.random.default_rng(2).standard_normal((3, 10)).astype(np.float32) / 30
    strided = [o for o in c.ops if o["kind"] == "conv" and o["stride"] == 2]
    assert len(strided) == 2 and strided[0]["x"] == strided[1]["x"]
    w = c.flat.copy()
    c.param(w, [o for o in strided if o["k"] == 3][0]["param_w"])[0, 0, 1, 1] = np.inf

    def run():
        c.pass_(c.flat, w, dz)
        return [c.read(strided[0]["x"], "grad_offset")]
    for a, b in _both_forms(monkeypatch, run):
        _same(a, b, tol, "input gradient")


def test_more_layers_than_a_weight_gradient_launch_takes():
    """17 layers (the six of at most 1024 weights go to the plain kernel): weight gradients in launches of 16 and 1, four channels per load and
    one, 507, 147 and 48 pixels (several splits and one, the last step ragged)."""
    c = Case(dict(kind=1, widths=[20, 36, 9], blocks=[4, 4, 2], stem_width=20), nets.resnet20(widths=(20, 36, 9), blocks=(4, 4, 2)), "f32", 3, 13, 10)
    check_layers(c, c.gpu())


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("widths", [(16, 40), (5, 35)])
@pytest.mark.parametrize("batch,h,w", [(1, 8, 16), (2, 13, 16), (26, 37, 32)])
def test_bias_gradients_with_the_weight_gradients(dtype, widths, batch, h, w):
    """One split, four and some hundred, channel counts that end inside a tile and inside a block of the splits' sum, against the float64 sums of
    the dy that the pass left.  A lane adds at most 8 values in fp32 and the rest in fp64: 8 half places of the sum of magnitudes, and one to round."""
    from paper_2010_02838_amd import binding as B
    if dtype == "bf16" and widths == (16, 40):
        pytest.skip("on the bf16 matrix cores")
    m = B.Model(B.arch_preset(B.CD_ARCH_TINY_CNN, in_h=h, in_w=w, widths=list(widths)), B.CD_F32 if dtype == "f32" else B.CD_BF16)
    dev, gen, dt = "cuda:0", torch.Generator().manual_seed(3), m.torch_dtype
    params = to_device(pack_flat(m, synth.he_init(m.param_table(), 1, 0.1)), dt)
    x = torch.randn(batch, h, w, 3, generator=gen).to(dev, dt)
    ws = torch.empty(m.workspace_bytes(batch, True), dtype=torch.uint8, device=dev)
    z, grads = torch.empty(batch, 10, device=dev), torch.full((m.n_elements,), 7.0, device=dev)
    B.codistill_forward(m, params, x, ws, z, True)
    B.codistill_backward(m, params, x, ws, torch.randn(batch, 10, generator=gen).to(dev), grads)
    torch.cuda.synchronize()
    ops, ts = m.graph(batch)
    for o in ops:
        if o["kind"] == "conv":
            t, p = ts[o["y"]], m.params[o["param_b"]]
            n = dt.itemsize * batch * h * w * t["c"]
            dy = ws[t["grad_offset"]:t["grad_offset"] + n].view(dt).view(-1, t["c"]).double()
            got = grads[p["offset"]:p["offset"] + p["size"]].double()
            assert bool(((got - dy.sum(0)).abs() <= 9 * 2.0 ** -24 * dy.abs().sum(0)).all())


@pytest.mark.parametrize("dtype,tol", [("f32", 1e-4), ("bf16", 3e-2)])
@pytest.mark.parametrize("width,batch,hw", [(12, 69, 31), (36, 5, 17), (5, 3, 13)])
@pytest.mark.parametrize("odd", [False, True])
def test_statistics_from_the_convolution(dtype, tol, width, batch, hw, odd):
    """The BatchNorms' mean and 1 / sqrt(var + eps) from the column sums that their convolutions left (128- and 64-row blocks, ragged last ones, one and
    four channels per load; that they leave them: test_launch_order_host.py) against float64 sums of what they stored.  odd: images one pixel
    high and infinite filter elements in the taps above and below them: every element of their channels is a NaN to the matrix instruction,
    counts as zero there, and is computed again from its definition, finite, behind the sums."""
    n = _Net(dtype, batch, 1 if odd else hw, hw * hw if odd else hw, kind=1, widths=[width], blocks=[1], stem_width=width)
    w = n.flat.copy()
    convs = [k for k, o in enumerate(n.ops) if o["kind"] == "conv" and n.ops[k + 1]["kind"] == "bn"]
    assert convs[0] == 0 and len(convs) == 3
    if odd:
        for k in convs:
            n.param(w, n.ops[k]["param_w"])[1::2, 0, 1, 1] = np.inf
            n.param(w, n.ops[k]["param_w"])[-1, 2, 0, 2] = -np.inf
    n.pass_(w)
    for k in convs:
        conv, bn = n.ops[k], n.ops[k + 1]
        x, y = n.read(conv["y"], "act_offset"), n.read(bn["y"], "act_offset")
        assert np.isfinite(x).all() and np.isfinite(y).all()
        g, b = n.param(n.flat, bn["param_w"]), n.param(n.flat, bn["param_b"])
        want = (x - x.mean((0, 1, 2))) / np.sqrt(x.var((0, 1, 2)) + 1e-5) * g + b
        if bn["res"] >= 0:
            want = want + n.read(bn["res"], "act_offset")
        assert rel(y, np.maximum(want, 0)) <= tol


@pytest.mark.parametrize("scale", [1.0, 2.0 ** 51])
@pytest.mark.parametrize("dtype,width,batch", [("f32", 16, 32), ("f32", 16, 33), ("f32", 20, 66), ("f32", 16, 105), ("f32", 20, 131), ("bf16", 20, 33), ("bf16", 36, 151)])
def test_statistics_of_many_partial_sums_are_added_in_fp64(dtype, width, batch, scale):
    """Channels that copy an image of integers 250 - 3 .. 250 + 3 (times a power of two with which the squares of a block's rows have a finite
    sum in fp32 and those of the tensor have not): every sum over the rows of a block is exact in fp32 (128 x 253^2 < 2^24), those
    over the tensor are not, and the variance is a 15000th of the mean square.  fp64 totals give it to the rounding of 1 / sqrt(var + eps) and of
    the update, an fp32 total of 2^31 is off by up to 2^-25, 1e-3 of the variance.  512 partial sums (added up by the elementwise pass), more
    (by the finalize), more than that takes (by a reduction pass) and more than 8 MB of them (folded in fp64 first)."""
    c = _Net(dtype, batch, 32, 32, kind=1, widths=[width], blocks=[1], stem_width=width)
    conv, bn = c.ops[0], c.ops[1]
    assert conv["kind"] == "conv" and bn["kind"] == "bn"
    gen = torch.Generator().manual_seed(5)
    c.x = (scale * (250 + torch.randint(-3, 4, (batch, 32, 32, 3), generator=gen))).to("cuda:0", c.m.torch_dtype)
    w = c.flat.copy()
    filt = c.param(w, conv["param_w"])
    filt[:] = 0
    for k in range(width):
        filt[k, 1, 1, k % 3] = 1
    running = torch.zeros(c.m.bn_running_elements(), device="cuda:0")
    c.B.codistill_forward(c.m, to_device(w, c.m.torch_dtype), c.x, c.ws, torch.empty(batch, 10, device="cuda:0"), True, c.B.CD_BN_BATCH_STATS, running)
    got = running[:2 * width].double().cpu().numpy().reshape(2, width)
    x = c.x.double().reshape(-1, 3)
    mean, var = (v.cpu().numpy()[np.arange(width) % 3] for v in (x.mean(0), x.var(0, unbiased=False)))
    M = batch * 1024
    # mean and 0.1 mean; 1 / sqrt rounded (twice in its square), the square, its inverse, minus eps, times two factors rounded themselves
    assert np.abs(got[0] / (0.1 * mean) - 1).max() <= 3 * 2.0 ** -24
    assert np.abs(got[1] / (0.1 * var * M / (M - 1)) - 1).max() <= 10 * 2.0 ** -24
