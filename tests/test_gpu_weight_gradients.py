"""Weight gradients that several layers of a pass share a launch for: their distance from the float64 product of the very operands
that lie in the workspace, and infinite operands."""
import pytest
import torch

from paper_2010_02838_amd import synth
from paper_2010_02838_amd.runner import pack_flat, to_device

pytestmark = pytest.mark.gpu

CASES = {   # architecture, batch, resolution
    # 448 tiles of 128x128 over 4096 rows: one or two splits a layer
    "dense": (dict(kind=4, in_h=128, in_w=128, classes=256, widths=[512, 2048, 8], blocks=[1, 1]), 32, None),
    # 3x3 onto 512 columns: 144 tiles a layer, 3072 rows
    "spatial": (dict(kind=1, classes=10, widths=[512], blocks=[3], stem_width=16), 48, 8),
    # 64x128 tiles, 64 columns over 8192 rows
    "narrow": (dict(kind=1, classes=10, widths=[64], blocks=[5], stem_width=16), 128, 8),
}


def _pass(name, poison=None):
    """One forward and backward pass: (model, gradients, {op index: (x, dy)} of the convolutions, ops).  poison(ops, read) may
    change the saved activations in between."""
    from paper_2010_02838_amd import binding as B
    kw, batch, res = CASES[name]
    kw = dict(kw)
    if res:
        kw.update(in_h=res, in_w=res)
    m = B.Model(B.arch_preset(kw.pop("kind"), **kw), B.CD_BF16)
    dev = "cuda:0"
    params = to_device(pack_flat(m, synth.he_init(m.param_table(), 1, 0.1)), torch.bfloat16)
    x = torch.from_numpy(synth.tokens(batch, 256, 256, seed=0)).to(dev) if res is None else to_device(synth.images(batch, res, res, 3, seed=0), torch.bfloat16)
    rows = batch * m.rows_per_sample
    ws = torch.empty(m.workspace_bytes(batch, True), dtype=torch.uint8, device=dev)
    logits, grads = torch.empty(rows, m.classes, device=dev), torch.empty(m.n_elements, device=dev)
    dz = torch.randn(rows, m.classes, generator=torch.Generator().manual_seed(5)).to(dev) / rows
    ops, ts = m.graph(batch)

    def read(t, key):
        d = ts[t]
        n = batch * d["h"] * d["w"] * d["c"]
        return ws[d[key]:d[key] + 2 * n].view(torch.bfloat16).view(batch, d["h"], d["w"], d["c"])

    B.codistill_forward(m, params, x, ws, logits, True)
    if poison:
        torch.cuda.synchronize()
        poison(ops, read)
    B.codistill_backward(m, params, x, ws, dz, grads)
    torch.cuda.synchronize()
    convs = {i: (read(o["x"], "act_offset"), read(o["y"], "grad_offset")) for i, o in enumerate(ops) if o["kind"] == "conv" and o["x"]}
    return m, grads, convs, ops


def _dw(m, grads, o):
    p = m.params[o["param_w"]]
    return grads[p["offset"]:p["offset"] + p["size"]].view(p["shape"])


def _own_rows(M, N, K, taps):
    """Rows of a split of a layer by itself, which are what one chain of additions covers at the most (wgrad_plan in conv_rules.h)"""
    up = lambda a, b: -(-a // b)   # noqa: E731
    tiles = up(N, 128 if N > 64 else 64) * up(K, 128 if K > 64 else 64)
    target = 1024 if taps > 1 else 256 if N * K / (N + K) < 150 else 512
    splits = min(up(target, tiles), up(M, 128))
    return up(up(M, splits), 32) * 32


@pytest.mark.parametrize("name", list(CASES))
def test_distance_from_the_float64_product(name):
    """A chain of fp32 additions over R rows of one dw element takes 16 rows a time; each of its R / 16 roundings is off by
    u / sqrt(3) of the sum at hand in the mean square (u = 2^-24), and that sum is taken to be no larger than the whole block's, P_b:
    the square of the error is at most R / 16 * u^2 / 3 * sum_b P_b^2, and one more rounding of the total.  (A single chain over all rows
    was at up to 2.0 times the bound in "dense", 1.07 in "spatial" and 1.5 in "narrow".)"""
    u = 2.0 ** -24
    m, grads, convs, ops = _pass(name)
    worst = 0.0
    for i, (x, dy) in convs.items():
        o = ops[i]
        if x.shape[-1] <= 16:
            continue   # (a layer by itself)
        k, s, pad = o["k"], o["stride"], o["pad"]
        xp = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad)) if pad else x
        ho, wo = dy.shape[1:3]
        d = dy.reshape(-1, dy.shape[-1]).double()
        R = _own_rows(d.shape[0], d.shape[1], x.shape[-1] * k * k, k * k)
        err = total = blocks = 0.0
        got = _dw(m, grads, o).double()
        for r in range(k):
            for q in range(k):
                t = xp[:, r:r + (ho - 1) * s + 1:s, q:q + (wo - 1) * s + 1:s].reshape(-1, x.shape[-1]).double()
                ref = 0
                for at in range(0, d.shape[0], R):
                    P = d[at:at + R].t().contiguous() @ t[at:at + R]
                    ref = ref + P
                    blocks += float(P.square().sum())
                err += float((got[:, r, q] - ref).square().sum())
                total += float(ref.square().sum())
        bound = (R / 16 * u * u / 3 * blocks) ** 0.5 + u / 3 ** 0.5 * total ** 0.5
        print("%s op %d: error %.2e of dw, bound %.2e" % (name, i, (err / total) ** 0.5, bound / total ** 0.5))
        worst = max(worst, err ** 0.5 / bound)
    assert worst <= 1.0


def test_infinite_operands():
    """An infinite element of a saved input makes its column of dw infinite with the sign of dy (and NaN where two infinities of opposite
    signs meet), whatever is added afterwards; every other element is as it was."""
    name = "dense"
    m, clean, convs, ops = _pass(name)
    # dense layers behind an attention op: nothing else in the backward pass reads their input (a ReLU's output gates its own gradient)
    at = {i: 3 + 5 * i for i in convs if ops[i]["x"] == ops[i - 1]["y"] and ops[i - 1]["kind"] == "attn"}
    assert len(at) == 3

    def poison(ops, read):
        for i, c in at.items():
            x = read(ops[i]["x"], "act_offset").view(4096, -1)
            x[7, c] = float("inf")
            x[2049, c + 1] = -float("inf")
            x[40, c + 2] = x[3999, c + 2] = float("inf")

    m, grads, convs, ops = _pass(name, poison)
    inf = float("inf")
    for i, c in at.items():
        got, was = _dw(m, grads, ops[i]).view(512, -1), _dw(m, clean, ops[i]).view(512, -1)
        dy = convs[i][1].view(4096, -1).float()
        want = was.clone()
        for col, rows in ((c, ((7, inf),)), (c + 1, ((2049, -inf),)), (c + 2, ((40, inf), (3999, inf)))):
            want[:, col] = sum(dy[r] * v for r, v in rows)
        assert bool(torch.isinf(want[:, c]).any()) and bool(torch.isnan(want[:, c + 2]).any())
        assert torch.equal(torch.nan_to_num(got, nan=1.5), torch.nan_to_num(want, nan=1.5)), "op %d" % i


@pytest.mark.parametrize("batch,h,w", [(1, 8, 16), (2, 8, 16), (16, 8, 16), (17, 8, 16), (26, 37, 32)])
def test_bias_gradients(batch, h, w):
    """1, 2, 16, 17 and 240 splits of 40 channels (three blocks of 16, the last one partial), a layer that goes by itself: sums of bf16 in
    fp32 over eight pixels, in fp64 over the rest."""
    from paper_2010_02838_amd import binding as B
    m = B.Model(B.arch_preset(B.CD_ARCH_TINY_CNN, in_h=h, in_w=w, widths=[16, 40]), B.CD_BF16)
    dev, g = "cuda:0", torch.Generator().manual_seed(3)
    params = to_device(pack_flat(m, synth.he_init(m.param_table(), 1, 0.1)), torch.bfloat16)
    x = torch.randn(batch, h, w, 3, generator=g).to(dev, torch.bfloat16)
    ws = torch.empty(m.workspace_bytes(batch, True), dtype=torch.uint8, device=dev)
    z, grads = torch.empty(batch, 10, device=dev), torch.empty(m.n_elements, device=dev)
    B.codistill_forward(m, params, x, ws, z, True)
    B.codistill_backward(m, params, x, ws, torch.randn(batch, 10, generator=g).to(dev), grads)
    torch.cuda.synchronize()
    ops, ts = m.graph(batch)
    for o in ops:
        if o["kind"] == "conv":
            t, p = ts[o["y"]], m.params[o["param_b"]]
            n = 2 * batch * h * w * t["c"]
            dy = ws[t["grad_offset"]:t["grad_offset"] + n].view(torch.bfloat16).view(-1, t["c"]).double()
            got = grads[p["offset"]:p["offset"] + p["size"]].double()
            assert bool(((got - dy.sum(0)).abs() <= 8 * 2.0 ** -24 * dy.abs().sum(0)).all())
