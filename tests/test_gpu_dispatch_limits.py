"""Calls on either side of the line that a dispatch rule draws (which kernel each takes is asserted on the host,
test_launch_order_host.py), against float64 products and sums of the operands that lie in the workspace."""
import pytest
import torch

from paper_2010_02838_amd import synth
from paper_2010_02838_amd.runner import pack_flat, to_device

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


def _pass(kind, dtype, batch, backward=True, **arch):
    """One pass on random inputs: (model, ops, reader of workspace tensors, logits, dlogits, gradient by parameter index)"""
    from paper_2010_02838_amd import binding as B
    m = B.Model(B.arch_preset(kind, **arch), B.CD_BF16 if dtype == "bf16" else B.CD_F32)
    dev, t = "cuda:0", m.torch_dtype
    params = to_device(pack_flat(m, synth.he_init(m.param_table(), 1, 0.1)), t)
    g = torch.Generator().manual_seed(3)
    shape = (batch, 1, 1, arch["widths"][0]) if kind == B.CD_ARCH_TRANSFORMER_HEAD else (batch, arch["in_h"], arch["in_w"], 3)
    x = torch.randn(shape, generator=g).to(dev, t)
    ws = torch.empty(m.workspace_bytes(batch, True), dtype=torch.uint8, device=dev)
    z, grads = torch.empty(batch, m.classes, device=dev), torch.empty(m.n_elements, device=dev)
    dz = torch.randn(batch, m.classes, generator=g).to(dev) / batch
    ops, ts = m.graph(batch)

    def read(i, key="act_offset"):
        d = ts[i]
        n = batch * d["h"] * d["w"] * d["c"] * t.itemsize
        return ws[d[key]:d[key] + n].view(t).view(-1, d["c"]).double()

    def stats(o):
        n = 16 * ts[o["x"]]["c"]
        return ws[o["stats_offset"]:o["stats_offset"] + n].view(torch.float32).view(4, -1).double()

    B.codistill_forward(m, params, x, ws, z, True)
    if backward:
        B.codistill_backward(m, params, x, ws, dz, grads)
    torch.cuda.synchronize()
    of = lambda buf, i: buf[m.params[i]["offset"]:m.params[i]["offset"] + m.params[i]["size"]].view(m.params[i]["shape"]).double()   # noqa: E731
    return m, ops, read, stats, z, dz, lambda i: of(grads, i), lambda i: of(params, i)


@pytest.mark.parametrize("batch", [200, 201])
def test_backward_sums_of_a_batchnorm(batch):
    """1600 and 1608 partial sums of 128 rows.  Each term of a sum is rounded three times (the difference, the product with 1 / std, that with
    dz), then at most 128 fp32 additions inside a partial sum, 51 more where they are folded, the rest in fp64, and the result's rounding."""
    from paper_2010_02838_amd import binding as B
    m, ops, read, stats, _, _, grad, _ = _pass(B.CD_ARCH_RESNET_BASIC, "bf16", batch, in_h=32, in_w=32, classes=10, widths=[72], blocks=[1], stem_width=72)
    seen = 0
    for o, after in zip(ops, ops[1:]):
        if o["kind"] != "bn" or after["kind"] != "conv" or after["x"] != o["y"]:
            continue
        mean, istd = stats(o)[:2]
        dz = read(o["y"], "grad_offset") * (read(o["y"]) > 0)
        xh = (read(o["x"]) - mean) * istd
        for got, terms in ((grad(o["param_b"]), dz), (grad(o["param_w"]), dz * xh)):
            assert bool(((got - terms.sum(0)).abs() <= (128 + 51 + 4) * U * terms.abs().sum(0)).all())
        seen += 1
    assert seen == 2


@pytest.mark.parametrize("rows,features,classes", [(16384, 64, 64), (16385, 64, 64), (16321, 64, 3), (16384, 56, 64), (16384, 200, 61), (1, 64, 1)])
def test_logits_of_a_classifier(rows, features, classes):
    """64x64 and 128x128 tiles on both sides of the line, ragged last rows, columns and steps: products of bf16 are exact, at most one rounding
    for each of the `features` additions."""
    from paper_2010_02838_amd import binding as B
    m, ops, read, _, z, _, _, param = _pass(B.CD_ARCH_TRANSFORMER_HEAD, "bf16", rows, False, widths=[features, 64], classes=classes)
    x, w = read(ops[-1]["x"]), param(ops[-1]["param_w"])
    assert bool(((z.double() - x @ w.t()).abs() <= features * U * (x.abs() @ w.abs().t())).all())


@pytest.mark.parametrize("rows", [1, 15, 16, 70])
@pytest.mark.parametrize("features,classes", [(64, 512), (64, 513), (63, 1024), (5, 3)])
def test_dense_weight_gradient(rows, features, classes):
    """16 and 4 row groups (256 and 258 blocks), fewer rows than groups, no whole columns or classes: a product and an addition a row, and the sum
    of the groups."""
    from paper_2010_02838_amd import binding as B
    m, ops, read, _, _, dz, grad, _ = _pass(B.CD_ARCH_TRANSFORMER_HEAD, "f32", rows, widths=[features, 8], classes=classes)
    x, d = read(ops[-1]["x"]), dz.double()
    assert bool(((grad(ops[-1]["param_w"]) - d.t() @ x).abs() <= (2 * rows + 16) * U * (d.abs().t() @ x.abs())).all())
