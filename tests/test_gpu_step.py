"""GPU parity of the whole codistillation step (forward x2, loss, backward, momentum-SGD)
against the float64 oracle, through the C ABI.

fp32 models are held to tight end-to-end tolerances.  For bf16 models two things are checked:

  * every layer, at its real shape inside the real pipeline, "teacher forced": the oracle's
    layer function is applied to the very tensors the GPU kernel consumed (read back from the
    workspace) and must reproduce the tensor the kernel wrote, to bf16 rounding (forward
    activations, activation gradients) or to fp32 accumulation error (parameter gradients,
    BatchNorm statistics);
  * end to end against the float64 oracle, quantity by quantity (logits, loss terms, the norm of
    every parameter-gradient tensor) to the stated 2e-2 - or, for a quantity that rounding the
    stored activations to bf16 alone (float64 arithmetic, the oracle's `perturb` map filled in by
    gpu_util.bf16_storage_points) already moves further than 1e-2, to twice that quantity's own
    measured sensitivity; see compare_bf16.  At random initialisation on N(0,1) images all
    samples of a batch look alike, the informative part of every activation and gradient is a
    small difference of large common terms, and BatchNorm with batch statistics removes the
    common part, so storage rounding is amplified layer after layer; that deviation is a
    property of the workload, not of a kernel, and the first check is what pins the kernels.
"""
import functools
import json
import os

import numpy as np
import pytest

from oracle import layers as L
from oracle import nets
from oracle.sgd import sgd_step
from paper_2010_02838_amd import synth

from gpu_util import Case, norm_err, rel

pytestmark = pytest.mark.gpu


# ----------------------------------------------------------------------------- fp32, end to end
def compare_f32(ref, got, arch, tol_logits, tol_loss, tol_grad, tol_theta):
    assert rel(got["logits"], ref["logits"]) <= tol_logits
    assert rel(got["peer_logits"], ref["peer_logits"][0]) <= tol_logits
    for a, b in zip(got["loss"], ref["loss"]):
        assert abs(a - b) <= tol_loss * abs(b), (got["loss"], ref["loss"])
    off = 0
    for name, shape, _, _ in arch.params:
        n = int(np.prod(shape))
        g, gr = got["grad"][off:off + n], ref["grad"][off:off + n]
        if np.linalg.norm(gr) > 1e-12:
            assert norm_err(g, gr) <= tol_grad and rel(g, gr) <= tol_grad, (name, rel(g, gr))
        else:
            assert np.linalg.norm(g) <= 1e-6
        off += n
    assert rel(got["theta"], ref["theta"]) <= tol_theta
    assert rel(got["v"], ref["v"]) <= tol_grad


def test_tiny_cnn_fp32_step():
    """Two tiny CNNs, fp32, batch 8 of 32x32x3, alpha 1, lr 0.1, momentum 0.9, one step from v = 0.
    Tolerances: 1e-5 on logits and loss, 1e-4 on per-tensor gradients (norm and L2), 1e-5 on weights."""
    c = Case(dict(kind=0), nets.tiny_cnn(), "f32", 8, 32, 10, jitter=0.0)
    ref, got = c.oracle(), c.gpu()
    compare_f32(ref, got, c.ref_arch, 1e-5, 1e-5, 1e-4, 1e-5)
    np.testing.assert_array_equal(got["v"], got["grad"])       # first step from v = 0


@pytest.mark.parametrize("dist", ["mse", "kl", "mse_centered"])
def test_tiny_cnn_fp32_step_variants(dist):
    c = Case(dict(kind=0), nets.tiny_cnn(), "f32", 5, 12, 10, v_scale=0.01)
    ref, got = c.oracle(alpha=0.5, wd=1e-3, dist=dist), c.gpu(alpha=0.5, wd=1e-3, dist=dist)
    compare_f32(ref, got, c.ref_arch, 1e-5, 1e-5, 1e-4, 1e-5)


SMALL = {
    "basic": (dict(kind=1, widths=[4, 8, 16], blocks=[2, 1, 1], stem_width=4),
              lambda: nets.resnet20(widths=(4, 8, 16), blocks=(2, 1, 1)), 6, 16, 10),
    "bottleneck": (dict(kind=2, widths=[4, 8, 8, 16], blocks=[2, 1, 1, 1], stem_width=8),
                   lambda: nets.resnet50(classes=7, widths=(4, 8, 8, 16), blocks=(2, 1, 1, 1), stem=8), 4, 40, 7),
    # channel counts that are multiples of 8: every convolution runs on the MFMA kernels (stride-2
    # 3x3, stride-2 1x1 shortcuts, the padded 7x7 stem) with ragged tiles in every dimension
    "bottleneck_mfma": (dict(kind=2, widths=[8, 16, 24, 32], blocks=[2, 1, 1, 1], stem_width=16),
                        lambda: nets.resnet50(classes=10, widths=(8, 16, 24, 32), blocks=(2, 1, 1, 1), stem=16),
                        5, 72, 10),
    "basic_mfma": (dict(kind=1, widths=[16, 24, 40], blocks=[1, 2, 1], stem_width=16),
                   lambda: nets.resnet20(widths=(16, 24, 40), blocks=(1, 2, 1)), 7, 20, 10),
    # grouped 3x3 convolutions (the ResNeXt family): 4, 8 and 12 channels per group in one slice of channels ...
    "resnext": (dict(kind=6, widths=[16, 32, 32, 48], out_widths=[24, 32, 48, 64], groups=4, blocks=[2, 1, 1, 1], stem_width=16),
                lambda: nets.resnext(classes=10, widths=(16, 32, 32, 48), outs=(24, 32, 48, 64), groups=4, blocks=(2, 1, 1, 1),
                                     stem=16), 5, 72, 10),
    # ... and 256 channels in two slices of 128 (four groups of 32 each), stride 1 and stride 2
    "resnext_slices": (dict(kind=6, widths=[256, 256], out_widths=[64, 64], groups=8, blocks=[1, 1], stem_width=32),
                       lambda: nets.resnext(classes=10, widths=(256, 256), outs=(64, 64), groups=8, blocks=(1, 1), stem=32),
                       3, 40, 10),
    # groups of 64 channels (slices of 64, the contraction runs over the group's channels only) and of 16 (two groups
    # per 32-channel slice), stride 1 and stride 2
    "resnext_cg64": (dict(kind=6, widths=[128, 128], out_widths=[32, 32], groups=2, blocks=[1, 1], stem_width=16),
                     lambda: nets.resnext(classes=10, widths=(128, 128), outs=(32, 32), groups=2, blocks=(1, 1), stem=16),
                     3, 40, 10),
    "resnext_cg16": (dict(kind=6, widths=[64, 64], out_widths=[32, 32], groups=4, blocks=[1, 1], stem_width=16),
                     lambda: nets.resnext(classes=10, widths=(64, 64), outs=(32, 32), groups=4, blocks=(1, 1), stem=16),
                     3, 40, 10),
    # the multi-view network (Section 5): a frozen first block, the rest sees one part of its output channels: 4 of 16
    # (plain kernels for the convolutions that read them) ...
    "wide_split": (dict(kind=7, widths=[16, 24, 32], blocks=[2, 1, 2], stem_width=8, n_splits=4, split=1),
                   lambda: nets.wide_resnet_split(split=1, n_splits=4, classes=10, widths=(16, 24, 32), blocks=(2, 1, 2), stem=8),
                   6, 16, 10),
    # ... and 16 of 32 (matrix-core kernels throughout)
    "wide_split_mfma": (dict(kind=7, widths=[32, 32, 48], blocks=[2, 1, 1], stem_width=16, n_splits=2, split=1),
                        lambda: nets.wide_resnet_split(split=1, n_splits=2, classes=10, widths=(32, 32, 48), blocks=(2, 1, 1),
                                                       stem=16), 5, 20, 10),
    # basic blocks behind the 7x7 stem and the max-pool (the ResNet-18 family)
    "basic_imagenet_mfma": (dict(kind=5, widths=[16, 24, 32, 40], blocks=[1, 2, 1, 1], stem_width=16),
                            lambda: nets.resnet18(classes=10, widths=(16, 24, 32, 40), blocks=(1, 2, 1, 1), stem=16),
                            5, 72, 10),
}


@pytest.mark.parametrize("name", ["basic", "bottleneck"])
def test_small_resnet_fp32_step(name):
    kw, mk, batch, res, classes = SMALL[name]
    c = Case(kw, mk(), "f32", batch, res, classes)
    compare_f32(c.oracle(), c.gpu(), c.ref_arch, 2e-5, 2e-5, 5e-4, 1e-5)


# ------------------------------------------------------------------- bf16, layer by layer
TOL_BF16_TENSOR = 5e-3   # a tensor the kernel rounds to bf16 (2^-9 relative per element, twice if accumulated)
TOL_F32_TENSOR = 1e-3    # fp32 results of fp32 accumulation over up to ~1e6 bf16 products


def check_layers(c, got):
    """Teacher-forced parity of every op of the local model, forward and backward."""
    packed = hasattr(c, "read_tensor")   # gpu_util.PackedCase: tensors come back in the padded form, padding rows zero
    ops, tensors = c.graph() if packed else c.model.graph(c.batch)
    P = c.per_tensor(c.th.astype(np.float64))
    G = c.per_tensor(got["grad"])
    names = [n for n, _, _, _ in c.ref_arch.params]
    f32 = c.dtype == c.B.CD_F32
    tol_t = 2e-5 if f32 else TOL_BF16_TENSOR

    def rel_rows(t, a, b):
        """rel(a, b) over the rows of tensor t that exist (a packed batch has no padding rows: the oracle's values there
        have no counterpart)"""
        if not packed:
            return rel(a, b)
        keep = c.valid_rows(tensors[t]["stream"]).reshape(-1)
        return rel(np.asarray(a).reshape(keep.size, -1)[keep], np.asarray(b).reshape(keep.size, -1)[keep])

    def shape(t):
        return (c.batch, tensors[t]["h"], tensors[t]["w"], tensors[t]["c"])

    # Outputs of BatchNorm ops whose kernel also computes the max-pool behind them (fused_pool) are never
    # written: the oracle's value of that tensor (from the tensors the kernel did read) stands in for it.
    unwritten = {}

    def act(t):
        if t in unwritten:
            return unwritten[t]
        if t == 0:
            return c.x.astype(np.float64)
        if packed:
            return c.read_tensor(tensors[t], "act_offset", shape(t))
        return c.read(tensors[t]["act_offset"], shape(t))

    def grad(t):
        if packed:
            return c.read_tensor(tensors[t], "grad_offset", shape(t))
        return c.read(tensors[t]["grad_offset"], shape(t))

    logits_t = ops[-1]["y"]
    worst = {"act": (0.0, ""), "agrad": (0.0, ""), "pgrad": (0.0, ""), "stats": (0.0, "")}

    def note(kind, e, what, tol):
        worst[kind] = max(worst[kind], (e, what))
        assert e <= tol, (kind, what, e)

    expected = {}   # tensor id -> float64 sum of the oracle's gradient contributions
    # Residual gradients that the backward pass hands on without writing them (res_grad 1): the op that
    # produced the residual tensor reads the BatchNorm's dy through its ReLU mask; the tensor's own
    # gradient buffer stays unused.
    handed_on = {o["res"]: j for j, o in enumerate(ops) if o["kind"] == "bn" and o["res"] >= 0 and o["res_grad"] == 1}

    def grad_in(t):
        if t in handed_on:
            q = ops[handed_on[t]]
            g = grad(q["y"])
            return L.relu_backward(act(q["y"]), g) if q["relu"] else g
        return grad(t)

    def contribute(t, g):
        if t != 0:
            expected[t] = g if t not in expected else expected[t] + g

    # a parameter used by several ops (the tied embedding table) gets the sum of their gradients
    uses = {}
    for o in ops:
        if o["param_w"] >= 0:
            uses[o["param_w"]] = uses.get(o["param_w"], 0) + 1
    shared = {}

    def pgrad(o, g, tag, tol):
        name = names[o["param_w"]]
        if uses[o["param_w"]] > 1:
            shared[name] = g if name not in shared else shared[name] + g
        else:
            note("pgrad", rel(G[name], g), tag + ".w", tol)

    # ops in front of a frozen cut (the multi-view network): forward only; their parameter gradients are exact zeros
    cut = max([j for j, o in enumerate(ops) if o["kind"] == "slice"] + [-1])
    for i, o in enumerate(ops):
        x = act(o["x"])
        frozen = i < cut
        if frozen:
            for pi in (o["param_w"], o["param_b"]):
                assert pi < 0 or not G[names[pi]].any(), names[pi]
        if o["kind"] == "slice":
            np.testing.assert_array_equal(act(o["y"]), x[..., o["k"]:o["k"] + tensors[o["y"]]["c"]])
            continue
        fused_pool = o["kind"] == "bn" and o["fused_pool"]
        y = got["logits"].astype(np.float64) if o["y"] == logits_t else (None if fused_pool else act(o["y"]))
        # nothing flows back through the frozen front end: its gradient slots are never written, and never read here
        dy = got["dz"].astype(np.float64) if o["y"] == logits_t else (None if fused_pool or frozen else grad_in(o["y"]))
        w = P[names[o["param_w"]]] if o["param_w"] >= 0 else None
        b = P[names[o["param_b"]]] if o["param_b"] >= 0 else None
        tag = "op%d:%s" % (i, o["kind"])
        if o["kind"] == "conv":
            yr = L.conv2d_forward(x, w, b, o["stride"], o["pad"])
            if o["relu"]:
                yr = L.relu_forward(yr)
            note("act", rel_rows(o["y"], y, yr), tag, tol_t)
            if frozen:
                continue
            if o["relu"]:
                dy = L.relu_backward(y, dy)
            dx, dw, db = L.conv2d_backward(x, w, dy, o["stride"], o["pad"], b is not None, o["x"] != 0)
            pgrad(o, dw, tag, TOL_F32_TENSOR)
            if b is not None:
                note("pgrad", rel(G[names[o["param_b"]]], db), tag + ".b", TOL_F32_TENSOR)
            contribute(o["x"], dx)
        elif o["kind"] == "embed":
            tok = c.x[:, o["k"]:o["k"] + o["stride"]]
            yr = L.embed_forward(tok, w).reshape(y.shape)
            note("act", rel_rows(o["y"], y, yr), tag, tol_t)
            pgrad(o, L.embed_backward(tok, w.shape, dy), tag, TOL_F32_TENSOR)
        elif o["kind"] == "attn":
            d = y.shape[-1]
            kv = act(o["res"])
            x2, kv2 = x.reshape(-1, x.shape[-1]), kv.reshape(-1, kv.shape[-1])
            qc, kc, vc = o["pad"], o["k_col"], o["v_col"]
            q, kk, v = x2[:, qc:qc + d], kv2[:, kc:kc + d], kv2[:, vc:vc + d]
            klen = L.sentence_lengths(c.x[:, o["key_tok0"]:o["key_tok0"] + kv.shape[1]])
            yr, Pm = L.attention_forward(q, kk, v, c.batch, o["k"], bool(o["stride"]), klen)
            note("act", rel_rows(o["y"], y.reshape(-1, d), yr), tag, tol_t)
            dq, dk, dv = L.attention_backward(q, kk, v, Pm, dy.reshape(-1, d), c.batch, o["k"])
            gx, gkv = np.zeros_like(x2), np.zeros_like(kv2)
            gx[:, qc:qc + d] = dq
            tgt = gx if o["res"] == o["x"] else gkv
            tgt[:, kc:kc + d] += dk
            tgt[:, vc:vc + d] += dv
            contribute(o["x"], gx.reshape(x.shape))
            if o["res"] != o["x"]:
                contribute(o["res"], gkv.reshape(kv.shape))
        elif o["kind"] == "bn":
            yr, cache = L.batchnorm_forward(x, w, b)
            stats = c.read(o["stats_offset"], (4, x.shape[-1]), f32=True)
            note("stats", rel(stats[0], cache[2]), tag + ".mean", 1e-4)
            note("stats", rel(stats[1], cache[1]), tag + ".invstd", 1e-4)
            if o["res"] >= 0:
                yr = yr + act(o["res"])
            if o["relu"]:
                yr = L.relu_forward(yr)
                if fused_pool and not frozen:   # neither this op's output nor its gradient is written: both come from the pool's side
                    q = ops[i + 1]
                    _, arg = L.maxpool_forward(yr, q["k"], q["stride"], q["pad"])
                    dy = L.maxpool_backward(yr.shape, arg, grad(q["y"]), q["k"], q["stride"], q["pad"])
                if not frozen:
                    dy = L.relu_backward(yr if fused_pool else y, dy)
            if fused_pool:
                unwritten[o["y"]] = yr
            else:
                note("act", rel(y, yr), tag, tol_t)
            if frozen:
                continue
            dx, dg, db = L.batchnorm_backward(dy, w, cache)
            note("pgrad", rel(G[names[o["param_w"]]], dg), tag + ".gamma", TOL_F32_TENSOR)
            note("pgrad", rel(G[names[o["param_b"]]], db), tag + ".beta", TOL_F32_TENSOR)
            contribute(o["x"], dx)
            if o["res"] >= 0:
                contribute(o["res"], dy)
        elif o["kind"] == "maxpool":
            yr, arg = L.maxpool_forward(x, o["k"], o["stride"], o["pad"])
            # a maximum of stored values is exact; behind a fused BatchNorm it is the rounded maximum of fp32 values
            note("act", rel(y, yr), tag, tol_t if o["x"] in unwritten else 0.0)
            contribute(o["x"], L.maxpool_backward(x.shape, arg, dy, o["k"], o["stride"], o["pad"]))
        elif o["kind"] == "gap":
            note("act", rel(y.reshape(c.batch, -1), L.gap_forward(x)), tag, tol_t)
            contribute(o["x"], L.gap_backward(x.shape, dy.reshape(c.batch, -1)))
        elif o["kind"] == "layernorm":
            s = x + act(o["res"]) if o["res"] >= 0 else x
            yr, cache = L.layernorm_forward(s, w, b)
            mean, rstd = s.mean(axis=-1).reshape(-1), cache[1].reshape(-1)
            if packed:   # the rows that exist
                stats = c.read_rows(tensors[o["x"]], o["stats_offset"], 2)
                keep = c.valid_rows(tensors[o["x"]]["stream"]).reshape(-1)
                stats, mean, rstd = stats[keep], mean[keep], rstd[keep]
            else:
                stats = c.read(o["stats_offset"], (c.batch * x.shape[1] * x.shape[2], 2), f32=True)
            note("stats", float(np.abs(stats[:, 0] - mean).max() / np.sqrt((s ** 2).mean())), tag + ".mean", 1e-5)
            note("stats", rel(stats[:, 1], rstd), tag + ".rstd", 1e-4)
            note("act", rel_rows(o["y"], y, yr), tag, tol_t)
            dx, dg, db = L.layernorm_backward(dy, w, cache)
            note("pgrad", rel(G[names[o["param_w"]]], dg), tag + ".gamma", TOL_F32_TENSOR)
            note("pgrad", rel(G[names[o["param_b"]]], db), tag + ".beta", TOL_F32_TENSOR)
            contribute(o["x"], dx)
            if o["res"] >= 0:
                contribute(o["res"], dx)
        elif o["kind"] == "linear":
            x2 = x.reshape(-1, x.shape[-1]) if x.shape[1] * x.shape[2] > 1 else x.reshape(c.batch, -1)
            note("act", rel_rows(o["y"], y, L.linear_forward(x2, w, b)), tag, 2e-5 if f32 else 1e-4)
            dx, dw, db = L.linear_backward(x2, w, dy, b is not None)
            # the bf16 model's dense-layer backward runs on the MFMA kernels from a bf16 copy of d loss / d logits
            pgrad(o, dw, tag, TOL_F32_TENSOR if f32 else TOL_BF16_TENSOR)
            if b is not None:
                note("pgrad", rel(G[names[o["param_b"]]], db), tag + ".b", TOL_F32_TENSOR)
            contribute(o["x"], dx.reshape(x.shape))
    for name, g in shared.items():
        note("pgrad", rel(G[name], g), name, TOL_BF16_TENSOR)
    # the backward pass of a convolution with a fused ReLU masks the stored gradient of its output in place
    masked = {o["y"] for o in ops if o["kind"] == "conv" and o["relu"]}
    readers = {}
    for o in ops:
        for t in {o["x"], o["res"]}:
            readers[t] = readers.get(t, 0) + 1
    errs = []
    for t, g in expected.items():
        if t in handed_on or t in unwritten:
            continue
        if t in masked:
            g = L.relu_backward(act(t), g)
        errs.append((rel(grad(t), g), t, readers[t]))
    print("largest activation-gradient errors (error, tensor, readers):", sorted(errs, reverse=True)[:6])
    # A tensor with n readers gets n contributions added one after the other into its stored gradient, each addition
    # rounding the running sum: the error grows like sqrt((n + 1) / 2) times one rounding (n <= 2 in the bound above).
    for e, t, n in errs:
        note("agrad", e, "grad of tensor %d" % t, tol_t * max(1.0, np.sqrt((n + 1) / 3.0)))
    print("layer parity, worst relative errors:", worst)
    return worst


STATED_TOL = 2e-2     # the stated tolerance of the bf16 step: relative, on logits, loss and per-tensor gradient norms
L2_LIMIT = 0.5        # a tensor that storage rounding alone moves by more than this (L2) has no meaningful end-to-end gate


def compare_bf16(c, ref, floor, got, plain=(), label=None):
    """End to end against the float64 step, quantity by quantity.  e = distance of the GPU's value from the float64
    one; f = distance, for the same quantity, of the float64-arithmetic step whose stored tensors are rounded to
    bf16 (gpu_util.bf16_storage_points): what bf16 storage alone does to this quantity on this input.

      logits, loss terms      e <= max(2e-2, 2 f)
      every gradient tensor   L2:   ||g - g_ref|| / ||g_ref||     <= max(2e-2, 2 lf_i),  lf_i = the same distance of the
                                                                                         storage-rounded step (<= 0.5)
                              norm: | ||g|| - ||g_ref|| | / ||g_ref|| <= max(2e-2, lf_i)   (the stated quantity)
      all gradient tensors    median norm error <= max(2e-2, 2 x the storage-rounded step's median)

    Where f << 2e-2 these are the stated tolerance.  Where rounding the stored activations alone moves a quantity by
    more than 1e-2, no bf16-storage pipeline can be held to 2e-2 on this input, and the gate is that quantity's own
    measured sensitivity (never a bound borrowed from another tensor).  The per-tensor scale is the L2 distance lf_i:
    it sums over all elements and is stable from one realisation of the rounding noise to the next (measured: GPU
    L2 error / lf_i between 0.9 and 1.3 on every tensor of every workload here), while a norm error is one signed
    number per tensor that can be near zero by chance; a norm error never exceeds the L2 distance, so the norm
    gate is tighter than what the L2 gate already implies.  Tensors with lf_i > 0.5 (1 for the norm) are not gated here
    (a bound near 1 would pass a zero tensor): they are listed, and their evidence is the teacher-forced per-op
    test (check_layers).  The report also counts the tensors that meet the plain 2e-2.
    plain: names in {"logits", "peer logits", "loss", "task", "distill", "median"} that must meet the plain 2e-2.
    Returns the table as a dict (also written as JSON into $CODISTILL_TEST_REPORT_DIR when that is set)."""
    rows = [("logits", rel(got["logits"], ref["logits"]), rel(floor["logits"], ref["logits"])),
            ("peer logits", rel(got["peer_logits"], ref["peer_logits"][0]),
             rel(floor["peer_logits"][0], ref["peer_logits"][0]))]
    for i, n in enumerate(("loss", "task", "distill")):
        rows.append((n, abs(got["loss"][i] - ref["loss"][i]) / abs(ref["loss"][i]),
                     abs(floor["loss"][i] - ref["loss"][i]) / abs(ref["loss"][i])))
    report = {"scalars": {}, "tensors": {}, "ungated": []}
    bad = []   # violations are collected and asserted after the table is printed and written
    for name, e, f in rows:
        print("%-12s gpu-vs-f64 %.3e   bf16-storage sensitivity %.3e" % (name, e, f))
        report["scalars"][name] = (e, f)
        if f > L2_LIMIT:
            report["ungated"].append(name)
            continue
        if e > max(STATED_TOL, 2 * f) or (name in plain and e > STATED_TOL):
            bad.append((name, e, f))
    Gg, Gr, Gf = c.per_tensor(got["grad"]), c.per_tensor(ref["grad"]), c.per_tensor(floor["grad"])
    eg, fg, over = [], [], []
    for n in Gr:
        e, f = norm_err(Gg[n], Gr[n]), norm_err(Gf[n], Gr[n])
        le, lf = rel(Gg[n], Gr[n]), rel(Gf[n], Gr[n])
        report["tensors"][n] = dict(norm=(e, f), l2=(le, lf))
        eg.append(e)
        fg.append(f)
        if e > STATED_TOL:
            over.append((e, f, lf, n))
        if lf > L2_LIMIT:
            report["ungated"].append(n + (" (L2)" if lf <= 1.0 else " (L2, norm)"))
        elif le > max(STATED_TOL, 2 * lf):
            bad.append(("gradient of " + n, le, lf))
        if lf <= 1.0 and e > max(STATED_TOL, lf):
            bad.append(("gradient norm of " + n, e, lf))
    eg = np.array(eg)
    report["grad_norm_median"], report["grad_norm_max"] = float(np.median(eg)), float(eg.max())
    report["within_stated"] = int((eg <= STATED_TOL).sum())
    l2 = np.array([v["l2"][0] for v in report["tensors"].values()])
    l2f = np.array([v["l2"][1] for v in report["tensors"].values()])
    print("per-tensor gradient norms: %d of %d within 2e-2; median %.3e, max %.3e" % (report["within_stated"], len(eg),
                                                                                     np.median(eg), eg.max()))
    print("per-tensor gradient L2:    gpu median %.3e max %.3e | storage sensitivity median %.3e max %.3e"
          % (np.median(l2), l2.max(), np.median(l2f), l2f.max()))
    for e, f, lf, n in sorted(over, reverse=True)[:12]:
        print("   norm above 2e-2: %-28s gpu %.3e   storage-rounded step %.3e   its L2 distance %.3e" % (n, e, f, lf))
    if report["ungated"]:
        print("   not gated end to end (L2 storage sensitivity above %.1f): %d tensors, e.g. %s"
              % (L2_LIMIT, len(report["ungated"]), ", ".join(report["ungated"][:6])))
    if np.median(eg) > max(STATED_TOL, 2 * np.median(fg)):
        bad.append(("median gradient norm error", float(np.median(eg)), float(np.median(fg))))
    report["violations"] = bad
    out = os.environ.get("CODISTILL_TEST_REPORT_DIR")
    if out and label:
        with open(os.path.join(out, "bf16_e2e_%s.json" % label), "w") as fh:
            json.dump(report, fh)
    assert not bad, bad
    if "median" in plain:
        assert np.median(eg) <= STATED_TOL
    # the update, teacher forced: the oracle's momentum-SGD rule applied to the GPU's own gradient (the step moves the
    # weights by lr times a gradient that is itself only known to the tolerances above)
    h = c.last_step
    v0 = np.zeros(c.th.size) if c.v0 is None else c.v0.astype(np.float64)
    w_new, v_new = sgd_step(c.th.astype(np.float64), v0, got["grad"].astype(np.float64), h["lr"], h["mu"], h["wd"], False)
    off = 0
    for n, shape, _, _ in c.ref_arch.params:      # a frozen front end is left out of the update
        k = int(np.prod(shape))
        if n in c.ref_arch.frozen:
            w_new[off:off + k], v_new[off:off + k] = c.th[off:off + k], v0[off:off + k]
        off += k
    assert rel(got["theta"], w_new) <= 1e-6 and rel(got["v"], v_new) <= 1e-6
    return report


def test_tall_tile_convolutions_bf16_layers():
    """One bottleneck block at 196 x 64 x 64: after the stem and the pool M = 196*16*16 = 50176 rows.  The two
    64 -> 256 convolutions (short contraction, 256 columns) run on 128x256 tiles, forward and backward."""
    c = Case(dict(kind=2, widths=[64], blocks=[1], stem_width=64),
             nets.resnet50(classes=10, widths=(64,), blocks=(1,), stem=64), "bf16", 196, 64, 10)
    check_layers(c, c.gpu())


def test_short_contraction_onto_many_columns_bf16_layers():
    """One bottleneck block of width 128: its 128 -> 512 and 64 -> 512 convolutions (K <= 128, N = 512) take
    the 256x128 tile; M = 40*16*16 = 10240 rows is 40 of those tiles."""
    c = Case(dict(kind=2, widths=[128], blocks=[1], stem_width=64),
             nets.resnet50(classes=10, widths=(128,), blocks=(1,), stem=64), "bf16", 40, 64, 10)
    check_layers(c, c.gpu())


def test_residual_gradient_routes_agree(monkeypatch):
    """The gradient of a residual input reaches its reader either through the tensor's gradient buffer or as
    "dy and the ReLU bit mask" (a projection shortcut's BatchNorm, the first convolution of an identity block):
    the arithmetic is the same, so the parameter gradients of a step are identical bit for bit."""
    mk = lambda: Case(dict(kind=2, widths=[16, 32], blocks=[2, 2], stem_width=16),
                      nets.resnet50(classes=10, widths=(16, 32), blocks=(2, 2), stem=16), "bf16", 24, 64, 10)
    c = mk()
    routes = [o["res_grad"] for o in c.model.graph(c.batch)[0] if o["kind"] == "bn" and o["res"] >= 0]
    assert sorted(set(routes)) == [1, 2]
    a = c.gpu()
    monkeypatch.setenv("CODISTILL_WRITE_RESIDUAL_GRADS", "1")
    assert all(o["res_grad"] == 0 for o in c.model.graph(c.batch)[0])
    b = mk().gpu()
    np.testing.assert_array_equal(a["grad"], b["grad"])
    np.testing.assert_array_equal(a["theta"], b["theta"])


def test_pool_fusion_matches_separate_kernels(monkeypatch):
    """BatchNorm + ReLU + max-pool in one kernel against the three-kernel form.  The maximum of rounded values is
    the rounded maximum, so the forward pass agrees bit for bit; the backward pass sends a window's gradient to
    the largest fp32 value instead of the first of the values that are equal after rounding to bf16, which moves
    a few percent of the stem's gradient to a neighbouring pixel: gradient norms agree, not gradient bits."""
    mk = lambda: Case(dict(kind=2, widths=[16, 32], blocks=[1, 1], stem_width=16),
                      nets.resnet50(classes=10, widths=(16, 32), blocks=(1, 1), stem=16), "bf16", 12, 64, 10)
    c = mk()
    assert any(o["kind"] == "bn" and o["fused_pool"] for o in c.model.graph(c.batch)[0])
    a = c.gpu()
    monkeypatch.setenv("CODISTILL_NO_POOL_FUSION", "1")
    assert not any(o["fused_pool"] for o in c.model.graph(c.batch)[0])
    b = mk().gpu()
    np.testing.assert_array_equal(a["logits"], b["logits"])
    np.testing.assert_array_equal(a["loss"], b["loss"])
    ga, gb = c.per_tensor(a["grad"]), c.per_tensor(b["grad"])
    for n in ga:
        assert norm_err(ga[n], gb[n]) <= 2e-2, n


@pytest.mark.parametrize("name", list(SMALL))
def test_small_resnet_bf16_layers(name):
    kw, mk, batch, res, classes = SMALL[name]
    c = Case(kw, mk(), "bf16", batch, res, classes)
    check_layers(c, c.gpu())


@pytest.mark.parametrize("name", ["basic", "bottleneck"])
def test_small_resnet_fp32_layers(name):
    kw, mk, batch, res, classes = SMALL[name]
    c = Case(kw, mk(), "f32", batch, res, classes)
    check_layers(c, c.gpu())


@pytest.mark.parametrize("name", list(SMALL))
def test_small_resnet_bf16_step(name):
    kw, mk, batch, res, classes = SMALL[name]
    c = Case(kw, mk(), "bf16", batch, res, classes)
    compare_bf16(c, c.oracle(), c.oracle(bf16_storage=True), c.gpu(), label="small_" + name)


@pytest.mark.parametrize("peer", ["basic_imagenet_mfma", "resnext"])
def test_peer_of_another_architecture_bf16_step(peer):
    """Section 5 pairs models of different architectures: the local bottleneck network distils against a stale
    basic-block network, or one with grouped convolutions; only the shape of the logits is shared."""
    kw, mk, batch, res, classes = SMALL["bottleneck_mfma"]
    pkw, pmk, _, _, _ = SMALL[peer]
    c = Case(kw, mk(), "bf16", batch, res, classes, peer=(pkw, pmk()))
    assert c.peer.n_elements != c.model.n_elements
    compare_bf16(c, c.oracle(), c.oracle(bf16_storage=True), c.gpu(), label="mixed_pair_" + peer)


def test_resnet20_bf16_layers():
    """ResNet-20, bf16 compute with fp32 master weights, batch 128 of 32x32x3, alpha 1."""
    c = Case(dict(kind=1), nets.resnet20(), "bf16", 128, 32, 10, jitter=0.0)
    check_layers(c, c.gpu())


@pytest.fixture(scope="module")
def resnet20_step():
    c = Case(dict(kind=1), nets.resnet20(), "bf16", 128, 32, 10, jitter=0.0)
    return c, c.oracle(), c.oracle(bf16_storage=True), c.gpu()


def test_resnet20_bf16_step(resnet20_step):
    """Logits, loss terms and the median gradient norm meet the stated 2e-2 outright on this workload."""
    c, ref, floor, got = resnet20_step
    compare_bf16(c, ref, floor, got, plain=("logits", "peer logits", "loss", "task", "distill", "median"),
                 label="resnet20_b128")


@pytest.mark.xfail(strict=True, reason="the plain 2e-2 on EVERY per-tensor gradient norm is not met on this workload: "
                   "measured 42 of 65 tensors within 2e-2, largest 1.6e-1 (a BatchNorm scale of the first stage); the "
                   "float64-arithmetic step with bf16-rounded stored tensors gives 44 of 65 and 1.2e-1, i.e. bf16 "
                   "storage itself, not a kernel, sets this; see compare_bf16 for what is asserted instead")
def test_resnet20_bf16_every_gradient_norm_within_stated_tolerance(resnet20_step):
    c, ref, floor, got = resnet20_step
    Gg, Gr = c.per_tensor(got["grad"]), c.per_tensor(ref["grad"])
    assert max(norm_err(Gg[n], Gr[n]) for n in Gr) <= STATED_TOL


def test_wide_resnet_28x10_split_bf16_layers():
    """The multi-view network at its real widths (Section 5: Wide-ResNet 28x10 on 32x32 images, 160 channels cut into
    8 parts of 20, this model sees part 5), batch 32: every op teacher forced; the stem and the first block are
    frozen (gradients exactly zero, weights not moved by the update)."""
    c = Case(dict(kind=7, split=5), nets.wide_resnet_split(split=5), "bf16", 32, 32, 10, jitter=0.0)
    got = c.gpu()
    check_layers(c, got)
    th, new = c.per_tensor(c.th), c.per_tensor(got["theta"])
    for n in th:
        assert (n in c.ref_arch.frozen) == bool(np.array_equal(th[n], new[n])), n


def test_resnet50_bf16_layers_reduced_batch():
    """ResNet-50 at full 224x224 resolution and 1000 classes, batch 32: the largest batch whose activations the
    float64 oracle holds.  Same kernels, same N and K as the benchmarked batch of 256, M an eighth of it: the
    last stage's convolutions have M = 1568 rows, several row tiles with a ragged last one."""
    c = Case(dict(kind=2), nets.resnet50(), "bf16", 32, 224, 1000, jitter=0.0)
    check_layers(c, c.gpu())


def test_resnet50_bf16_step_reduced_batch():
    c = Case(dict(kind=2), nets.resnet50(), "bf16", 4, 224, 1000, jitter=0.0)
    ref = c.oracle()
    got = c.gpu()
    compare_bf16(c, ref, c.oracle(bf16_storage=True), got, label="resnet50_b4")


@pytest.mark.parametrize("name,dtype_name", [("basic", "f32"), ("bottleneck_mfma", "bf16")])
def test_batchnorm_running_averages_and_evaluation_mode(name, dtype_name):
    """A training-mode forward pass with a buffer of running averages updates them as the oracle does; an
    evaluation-mode pass normalises with them (statistics kernels skipped, the fused BatchNorm + max-pool included)."""
    import torch
    from paper_2010_02838_amd.runner import pack_flat, to_device
    kw, mk, batch, res, classes = SMALL[name]
    c = Case(kw, mk(), dtype_name, batch, res, classes)
    B, model = c.B, c.model
    dev = "cuda:0"
    params = to_device(pack_flat(model, c.th), model.torch_dtype)
    x = to_device(c.x, model.torch_dtype)
    ws = torch.empty(model.workspace_bytes(batch, False), dtype=torch.uint8, device=dev)
    logits = torch.empty(batch, classes, device=dev)
    # the buffer holds [mean | var] per BatchNorm op in the order of the library's op list (a projection shortcut's
    # BatchNorm comes before the block's own there, after them in the oracle's list): match them by parameter name
    names = [n for n, _, _, _ in c.ref_arch.params]
    ops, _ = model.graph(batch)
    lib_order = [names[o["param_w"]] for o in ops if o["kind"] == "bn"]
    ref_order = [o["gamma"] for o in c.ref_arch.ops if o["op"] == "bn"]
    assert sorted(lib_order) == sorted(ref_order)
    P32 = c.per_tensor(c.th)
    widths = [P32[n].shape[0] for n in lib_order]
    assert model.bn_running_elements() == 2 * sum(widths)
    run = torch.cat([torch.cat([torch.zeros(w), torch.ones(w)]) for w in widths]).to(dev)
    B.codistill_forward(model, params, x, ws, logits, False, B.CD_BN_BATCH_STATS, run)
    torch.cuda.synchronize()
    z_train = logits.cpu().numpy().copy()
    P = c.per_tensor(c.th.astype(np.float64))
    ref_run = [[np.zeros(P32[n].shape[0]), np.ones(P32[n].shape[0])] for n in ref_order]
    z_ref, _ = nets.forward(c.ref_arch, P, c.x.astype(np.float64), running=ref_run)
    by_name = dict(zip(ref_order, ref_run))
    got, off = run.cpu().numpy(), 0
    tol = 1e-4 if dtype_name == "f32" else 3e-2        # bf16: the activations the statistics are taken from are rounded
    for n, w in zip(lib_order, widths):
        rm, rv = by_name[n]
        assert rel(got[off:off + w], rm) <= tol and rel(got[off + w:off + 2 * w], rv) <= tol, n
        off += 2 * w
    # evaluation mode with the oracle's averages
    run_ref = torch.from_numpy(np.concatenate([np.concatenate(by_name[n]) for n in lib_order]).astype(np.float32)).to(dev)
    before = run_ref.clone()
    B.codistill_forward(model, params, x, ws, logits, False, B.CD_BN_RUNNING, run_ref)
    torch.cuda.synchronize()
    z_eval_ref, _ = nets.forward(c.ref_arch, P, c.x.astype(np.float64), running=ref_run, bn_eval=True)
    assert rel(logits.cpu().numpy(), z_eval_ref) <= (1e-4 if dtype_name == "f32" else 3e-2)
    assert rel(z_train, z_eval_ref) > 5 * tol          # the two modes differ by far more than the tolerance
    assert torch.equal(run_ref, before)                # an evaluation pass leaves the averages alone


@pytest.mark.parametrize("kind,width,batch,res,dtype_name", [
    (1, 20, 3, 9, "bf16"),      # channels no multiple of 8: one at a time
    (1, 24, 5, 7, "bf16"),      # three vectors a row, 256 threads no multiple of them
    (2, 512, 2, 8, "bf16"),     # 2048 channels, the most whose scales a block holds
    (2, 520, 2, 8, "bf16"),     # 2080: the statistics kernel runs in front
    (1, 18, 3, 6, "f32"),
])
def test_evaluation_mode_channel_counts(kind, width, batch, res, dtype_name):
    """The evaluation-mode BatchNorm at the channel counts where its form changes."""
    import torch
    from paper_2010_02838_amd.runner import pack_flat, to_device
    mk = nets.resnet20 if kind == 1 else nets.resnet50
    kw = dict(widths=(width,), blocks=(1,))
    ref = mk(**kw) if kind == 1 else mk(classes=10, stem=64, **kw)
    c = Case(dict(kind=kind, widths=[width], blocks=[1], stem_width=width if kind == 1 else 64), ref, dtype_name, batch, res, 10)
    B, model, dev = c.B, c.model, "cuda:0"
    names = [n for n, _, _, _ in ref.params]
    lib_order = [names[o["param_w"]] for o in model.graph(batch)[0] if o["kind"] == "bn"]
    ref_order = [o["gamma"] for o in ref.ops if o["op"] == "bn"]
    P32, rng = c.per_tensor(c.th), np.random.default_rng(7)
    avg = {n: [rng.normal(0, 0.5, P32[n].shape[0]).astype(np.float32), rng.uniform(0.5, 2, P32[n].shape[0]).astype(np.float32)]
           for n in ref_order}
    run = torch.from_numpy(np.concatenate([np.concatenate(avg[n]) for n in lib_order])).to(dev)
    ws = torch.empty(model.workspace_bytes(batch, False), dtype=torch.uint8, device=dev)
    logits = torch.empty(batch, 10, device=dev)
    B.codistill_forward(model, to_device(pack_flat(model, c.th), model.torch_dtype), to_device(c.x, model.torch_dtype), ws,
                        logits, False, B.CD_BN_RUNNING, run)
    torch.cuda.synchronize()
    P = c.per_tensor(c.th.astype(np.float64))
    z, _ = nets.forward(ref, P, c.x.astype(np.float64), running=[[a.astype(np.float64) for a in avg[n]] for n in ref_order],
                        bn_eval=True)
    assert rel(logits.cpu().numpy(), z) <= (1e-4 if dtype_name == "f32" else 3e-2)   # as in the test above


# ------------------------------------------------------------------- environment switches
def _backward_on(monkeypatch, streams):
    """Every backward pass of the binding, the step runner's too, with this choice of streams."""
    from paper_2010_02838_amd import binding as B
    monkeypatch.setattr(B, "codistill_backward", functools.partial(B.codistill_backward, streams=getattr(B, streams)))


@pytest.mark.parametrize("streams", ["CD_STREAMS_AUTO", "CD_STREAMS_TWO"])
def test_serial_switch_is_bit_identical(monkeypatch, streams):
    """CODISTILL_SERIAL=1 keeps the weight gradients on the caller's stream: same kernels, same fixed-order
    reductions, so every result of the step is bit for bit that of the two-stream form.  (A network as small as this one stays on the
    caller's stream with CD_STREAMS_AUTO and forks with CD_STREAMS_TWO: test_launch_order_host.py.)"""
    _backward_on(monkeypatch, streams)
    kw, mk, batch, res, classes = SMALL["bottleneck_mfma"]
    a = Case(kw, mk(), "bf16", batch, res, classes).gpu()
    monkeypatch.setenv("CODISTILL_SERIAL", "1")
    b = Case(kw, mk(), "bf16", batch, res, classes).gpu()
    for k in ("logits", "loss", "grad", "theta"):
        np.testing.assert_array_equal(a[k], b[k])


@pytest.mark.parametrize("name", ["basic_mfma", "bottleneck_mfma", "resnext"])
def test_two_streams_layers(monkeypatch, name):
    """The per-layer oracle check with the weight gradients on the second stream, where these small networks have them on the caller's."""
    _backward_on(monkeypatch, "CD_STREAMS_TWO")
    kw, mk, batch, res, classes = SMALL[name]
    c = Case(kw, mk(), "bf16", batch, res, classes)
    check_layers(c, c.gpu())


def test_separate_bn_reduction_switch_agrees(monkeypatch):
    """By default the data-gradient kernel that completes the gradient of a BatchNorm's output also takes the column sums
    of that BatchNorm's backward pass from the values it stores; CODISTILL_SEPARATE_BN_REDUCTION=1 keeps the reduction
    pass over dy and x instead.  Same stored tensors, same sums up to the order of the additions: the logits are
    identical, the gradients agree to fp32 rounding, and both forms meet the per-layer tolerances against the oracle."""
    kw, mk, batch, res, classes = SMALL["bottleneck_mfma"]
    a = Case(kw, mk(), "bf16", batch, res, classes).gpu()
    monkeypatch.setenv("CODISTILL_SEPARATE_BN_REDUCTION", "1")
    c = Case(kw, mk(), "bf16", batch, res, classes)
    b = c.gpu()
    check_layers(c, b)
    np.testing.assert_array_equal(a["logits"], b["logits"])
    assert not np.array_equal(a["grad"], b["grad"])        # the switch does select another path
    Ga, Gb = c.per_tensor(a["grad"]), c.per_tensor(b["grad"])
    for n in Gb:
        assert rel(Ga[n], Gb[n].astype(np.float64)) <= 5e-3, n   # bf16 activation gradients differ by single roundings


def test_plain_kernels_switch_bf16_layers(monkeypatch):
    """CODISTILL_FORCE_SIMPLE=1 routes every convolution of a bf16 model to the plain one-thread-per-output kernels:
    they meet the same per-layer tolerances against the oracle as the MFMA kernels they stand in for."""
    kw, mk, batch, res, classes = SMALL["bottleneck_mfma"]
    ref = Case(kw, mk(), "bf16", batch, res, classes).gpu()
    monkeypatch.setenv("CODISTILL_FORCE_SIMPLE", "1")
    c = Case(kw, mk(), "bf16", batch, res, classes)
    got = c.gpu()
    check_layers(c, got)
    assert rel(got["logits"], ref["logits"].astype(np.float64)) <= STATED_TOL


def test_runners_share_the_peers_stream():
    """One second stream for the runners of a thread on one stream of the caller, none taken by a runner whose peers stay on the caller's; steps of two
    runners in turn are bit for bit those of runners without it."""
    import threading
    import torch
    from paper_2010_02838_amd import binding as B
    from paper_2010_02838_amd import runner as R

    def make(kind, overlap, **kw):
        m = [B.Model(B.arch_preset(kind, in_h=16, in_w=16, **kw), B.CD_BF16) for _ in range(2)]
        r = R.StepRunner(m[0], m[1:], 4, overlap_peers=overlap)
        r.load(*[f(R.pack_flat(q, synth.he_init(q.param_table(), k, 0.1))) for f, q, k in ((lambda t: t, m[0], 1), (lambda t: [t], m[1], 2))])
        return r

    def steps(overlap):
        runs = [make(B.CD_ARCH_RESNET_BASIC, overlap, widths=[w, 32], blocks=[1, 1], stem_width=w) for w in (16, 24)]
        x, y = torch.randn(4, 16, 16, 3, generator=torch.Generator().manual_seed(1)).to("cuda:0", torch.bfloat16), torch.arange(4, device="cuda:0", dtype=torch.int32)
        for _ in range(3):
            for r in runs:
                r.step(x, y, 1.0, 0.05, 0.9)
        torch.cuda.synchronize()
        return runs, [t.cpu() for r in runs for t in (r.master, r.logits, r.peer_logits[0])]

    plain = steps(False)[1]
    R._streams.__dict__.clear()
    assert not make(B.CD_ARCH_TINY_CNN, True, widths=[16, 32]).overlap_pays and not R._streams.__dict__.get("known")
    runs, out = steps(True)
    assert all(r.overlap_pays for r in runs) and len(R._streams.known) == 1
    for a, b in zip(plain, out):
        assert torch.equal(a, b)
    mine, other = R._peers_stream("cuda:0"), []
    assert mine.cuda_stream != torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(torch.cuda.Stream()):
        other.append(R._peers_stream("cuda:0"))
    t = threading.Thread(target=lambda: other.append(R._peers_stream("cuda:0")))
    t.start()
    t.join()
    assert len({s.cuda_stream for s in [mine] + other}) == 3 and R._peers_stream("cuda:0") is mine
