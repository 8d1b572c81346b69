"""The order of the backward pass's launches on its two streams, what happens where the runtime refuses one of its forks, and which
kernels a call takes on either side of a rule's line: looked at on the host, with a stand-in for the HIP runtime that enqueues nothing
(fake_hip.cpp)."""
import json
import os
import subprocess
import sys

import pytest

from paper_2010_02838_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))
MODELS = {
    "basic": dict(kind=B.CD_ARCH_RESNET_BASIC, dtype="bf16", batch=16, arch=dict(in_h=32, in_w=32, widths=[32, 64], blocks=[2, 2])),
    "big_stem": dict(kind=B.CD_ARCH_RESNET_BOTTLENECK, dtype="bf16", batch=4, arch=dict(in_h=64, in_w=64, widths=[64, 128], blocks=[1, 1])),
    "transformer": dict(kind=B.CD_ARCH_TRANSFORMER, dtype="bf16", batch=8, arch=dict(in_h=64, in_w=64, classes=512, widths=[256, 1024, 4], blocks=[1, 1])),
}


@pytest.fixture(scope="module")
def backward(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.cpp"), "-o", lib], check=True)

    def run(model, fail=None, call="backward", **env):
        req = dict(MODELS[model] if isinstance(model, str) else model, fail=fail, call=call)
        out = subprocess.run([sys.executable, os.path.join(HERE, "launch_log.py"), lib, json.dumps(req)],
                             check=True, capture_output=True, text=True, env=dict(os.environ, **env)).stdout
        return json.loads(out)
    return run


def _kernels(r, stream=None):
    return sorted(name for what, s, name, _ in r["log"] if what == "launch" and (stream is None or (s == r["main"]) == stream))


def _forks(r):
    """Checks that every run of launches on the second stream stands right behind a record on the caller's stream and a wait for it
    that both went well, and that the caller's stream waits for the last of them; returns the number of runs."""
    main, log, runs = r["main"], r["log"], 0
    last_side = -1
    for k, (what, s, name, code) in enumerate(log):
        if what != "launch" or s == main:
            continue
        last_side = k
        if log[k - 1][0] == "launch" and log[k - 1][1] == s:
            continue
        runs += 1
        (w0, s0, e0, c0), (w1, s1, e1, c1) = log[k - 2], log[k - 1]
        assert (w0, s0, c0, w1, s1, c1) == ("record", main, 0, "wait", s, 0) and e0 == e1, log[k - 3:k + 1]
    if runs:
        behind = [x for x in log[last_side + 1:] if x[0] != "launch"]
        assert [(x[0], x[1] == main) for x in behind[-2:]] == [("record", False), ("wait", True)] and behind[-2][2] == behind[-1][2]
    return runs


@pytest.mark.parametrize("name", list(MODELS))
def test_weight_gradients_run_on_the_second_stream(backward, name):
    r = backward(name)
    assert r["rc"] == 0 and _forks(r) >= 1
    assert any("wgrad_kernel" in k for k in _kernels(r, False))
    assert all("wgrad" in k or "unpack" in k or "unpad" in k for k in _kernels(r, False))
    serial = backward(name, CODISTILL_SERIAL="1")
    assert serial["rc"] == 0 and not _kernels(serial, False)
    assert _kernels(serial) == _kernels(r)


@pytest.mark.parametrize("name", list(MODELS))
@pytest.mark.parametrize("call", ["hipEventRecord", "hipStreamWaitEvent"])
def test_refused_fork_runs_on_the_callers_stream(backward, name, call):
    """The launches of a fork whose event cannot be recorded, or waited for, go to the caller's stream (with what belongs to them, the
    unpacking of a stem's gradient); the call succeeds, the other forks stay, and the same kernels run."""
    whole = backward(name)
    forks = _forks(whole)
    for n in range(1, forks + 1):
        r = backward(name, fail=[call, n])
        assert r["rc"] == 0, r["error"]
        assert sum(code != 0 for _, _, _, code in r["log"]) == 1
        assert _forks(r) == forks - 1
        assert _kernels(r) == _kernels(whole)
        assert any("wgrad_kernel" in k for k in _kernels(r, True))


def test_refused_join_is_reported(backward):
    forks = _forks(backward("basic"))
    r = backward("basic", fail=["hipEventRecord", forks + 1])
    assert r["rc"] == B.CD_ERR_HIP and "join" in r["error"]


@pytest.mark.parametrize("batch,folds", [(200, 0), (201, 2)])
def test_fold_of_many_backward_sums(backward, batch, folds):
    """A data gradient of 128-row tiles leaves 8 partial sums an image: 1600 of them are added up as they are, 1608 folded
    first (two BatchNorms with a convolution right behind them)."""
    r = backward(dict(kind=B.CD_ARCH_RESNET_BASIC, dtype="bf16", batch=batch, arch=dict(in_h=32, in_w=32, widths=[72], blocks=[1], stem_width=72)))
    assert r["rc"] == 0 and sum("col_fold_k" in k for k in _kernels(r)) == folds


@pytest.mark.parametrize("rows,features,classes,small", [
    (16384, 64, 64, 1), (16385, 64, 64, 0), (16384, 56, 64, 0), (16384, 64, 65, 1), (16385, 64, 65, 0)])
def test_tiles_of_a_classifier(backward, rows, features, classes, small):
    """At most 64 classes: 64x64 tiles up to 16384 rows, if the features fill a 64-wide step (65 classes: two columns of 64x64 tiles for each of
    128x128, up to the same number of rows)."""
    r = backward(dict(kind=B.CD_ARCH_TRANSFORMER_HEAD, dtype="bf16", batch=rows, arch=dict(widths=[features, 64], classes=classes)), call="forward")
    logits = [k for k in _kernels(r) if "igemm_kernel" in k and "ELb1ELi0ELi1ELb0" in k]   # fp32 output
    assert r["rc"] == 0 and len(logits) == 1 and ("ILi0ELi64ELi64E" in logits[0]) == bool(small), logits


@pytest.mark.parametrize("classes,groups", [(512, 16), (513, 4)])
def test_row_groups_of_a_dense_weight_gradient(backward, classes, groups):
    """256 and 258 blocks of 64 features and 4 classes."""
    r = backward(dict(kind=B.CD_ARCH_TRANSFORMER_HEAD, dtype="f32", batch=70, arch=dict(widths=[64, 8], classes=classes)))
    dw = [k for k in _kernels(r) if "linear_dw_k" in k]
    assert r["rc"] == 0 and len(dw) == 1 and "IfLi%dEE" % groups in dw[0], dw


@pytest.mark.parametrize("features,matrix", [(2040, 1), (2048, 0)])
def test_dense_layer_on_very_many_inputs(backward, features, matrix):
    """2^20 rows: the matrix-core kernel takes inputs of fewer than 2^31 elements (its offsets are 32 bits wide: of 2^31 and more it read
    zeros, or other rows), the plain kernel the rest."""
    r = backward(dict(kind=B.CD_ARCH_TRANSFORMER_HEAD, dtype="bf16", batch=1 << 20, arch=dict(widths=[features, 8], classes=8)), call="forward")
    assert r["rc"] == 0
    assert sum("igemm_kernel" in k and "ELb1ELi0ELi1ELb0" in k for k in _kernels(r)) == matrix
    assert sum("linear_fwd_k" in k for k in _kernels(r)) == 1 - matrix


@pytest.mark.parametrize("peers", [1, 2])
@pytest.mark.parametrize("rows,cols,counted", [(1024, 1024, 0), (1025, 12, 1), (1283, 749, 1), (64, 1025, 1)])
def test_launch_that_counts_the_valid_rows_of_a_loss(backward, peers, rows, cols, counted):
    """Up to 1024 rows of 1024 columns the row kernel counts for itself; above that a launch in front is the shorter way."""
    r = backward(dict(loss=[rows, cols, peers]))
    assert r["rc"] == 0
    assert sum("loss_prep_kernel" in k for k in _kernels(r)) == counted
    assert sum("loss_row_generic_kernel" in k for k in _kernels(r)) == peers - 1


@pytest.mark.parametrize("batch,apart", [(16, 0), (80, 0), (200, 1)])
def test_weight_gradients_of_a_small_network_at_the_end_of_the_pass(backward, batch, apart):
    """With CD_STREAMS_AUTO the layers of a small network (less than 65536 tile steps in all) go at the end, on the caller's stream, a class to a
    launch and nothing forked; a larger one forks as CD_STREAMS_TWO does."""
    model = dict(MODELS["basic"], batch=batch)
    auto, two = backward(model, call="backward_auto"), backward(model)
    assert auto["rc"] == two["rc"] == 0 and _forks(two) >= 1
    assert (_forks(auto) >= 1) == bool(apart)
    names = [n for what, _, n, _ in auto["log"] if what == "launch"]
    if apart:
        assert auto["log"] == two["log"]
    else:
        assert not any(what in ("record", "wait") for what, _, _, _ in auto["log"])
        waiting = [k for k, n in enumerate(names) if "wgrad_kernel" in n and "Li16EE" in n]
        assert waiting and min(waiting) > max(k for k, n in enumerate(names) if "igemm_kernel" in n)
    assert sum("wgrad_kernel" in n for n in names) <= sum("wgrad_kernel" in k for k in _kernels(two))


@pytest.mark.parametrize("batch,finalizes,reductions,folds", [(32, 0, 0, 0), (33, 3, 0, 0), (64, 1, 0, 0), (65, 6, 0, 0), (128, 5, 1, 0), (129, 6, 0, 1),
                                                              (201, 6, 0, 3), (400, 6, 0, 3)])
def test_launches_behind_the_column_sums_of_a_generic_convolution(backward, batch, finalizes, reductions, folds):
    """A two-block fp32 network: the BatchNorm adds up what its convolution left by itself, or behind a finalize, or behind an fp64 fold and a finalize:
    no more launches in front of any of its six elementwise passes than a reduction is (one where the tensor has at most 8 MB, else two)."""
    model = dict(kind=B.CD_ARCH_RESNET_BASIC, dtype="f32", batch=batch, arch=dict(in_h=32, in_w=32, widths=[16, 32], blocks=[1, 1], stem_width=16))
    r = backward(model, call="forward")
    assert r["rc"] == 0
    names = _kernels(r)
    count = lambda part: sum(part in k for k in names)   # noqa: E731
    assert count("conv_generic_k") == 6 and count("col_fold_kIfE") == 0
    assert (count("col_finalize_k"), count("col_reduce_k"), count("col_fold_kIdE")) == (finalizes, reductions, folds)
    assert len(names) == 14 + finalizes + reductions + folds <= (20 if batch <= 128 else 26)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("width,batch,h,w", [(12, 69, 31, 31), (36, 5, 17, 17), (5, 3, 13, 13), (12, 69, 1, 961), (36, 5, 1, 289), (5, 3, 1, 169)])
def test_generic_convolutions_leave_column_sums(backward, dtype, width, batch, h, w):
    """No reduction pass in front of the BatchNorms whose statistics test_gpu_generic_conv.py compares."""
    r = backward(dict(kind=B.CD_ARCH_RESNET_BASIC, dtype=dtype, batch=batch, arch=dict(in_h=h, in_w=w, widths=[width], blocks=[1], stem_width=width)), call="forward")
    assert r["rc"] == 0
    assert sum("conv_generic_k" in k for k in _kernels(r)) == 3 and not any("col_reduce_k" in k for k in _kernels(r))


@pytest.mark.parametrize("arch", [dict(kind=B.CD_ARCH_RESNET_BASIC, arch=dict(in_h=32, in_w=32, widths=[16, 32], blocks=[1, 1], stem_width=16)),
                                  dict(kind=B.CD_ARCH_RESNET_BOTTLENECK, arch=dict(in_h=96, in_w=96, widths=[64, 128], blocks=[1, 1])),
                                  dict(kind=B.CD_ARCH_RESNET_BOTTLENECK, arch=dict(in_h=64, in_w=64, widths=[16], blocks=[1]))])
def test_a_growing_batch_leaves_the_callers_stream_once(backward, arch):
    """Layers go by themselves once a batch is large, and their work counts like that of the waiting ones: from some batch on the pass forks as
    CD_STREAMS_TWO does, and below it has no event and no wait at all, layers by themselves included (the third network has one at its smallest sizes)."""
    forked = []
    for batch in (4, 32, 70, 120, 160, 226, 400, 512, 800, 1024, 2048):
        model = dict(arch, dtype="bf16", batch=batch)
        auto, two = backward(model, call="backward_auto"), backward(model)
        assert auto["rc"] == two["rc"] == 0
        forked.append(_forks(auto) >= 1)
        if forked[-1]:
            assert auto["log"] == two["log"]
        else:
            assert not any(what in ("record", "wait") for what, _, _, _ in auto["log"])
    assert forked == sorted(forked) and forked[-1] and not forked[0]


def test_small_networks_fork_with_two_streams_only(backward):
    """The network whose two-stream pass test_gpu_step.py compares bit for bit with the one-stream pass: the first forks, AUTO does not."""
    model = dict(kind=B.CD_ARCH_RESNET_BOTTLENECK, dtype="bf16", batch=5, arch=dict(in_h=72, in_w=72, classes=10, widths=[8, 16, 24, 32], blocks=[2, 1, 1, 1], stem_width=16))
    two, auto, serial = backward(model), backward(model, call="backward_auto"), backward(model, CODISTILL_SERIAL="1")
    assert _forks(two) >= 4 and _forks(auto) == _forks(serial) == 0
    assert _kernels(two) == _kernels(serial)


def test_streams_argument_is_checked():
    m = B.Model(B.arch_preset(B.CD_ARCH_TINY_CNN), B.CD_F32)
    at = [k << 32 for k in range(1, 7)]
    for streams in (-1, 2):
        assert B.lib.codistill_backward_streams(m._h, at[0], at[1], 2, at[2], 1 << 40, at[3], at[4], streams, None) == B.CD_ERR_INVALID_ARG
