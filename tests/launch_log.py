"""What the library enqueues, in order, without a GPU: `python launch_log.py FAKE_LIBRARY REQUEST` (a JSON object: kind, dtype, arch,
batch, and optionally call = "forward" (saving for a backward pass) or "backward_auto" and fail = [function, n-th call]) prints the log of one
codistill_backward or codistill_forward call as JSON; loss = [rows, columns, peers] in its place that of a codistill_loss_grad.

A process of its own: the stand-in for the HIP runtime (fake_hip.cpp) has to be loaded before anything else that uses HIP.  The
pointers that it hands over are never read, on the host or anywhere else."""
import ctypes
import json
import os
import sys
import types

if __name__ == "__main__":
    fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    fake.fake_hip_log.restype = ctypes.c_char_p
    sys.modules["torch"] = types.SimpleNamespace(bfloat16="bf16", float32="f32")   # (the binding needs it for device memory and streams only)
    sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    from paper_2010_02838_amd import binding as B

    req = json.loads(sys.argv[2])
    at = lambda k: ctypes.c_void_p(k << 32)   # noqa: E731
    m = None if "loss" in req else B.Model(B.arch_preset(req["kind"], **req["arch"]), B.CD_BF16 if req["dtype"] == "bf16" else B.CD_F32)
    fake.fake_hip_reset()
    if req.get("fail"):
        fake.fake_hip_fail(req["fail"][0].encode(), ctypes.c_long(req["fail"][1]))
    if not m:
        rows, cols, peers = req["loss"]
        cfg = B.LossCfg(1.0, 0.0, B.CD_DIST_KL, B.CD_MEAN_ALL, -1, peers, 1.0)
        rc = B.lib.codistill_loss_grad(at(1), (ctypes.c_void_p * max(peers, 1))(*[at(8 + j) for j in range(peers)]), at(2), rows, cols,
                                       ctypes.byref(cfg), at(4), at(5), at(3), 1 << 30, at(6))
    elif req.get("call") == "forward":
        rc = B.lib.codistill_forward(m._h, at(1), at(2), req["batch"], 1, B.CD_BN_BATCH_STATS, None, at(3), m.workspace_bytes(req["batch"], True), at(4), at(6))
    elif req.get("call") == "backward_auto":
        rc = B.lib.codistill_backward_streams(m._h, at(1), at(2), req["batch"], at(3), m.workspace_bytes(req["batch"], True), at(4), at(5),
                                              B.CD_STREAMS_AUTO, at(6))
    else:
        rc = B.lib.codistill_backward(m._h, at(1), at(2), req["batch"], at(3), m.workspace_bytes(req["batch"], True), at(4), at(5), at(6))
    log = [line.split(" ") for line in fake.fake_hip_log().decode().splitlines()]
    json.dump(dict(rc=rc, error=B.lib.codistill_last_error().decode(), main="%x" % (6 << 32),
                   log=[[what, stream, name, int(code)] for what, stream, name, code in log]), sys.stdout)
