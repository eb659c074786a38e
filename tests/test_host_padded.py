"""Host code of networks that are filled up to the fused scorer's widths, on a runtime without a GPU
(hip_stub.c): without memory for that second form of the weights the model is accepted and scored all the same."""
import ctypes as C
import os
import subprocess
import sys

import numpy as np
import pytest

from test_host_paths import ROOT, context, make_library, stub_path  # noqa: F401


def scored(stub, vf, failing, dims=(256, 256, 128, 1)):
    """The kernels that a call on 1000 vectors launches; allocations of `failing` bytes fail meanwhile."""
    from paper_2011_14486_amd import inputs as I
    dims = list(dims)
    if failing:
        stub.stub_fail(failing, failing)
    ctx = context(vf, np.stack([I.resnet18_shaped()]), I.resnet18_space(256), I.model_record(I.MLP, dims, I.BF16), I.mlp_weights(dims))
    stub.stub_fail(1, 0)
    stub.stub_clear()
    out = np.zeros(1000, np.float32)  # (addresses are written down, not used)
    p, n = C.c_void_p(out.ctypes.data), C.c_int64(1000)
    assert vf.vf_score(ctx, p, 0, n, n, C.c_int32(0), p, p, p) == 0
    log = stub.stub_log().decode()
    vf.vf_destroy(ctx)
    return log


# 8 waves of (16 + 16 + 8) k-steps of one row tile, 1 KB each; two hidden layers' biases, the output's, its weights
@pytest.mark.parametrize("failing", [8 * 40 * 1024, (256 + 256 + 4 + 256) * 4])
def test_padded_weights_without_memory(stub_path, failing):  # noqa: F811
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stub_path, str(failing)], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


def test_which_networks(stub_path):  # noqa: F811
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stub_path, "widths"], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


def widths(stub, vf):
    """Networks just inside the line and just outside of it, both sides of which were measured."""
    inside = [[256, 544, 128, 1], [64, 288, 288, 1], [256, 768, 32, 1], [128, 544, 544, 1], [64, 640, 640, 1], [64, 32, 256, 1],
              [64, 160, 64, 64, 64, 1], [512, 160, 1], [1024, 608, 1], [64, 448, 448, 448, 448, 1]]
    outside = [[64, 288, 256, 128, 64, 1], [64, 288, 160, 96, 1], [256, 640, 320, 160, 1], [64, 544, 288, 1], [192, 544, 128, 1],
               [512, 544, 288, 96, 1], [64, 288, 128, 1], [64, 160, 32, 32, 1]]
    for dims in inside + outside:
        log = scored(stub, vf, 0, dims)
        assert ("k_mlp_fast" in log) == (dims in inside) and ("k_mlp_bf16" in log) == (dims in outside), (dims, log)


if __name__ == "__main__":
    sys.path.insert(0, ROOT)
    args = make_library(sys.argv[1])
    if sys.argv[2] == "widths":
        widths(*args)
        sys.exit()
    assert "k_mlp_fast" in scored(*args, 0)
    log = scored(*args, int(sys.argv[2]))
    assert "k_mlp_bf16" in log and "k_mlp_fast" not in log, log
