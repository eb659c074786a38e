"""Host code of networks that are filled up to the fused scorer's widths, on a runtime without a GPU
(hip_stub.c): without memory for that second form of the weights the model is accepted and scored all the same."""
import ctypes as C
import os
import subprocess
import sys

import numpy as np
import pytest

from test_host_paths import ROOT, context, make_library, stub_path  # noqa: F401


def scored(stub, vf, failing):
    """The kernels that a call on 1000 vectors launches; allocations of `failing` bytes fail meanwhile."""
    from paper_2011_14486_amd import inputs as I
    dims = [256, 256, 128, 1]
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


if __name__ == "__main__":
    sys.path.insert(0, ROOT)
    args = make_library(sys.argv[1])
    assert "k_mlp_fast" in scored(*args, 0)
    log = scored(*args, int(sys.argv[2]))
    assert "k_mlp_bf16" in log and "k_mlp_fast" not in log, log
