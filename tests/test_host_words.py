"""Host code around the words that workgroups exchange, on a runtime without a GPU (hip_stub.c)."""
import ctypes as C
import os
import subprocess
import sys

import numpy as np
import pytest

from test_host_paths import ROOT, context, make_library, stub_path  # noqa: F401


def small(vf):
    from paper_2011_14486_amd import inputs as I
    dims = [64, 128, 128, 1]
    return context(vf, I.random_pipeline(20, 5)[None], I.tiny_space(64), I.model_record(I.MLP, dims, I.BF16), I.mlp_weights(dims))


def score(vf, ctx):
    out = np.zeros(1000, np.float32)  # (addresses are written down, not used)
    p, n = C.c_void_p(out.ctypes.data), C.c_int64(1000)
    assert vf.vf_score(ctx, p, 0, n, n, C.c_int32(0), p, p, p) == 0


def words_stay(stub, vf):
    """The words of vf_score's one minimum are not given back for a schedule that needs more of them: a graph
    captured from vf_score goes on using them."""
    ctx = small(vf)
    score(vf, ctx)
    assert "Li4EE" in stub.stub_log().decode()  # (the form with one minimum)
    before = stub.stub_frees()
    assert vf.vf_greedy_schedule(ctx, 0, 19, None, None, None) == 0
    assert stub.stub_frees() == before
    vf.vf_destroy(ctx)


def words_under_capture(stub, vf):
    """Words that a schedule has not got yet are not made while the stream is captured (they would be cleared by the
    graph, not by the call): it is decided layer by layer then, in one launch before and after."""
    from paper_2011_14486_amd import inputs as I
    dims = [256, 512, 512, 1]
    large = context(vf, I.resnet18_batch(2), I.resnet18_space(256), I.model_record(I.MLP, dims, I.BF16), I.mlp_weights(dims))
    for ctx, one, each in ((small(vf), "k_small", "k_small"), (large, "k_chain", "k_mlp_fast")):
        for capture, scorer, launches in ((1, each, 20), (0, one, 1), (1, one, 1)):
            assert vf.vf_reset_state(ctx) == 0
            stub.stub_clear()
            stub.stub_capture(capture)
            assert vf.vf_greedy_schedule(ctx, 0, 19, None, None, None) == 0
            stub.stub_capture(0)
            log = [l for l in stub.stub_log().decode().splitlines() if scorer in l and "clear" not in l]
            assert len(log) == launches, (capture, log)
        vf.vf_destroy(ctx)


@pytest.mark.parametrize("case", ["words_stay", "words_under_capture"])
def test_host_words(stub_path, case):  # noqa: F811
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stub_path, case], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    sys.path.insert(0, ROOT)
    globals()[sys.argv[2]](*make_library(sys.argv[1]))
