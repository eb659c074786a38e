"""The library's host code on a runtime without a GPU (hip_stub.c: launches are written down, not run):
allocation failures, launch limits, arguments of launches."""
import ctypes as C
import os
import re
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def make_library(stub_path):
    """libvf.so bound to the stub (which has to be in the process first)."""
    from paper_2011_14486_amd import binding
    stub = C.CDLL(stub_path, mode=C.RTLD_GLOBAL)
    stub.stub_fail.argtypes = [C.c_size_t, C.c_size_t]
    stub.stub_log.restype = C.c_char_p
    stub.stub_fail_launch.argtypes = [C.c_char_p, C.c_int]
    vf = C.CDLL(binding.LIB_PATH)
    vf.vf_create.argtypes = [C.POINTER(C.c_void_p), C.c_int, C.c_void_p]
    vf.vf_padded_count.restype = C.c_int64
    vf.vf_set_model.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_size_t]
    return stub, vf


def context(vf, pipes, space, model, w):
    ctx = C.c_void_p()
    keep = [np.ascontiguousarray(a) for a in (pipes, space, model, w)]
    p = [C.c_void_p(a.ctypes.data) for a in keep]
    assert vf.vf_create(C.byref(ctx), 0, None) == 0
    assert vf.vf_set_space(ctx, p[1]) == 0
    assert vf.vf_set_pipeline(ctx, p[0], pipes.shape[1], pipes.shape[0]) == 0
    assert vf.vf_set_model(ctx, p[2], p[3], w.size) == 0
    return ctx


def recurrent_weights(stub, vf):
    """The second form of the recurrent weights, or the rows of the candidates, cannot be had: the search goes on
    with the scorer that needs neither, now and when memory is back; the others never run without their weights."""
    from paper_2011_14486_amd import inputs as I
    B = 32
    for H, kernel in ((64, "k_seq_step_held"), (256, "k_seq_step_wide")):
        args = (np.stack([I.resnet18_shaped()] * B), I.resnet18_space(256), I.model_record(I.LSTM, [64, H, 1], I.BF16),
                I.lstm_weights(64, H))
        for size in (H // 32 * (2 * (H // 16) + 8) * 1024 * 2, B * 4096 * 128):
            ctx = context(vf, *args)
            assert vf.vf_padded_count(ctx) == 4096
            stub.stub_clear()
            stub.stub_fail(size, size)
            rc = vf.vf_argmin_step(ctx, 0, 1, None, None)
            stub.stub_fail(1, 0)
            assert rc == 0, rc
            assert vf.vf_argmin_step(ctx, 1, 1, None, None) == 0
            log = stub.stub_log().decode()
            steps = [l.split() for l in log.splitlines() if "k_seq_step" in l]
            assert len(steps) == 2 and all(s[2] == "1" for s in steps), steps
            assert "k_seq_step_" not in log and log.count("k_seq_compact") == 2 and "k_seq_open" not in log, log
            vf.vf_destroy(ctx)
        # with memory
        stub.stub_clear()
        ctx = context(vf, *args)
        assert vf.vf_argmin_step(ctx, 0, 1, None, None) == 0
        log = stub.stub_log().decode()
        assert kernel in log and "k_seq_open" in log and "k_seq_compact" not in log
        assert all(l.split()[2] == "1" for l in log.splitlines())
        vf.vf_destroy(ctx)


def recurrent_spaces(stub, vf):
    """A larger space behind a recurrent search: lists and rows of its size, not of the old one's."""
    from paper_2011_14486_amd import inputs as I
    H, B = 64, 4
    small = I.make_space([1, 2], [1, 2], [1, 2], I.ALL_PERMS[:1], 1, 1, [I.ROOT], 1, 64)
    large = I.make_space([1, 2, 4], [1, 2, 4], [1, 2, 4], I.ALL_PERMS, 2, 2, [I.ROOT, I.L1], 1, 64)
    ctx = context(vf, np.stack([I.random_pipeline(3, 5)] * B), small, I.model_record(I.LSTM, [64, H, 1], I.BF16),
                  I.lstm_weights(64, H))
    assert vf.vf_argmin_step(ctx, 0, 1, None, None) == 0
    assert vf.vf_set_space(ctx, C.c_void_p(large.ctypes.data)) == 0
    Mpad = vf.vf_padded_count(ctx)
    assert Mpad == 1536
    for each, rc, kernel in ((4, -3, None), (128, 0, "k_seq_compact")):  # lists; rows, without which the other scorer runs
        assert vf.vf_reset_state(ctx) == 0
        stub.stub_clear()
        stub.stub_fail(B * Mpad * each, B * Mpad * each)
        assert vf.vf_argmin_step(ctx, 0, 1, None, None) == rc
        stub.stub_fail(1, 0)
        log = stub.stub_log().decode()
        assert "k_seq_open" not in log and (rc != 0 or kernel in log), log
    vf.vf_destroy(ctx)


def refused_opening(stub, vf):
    """The launch that opens a decision and does the prefix's step is refused: the context does not take the
    step for done, the schedule goes on with it."""
    from paper_2011_14486_amd import inputs as I
    B = 4
    ctx = context(vf, np.stack([I.random_pipeline(4, 5)] * B), I.tiny_space(64), I.model_record(I.LSTM, [64, 64, 1], I.BF16),
                  I.lstm_weights(64, 64))
    stub.stub_fail_launch(b"k_seq_open", 1)
    assert vf.vf_greedy_schedule(ctx, 0, 3, None, None, None) == -4
    assert vf.vf_n_scheduled(ctx) == 1
    assert vf.vf_greedy_schedule(ctx, 1, 3, None, None, None) == 0
    grids = [int(l.split()[1]) for l in stub.stub_log().decode().splitlines() if "k_seq_open" in l]
    plain = B * vf.vf_padded_count(ctx) // 256
    assert grids == [plain] + [plain + 1] * 3, grids  # (four problems to a workgroup of the step)
    # a beam: the step goes from one set of states to the other
    assert vf.vf_reset_state(ctx) == 0
    stub.stub_clear()
    stub.stub_fail_launch(b"k_seq_open", 1)
    assert vf.vf_beam_search(ctx, 0, 3, None, None, None, None) == -4
    assert vf.vf_n_scheduled(ctx) == 1 and vf.vf_argmin_step(ctx, 1, 0, None, None) == 0
    grids = [int(l.split()[1]) for l in stub.stub_log().decode().splitlines() if "k_seq_open" in l]
    assert grids == [plain, plain + 1], grids
    vf.vf_destroy(ctx)


def prefix_step_in_call(stub, vf):
    """The prefix's step behind a call's last commit is launched by that call, whatever decided it; behind the last
    stage there is none."""
    from paper_2011_14486_amd import inputs as I
    B, S = 4, 5
    ctx = context(vf, np.stack([I.random_pipeline(S, 5)] * B), I.tiny_space(64), I.model_record(I.LSTM, [64, 64, 1], I.BF16),
                  I.lstm_weights(64, 64))
    plain = B * vf.vf_padded_count(ctx) // 256

    def steps(call, *args):
        """Prefix steps of a call: launches of their own, and workgroups next to an opening."""
        stub.stub_clear()
        assert call(ctx, *args) == 0
        lines = [l.split() for l in stub.stub_log().decode().splitlines()]
        return (sum("k_seq_advance" in l[0] for l in lines), sum(int(l[1]) - plain for l in lines if "k_seq_open" in l[0]))

    assert steps(vf.vf_argmin_step, 0, 0, None, None) == (0, 0)
    assert steps(vf.vf_argmin_step, 0, 1, None, None) == (1, 0)
    assert steps(vf.vf_greedy_schedule, 1, 2, None, None, None) == (1, 1)
    assert steps(vf.vf_beam_search, 3, 3, None, None, None, None) == (1, 0)
    assert steps(vf.vf_argmin_step, 4, 1, None, None) == (0, 0)
    assert vf.vf_reset_state(ctx) == 0
    assert steps(vf.vf_greedy_schedule, 0, S - 1, None, None, None) == (0, S - 1)
    vf.vf_destroy(ctx)


def small_networks(stub, vf):
    """Which ids the small networks' kernels take: as they come where a wave has one sub-tile of them or nearly all
    are valid (then with the columns per lane for as many), else the valid ones."""
    from paper_2011_14486_amd import inputs as I

    def kernel(B, space, dtype):
        dims = [64, 128, 128, 1]
        ctx = context(vf, np.stack([I.tiny_conv_relu()] * B), space, I.model_record(I.MLP, dims, dtype), I.mlp_weights(dims))
        stub.stub_clear()
        assert vf.vf_argmin_step(ctx, 0, 0, None, None) == 0
        vf.vf_destroy(ctx)
        name, = [l for l in stub.stub_log().decode().splitlines() if "k_small" in l]
        return [int(n) for n in re.findall(r"ILi(\d+)ELi(\d+)ELi(\d+)E", name)[0]]  # columns per lane, row tiles, which ids

    for dtype, rows in ((I.FP32, 8), (I.BF16, 4)):
        assert kernel(1, I.tiny_space(64), dtype) == [1, rows, 2]
        assert kernel(64, I.tiny_space(64), dtype) == [2, rows, 1]
        for last, ids in ((8, 2), (99, 2), (None, 1)):  # all valid, seven in eight, three in four
            fc = [1, 2, 4, 5, 6, 7, 8, 8][:7] + [last] if last else [1, 2, 4, 5, 6, 8, 99, 99]
            root = I.make_space([1, 2, 4, 8], [1, 2, 4, 8], fc, I.ALL_PERMS[:4], 2, 2, [I.ROOT], 1, 64)
            assert kernel(200, root, dtype) == [2, rows, ids], last


def sequence_widths(stub, vf):
    """Sequences: a network whose weights fit a compute unit is held there, whatever its widths."""
    from paper_2011_14486_amd import inputs as I
    widest = {32: 192, 64: 160, 96: 128, 128: 128, 160: 128, 192: 128, 224: 96, 256: 96}
    ctx = context(vf, np.stack([I.resnet18_shaped()]), I.resnet18_space(256), I.model_record(I.LSTM, [32, 32, 1], I.BF16),
                  I.lstm_weights(32, 32))
    at, n = C.c_void_p(4096), C.c_int64  # (addresses are written down, not used)
    for F in widest:
        for H in range(32, 257, 32):
            m, w = I.model_record(I.LSTM, [F, H, 1], I.BF16), I.lstm_weights(F, H)
            assert vf.vf_set_model(ctx, C.c_void_p(m.ctypes.data), C.c_void_p(w.ctypes.data), w.size) == 0
            stub.stub_clear()
            assert vf.vf_score(ctx, at, 1, n(1000), n(7), C.c_int32(0), at, at, at) == 0
            log = stub.stub_log().decode()
            assert ("k_lstm_held" in log) == (H <= widest[F]) and ("k_lstm_bf16" in log) == (H > widest[F]), (F, H, log)
    vf.vf_destroy(ctx)


def profiled_launches(stub, vf):
    """The recurrent search's launches that the per-kernel timing brackets, per decision: the one that makes the
    features, the scorer, the commit."""
    from paper_2011_14486_amd import inputs as I
    ctx = context(vf, np.stack([I.random_pipeline(4, 5)] * 2), I.tiny_space(64), I.model_record(I.LSTM, [64, 64, 1], I.BF16),
                  I.lstm_weights(64, 64))
    assert vf.vf_profile_enable(ctx, 1) == 0 and vf.vf_greedy_schedule(ctx, 0, 3, None, None, None) == 0
    for which in range(3):
        n = C.c_int64()
        assert vf.vf_profile_read(ctx, which, None, C.byref(n)) == 0 and n.value == 4, (which, n.value)
    vf.vf_destroy(ctx)


def candidate_lists(stub, vf):
    """No memory for the candidate lists: a greedy schedule is decided on id ranges, whether it would
    have run layer by layer (64 problems) or in one launch (200)."""
    from paper_2011_14486_amd import inputs as I
    dims = [256, 512, 512, 1]
    for B, kernel in ((64, "k_open_layer"), (200, "k_whole")):
        ctx = context(vf, np.stack([I.resnet18_shaped()] * B), I.resnet18_space(256), I.model_record(I.MLP, dims, I.BF16),
                      I.mlp_weights(dims))
        size = B * vf.vf_padded_count(ctx) * 4
        stub.stub_clear()
        stub.stub_fail(size, size)
        rc = vf.vf_greedy_schedule(ctx, 0, 19, None, None, None)
        stub.stub_fail(1, 0)
        log = stub.stub_log().decode()
        assert rc == 0 and vf.vf_n_scheduled(ctx) == 20, rc
        assert kernel not in log and log.count("k_mlp_fast") == 20, log
        # with memory
        assert vf.vf_reset_state(ctx) == 0
        stub.stub_clear()
        assert vf.vf_greedy_schedule(ctx, 0, 19, None, None, None) == 0
        assert kernel in stub.stub_log().decode()
        vf.vf_destroy(ctx)


def many_problems(stub, vf):
    """Features of 90,000 problems of a small space: 193 workgroups of 256 each would be more work-items
    than a launch takes."""
    from paper_2011_14486_amd import inputs as I
    B, sp = 90000, I.make_space([1, 2], [1, 2], [1, 2], [(0, 1, 2)], 1, 1, [I.ROOT], 1, 256)
    pipe = I.random_pipeline(1, 3)
    dims = [256, 512, 512, 1]
    ctx = context(vf, np.stack([pipe] * B), sp, I.model_record(I.MLP, dims, I.BF16), I.mlp_weights(dims))
    stub.stub_clear()
    rc = vf.vf_featurize(ctx, 0, C.c_void_p(4096))  # (written down, not run)
    assert rc == 0, rc
    grids = [int(l.split()[1]) for l in stub.stub_log().decode().splitlines() if "k_featurize" in l]
    assert len(grids) == 2 and B * 193 <= sum(grids) < (B + 8) * 193, grids
    vf.vf_destroy(ctx)


@pytest.fixture(scope="module")
def stub_path(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-o", out,
                    os.path.join(HERE, "hip_stub.c")], check=True)
    from paper_2011_14486_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2011_14486_amd.build import build_lib
        build_lib()
    return out


@pytest.mark.parametrize("case", ["recurrent_weights", "recurrent_spaces", "refused_opening", "prefix_step_in_call", "small_networks", "sequence_widths", "profiled_launches", "candidate_lists", "many_problems"])
def test_host_path(stub_path, case):
    # (a process of its own: the stub takes the place of the whole runtime)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stub_path, case], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    sys.path.insert(0, ROOT)
    globals()[sys.argv[2]](*make_library(sys.argv[1]))
