"""GPU parity of the recurrent search without memory for the candidates' feature rows, or for the second
form of the weights: the scorer that evaluates the candidates itself and streams the weights.  In a
process of its own, in which hip_limit.c refuses that one allocation."""
import ctypes as C
import os
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

pytestmark = pytest.mark.gpu


def without(shim):
    import torch  # noqa: F401  (its runtime first)
    limit = C.CDLL(shim, mode=C.RTLD_GLOBAL)
    limit.limit.argtypes = [C.c_size_t]
    import paper_2011_14486_amd as pkg
    from oracle import ovf
    from paper_2011_14486_amd import inputs as I
    from tests.test_gpu_beam import check_beam
    from tests.test_gpu_lstm_search import compare_schedule, setup
    from tests.util import TOL
    vf = pkg.load()
    sp = I.make_space([1, 2, 4], [1, 3, 4], [1, 2, 8], I.ALL_PERMS[:2], 2, 2, [I.ROOT, I.L1, I.L2, I.INLINE], 2, 64)
    hits = 0
    for H in (32, 128, 256):
        for B, what in ((1, "rows"), (9, "rows"), (70, "rows"), (9, "weights")):
            print("H", H, "problems", B, "without", what, flush=True)
            pipes = np.stack([I.random_pipeline(4, 60 + b % 9) for b in range(B)])
            ctx, model, w = setup(vf, pipes, sp, H)
            limit.limit(B * vf.vf_padded_count(ctx) * 128 if what == "rows" else H // 32 * (2 * (H // 16) + 8) * 2048)
            st, cids, vals = [t.cpu().numpy() for t in vf.vf_greedy_schedule(ctx)]
            vf.vf_reset_state(ctx)
            for i in range(4):                                  # and driven layer by layer
                vf.vf_argmin_step(ctx, i, True)
            again = [t.cpu().numpy() for t in vf.vf_greedy_schedule(ctx, 4, 3)]
            hits += 1
            assert limit.limit(0) == hits
            vf.vf_destroy(ctx)
            for b in range(min(B, 9)):
                compare_schedule(ovf, pipes[b], sp, model, w, cids[b], vals[b], st[b], TOL[1])
            for b in range(9, B):
                assert np.array_equal(cids[b], cids[b % 9]) and np.array_equal(vals[b], vals[b % 9])
            assert all(np.array_equal(x, y) for x, y in zip(again, (st, cids, vals)))
    K, pipe = 6, I.random_pipeline(4, 31)
    ctx, model, w = setup(vf, np.repeat(pipe[None], K, axis=0), sp, 64)
    limit.limit(K * vf.vf_padded_count(ctx) * 128)

    def run(last):
        vf.vf_reset_state(ctx)
        st, cids, vals, nb = vf.vf_beam_search(ctx, 0, last)
        return cids.cpu().numpy(), vals.cpu().numpy(), st.cpu().numpy(), int(nb.cpu()[0])
    print("beam", flush=True)
    check_beam(ovf, pipe, sp, model, w, run, K, TOL[1])
    assert limit.limit(0) == hits + 1
    vf.vf_destroy(ctx)


def test_without_rows_or_weights(tmp_path):
    shim = str(tmp_path / "hip_limit.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-Wall", "-o", shim, os.path.join(HERE, "hip_limit.c"), "-ldl"], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), shim], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    without(sys.argv[1])
