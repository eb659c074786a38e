"""GPU parity of the search with small networks: a wave collects the valid ids of its share of a decision
until a sub-tile is full.  Shares of one block and of many, blocks of 16, 32 and 64 ids, one and two
columns per lane, several problems per wave."""
import numpy as np
import pytest

from paper_2011_14486_amd import inputs as I
from tests.test_gpu_lstm_search import compare_schedule
from tests.util import TOL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vf():
    import paper_2011_14486_amd as pkg
    return pkg.load()


@pytest.mark.parametrize("dtype", [I.FP32, I.BF16])
@pytest.mark.parametrize("B,facs", [(1, 4), (5, 4), (9, 5), (40, 7), (70, 4), (300, 3), (1100, 2)])
def test_shares(vf, ovf, B, facs, dtype):
    """Ids, values and states of a batch are those of single problems, bit for bit, and the checker's; a beam's
    masked scores are +inf where an id is not valid (every survivor is a candidate of its parent)."""
    fac = [1, 2, 3, 4, 5, 6, 8][:facs]
    sp = I.make_space(fac, fac, fac, I.ALL_PERMS[:2], 2, 2, [I.ROOT, I.L1, I.L2, I.INLINE], 2, 64)
    dims = [64, 96, 32, 1]
    w, model = I.mlp_weights(dims, 5, bias_std=0.1), I.model_record(I.MLP, dims, dtype)
    pipes = np.stack([I.random_pipeline(3, 200 + b % 6) for b in range(B)])

    def run(p, beam=False):
        ctx = vf.vf_create(0)
        vf.vf_set_space(ctx, sp); vf.vf_set_pipeline(ctx, p); vf.vf_set_model(ctx, model, w)
        out = [t.cpu().numpy() for t in (vf.vf_beam_search(ctx)[:3] if beam else vf.vf_greedy_schedule(ctx))]
        vf.vf_destroy(ctx)
        return out
    st, cids, vals = run(pipes)
    for b in range(min(B, 6)):
        s1, c1, v1 = (a[0] for a in run(pipes[b]))
        if b < 3:
            compare_schedule(ovf, pipes[b], sp, model, w, c1, v1, s1, TOL[0 if dtype == I.FP32 else 1])
        for k in range(b, B, 6):
            assert np.array_equal(c1, cids[k]) and np.array_equal(v1, vals[k]) and np.array_equal(s1, st[k])
    if B <= 70:
        st, cids, vals = run(np.stack([pipes[0]] * B), beam=True)
        assert len(set(map(tuple, cids))) == B
        for j in range(0, B, 7):
            sc, ok = ovf.decision_scores(pipes[0], sp, model, w, cids[j, :2], 2)
            c = cids[j, 2]
            assert ok[c] and abs(sc[c] - vals[j, 2]) <= TOL[0 if dtype == I.FP32 else 1] * max(abs(sc[c]), np.sqrt(np.mean(sc[ok] ** 2)))


@pytest.mark.parametrize("dtype", [I.FP32, I.BF16])
@pytest.mark.parametrize("B,last", [(5, 8), (70, 8), (70, 99), (500, 99)])
def test_mostly_valid(vf, ovf, B, last, dtype):
    """Spaces of root-level candidates of which all or seven in eight are valid: a wave takes its ids as they
    come.  A batch as single problems, single problems as the oracle, a beam's survivors valid."""
    sp = I.make_space([1, 2, 4], [1, 2, 4], [1, 2, 4, 5, 6, 7, 8, last], I.ALL_PERMS[:5], 2, 1, [I.ROOT], 1, 64)
    pipe = I.tiny_conv_relu()
    pipes = np.stack([pipe] * B)
    assert (pipe[:, 1:4] >= [4, 4, 8]).all() and I.space_dense_count(sp) % 32 == 16
    dims = [64, 96, 32, 1]
    w, model = I.mlp_weights(dims, 5, bias_std=0.1), I.model_record(I.MLP, dims, dtype)
    tol = TOL[0 if dtype == I.FP32 else 1]

    def run(p, beam=False):
        ctx = vf.vf_create(0)
        vf.vf_set_space(ctx, sp); vf.vf_set_pipeline(ctx, p); vf.vf_set_model(ctx, model, w)
        out = [t.cpu().numpy() for t in (vf.vf_beam_search(ctx)[:3] if beam else vf.vf_greedy_schedule(ctx))]
        vf.vf_destroy(ctx)
        return out
    st, cids, vals = run(pipes)
    s1, c1, v1 = (a[0] for a in run(pipe))
    compare_schedule(ovf, pipe, sp, model, w, c1, v1, s1, tol)
    assert (cids == c1).all() and (vals == v1).all() and (st == s1).all()
    if B <= 70:
        _, cids, vals = run(pipes, beam=True)
        assert len(set(map(tuple, cids))) == B
        for j in range(0, B, 7):
            sc, ok = ovf.decision_scores(pipe, sp, model, w, cids[j, :1], 1)
            c = cids[j, 1]
            assert ok[c] and abs(sc[c] - vals[j, 1]) <= tol * max(abs(sc[c]), np.sqrt(np.mean(sc[ok] ** 2)))


@pytest.mark.parametrize("const", [True, False])
@pytest.mark.parametrize("K,fac", [(4, [1, 2, 4]), (5, [1, 2, 4]), (17, [1, 2, 4, 8]), (300, [1, 2, 4]), (1024, [1, 2])])
def test_selection_from_masked_scores(vf, ovf, K, fac, const):
    """One and several passes, up to four survivors and many; const: every state has the same value, so that all
    scores tie and the survivors are the first (slot, id) pairs."""
    sp = I.make_space(fac, fac, fac, I.ALL_PERMS[:2], 2, 2, [I.ROOT, I.L1, I.L2, I.INLINE], 2, 64)
    dims, pipe = [64, 32, 1], I.random_pipeline(3, 21)
    w = I.mlp_weights(dims, 5, bias_std=0.1)
    if const:
        w = np.zeros_like(w)
        w[-1] = 0.75
    model = I.model_record(I.MLP, dims, I.FP32)
    ctx = vf.vf_create(0)
    vf.vf_set_space(ctx, sp); vf.vf_set_pipeline(ctx, np.stack([pipe] * K)); vf.vf_set_model(ctx, model, w)
    st, cids, vals, nb = (t.cpu().numpy() for t in vf.vf_beam_search(ctx))
    vf.vf_destroy(ctx)
    ref = ovf.beam(pipe, sp, K, model, w)
    assert nb[0] == ref["n_beams"] > 0
    if const:
        assert np.array_equal(cids, ref["cids"]) and np.array_equal(vals, ref["values"])
    else:  # (fp32: the same survivors' values up to the tolerance, in order)
        n = int(nb[0])
        scale = np.maximum(np.abs(ref["values"][:n, -1]), np.sqrt(np.mean(ref["values"][:n, -1] ** 2)))
        assert np.all(np.diff(vals[:n, -1]) >= 0) and np.all(np.abs(vals[:n, -1] - ref["values"][:n, -1]) <= TOL[0] * scale)
