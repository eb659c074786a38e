"""GPU: decisions on lists of valid candidates (many tiles) against the scorers on id ranges (few
tiles) and, for the beam's selection, against the checker."""
import numpy as np
import pytest

from paper_2011_14486_amd import inputs as I
from tests.test_gpu_greedy import greedy_with_launches

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vf():
    import paper_2011_14486_amd as pkg
    return pkg.load()


def context(vf, pipes, sp, model, w):
    ctx = vf.vf_create(0)
    vf.vf_set_space(ctx, sp); vf.vf_set_pipeline(ctx, pipes); vf.vf_set_model(ctx, model, w)
    return ctx


# (widths, problems, ids per decision): more tiles than compute units on one side, one problem with
# one round of tiles on the other; ragged lists, one to three hidden layers, both tile shapes
@pytest.mark.parametrize("dims", [[256, 512, 512, 1], [256, 512, 1], [256, 512, 512, 512, 1], [256, 1024, 1024, 1],
                                  [64, 512, 512, 1]])
def test_batch_on_lists_equals_single_problems(vf, dims):
    """The same arithmetic candidate by candidate: ids and values of every layer are bit-identical,
    with noise, and with problems whose schedules end early (stage 1 has no valid candidate)."""
    B, sp = 45, I.make_space([1, 2, 4], [1, 2, 4, 8], [1, 8, 16], I.XC_INNER_PERMS, 2, 2, [I.ROOT, I.L1, I.L2, I.INLINE], 2,
                             dims[0])
    pipes = np.stack([I.random_pipeline(6, 70 + b) for b in range(B)])
    w, model = I.mlp_weights(dims, 4, bias_std=0.1), I.model_record(I.MLP, dims, I.BF16)
    many = context(vf, pipes, sp, model, w)
    vf.vf_set_noise(many, 0.2, 9, 0)
    vf.vf_profile_enable(many, True); vf.vf_profile_counts(many)
    whole = [t.cpu().numpy() for t in vf.vf_greedy_schedule(many)]
    scored, valid = vf.vf_profile_counts(many)
    assert scored == valid > 0                     # only listed candidates were scored
    vf.vf_profile_enable(many, False)
    vf.vf_reset_state(many)
    for i in range(6):
        vf.vf_argmin_step(many, i, True)
    steps = [t.cpu().numpy() for t in vf.vf_greedy_schedule(many, first=6)]
    for a, b in zip(whole, steps):
        assert np.array_equal(a, b)
    for b in range(0, B, 4):
        one = context(vf, pipes[b], sp, model, w)
        vf.vf_set_noise(one, 0.2, 9, b)
        st, cids, vals = (t.cpu().numpy()[0] for t in vf.vf_greedy_schedule(one))
        assert np.array_equal(cids, whole[1][b]) and np.array_equal(st, whole[0][b]) and np.array_equal(vals, whole[2][b])
        vf.vf_destroy(one)
    vf.vf_destroy(many)


# lists as long as a workgroup has threads, just shorter and just longer (all ids are valid): written by teams, by a
# workgroup per problem, by several workgroups per problem or between two launches
@pytest.mark.parametrize("n", [504, 512, 525, 1050])
@pytest.mark.parametrize("B", [24, 33, 170])
@pytest.mark.parametrize("dims", [[256, 512, 512, 1], [64, 1024, 1]])
def test_lists_around_the_workgroup_size(vf, n, B, dims):
    """Ids and values of every layer bit-identical to those of one problem alone, step by step."""
    f = lambda k: list(range(1, k + 1))
    nx, ny, nc, nperm, nvec = {504: (7, 8, 3, 3, 1), 512: (8, 8, 8, 1, 1), 525: (7, 5, 5, 3, 1), 1050: (7, 5, 5, 3, 2)}[n]
    sp = I.make_space(f(nx), f(ny), f(nc), I.ALL_PERMS[:nperm], nvec, 1, [I.ROOT], 1, dims[0])
    assert I.space_dense_count(sp) == n
    pipes = I.resnet18_batch(B, seed=3)[:, :4].copy()
    pipes[:, :, 1:4] = np.maximum(pipes[:, :, 1:4], 8)
    w, model = I.mlp_weights(dims, 4, bias_std=0.1), I.model_record(I.MLP, dims, I.BF16)
    many = context(vf, pipes, sp, model, w)
    whole = [t.cpu().numpy() for t in vf.vf_greedy_schedule(many)]
    vf.vf_sync_status(many)
    vf.vf_reset_state(many)
    assert vf.vf_enumerate(many, 0)[2].tolist() == [n] * B
    for i in range(4):
        vf.vf_argmin_step(many, i, True)
    for a, b in zip(whole, vf.vf_greedy_schedule(many, first=4)):
        assert np.array_equal(a, b.cpu().numpy())
    vf.vf_destroy(many)
    for b in range(0, B, 11):
        one = context(vf, pipes[b], sp, model, w)
        for i in range(4):
            best, value = (t.cpu().numpy() for t in vf.vf_argmin_step(one, i, True))
            assert best[0] == whole[1][b, i] and value[0] == whole[2][b, i]
        vf.vf_destroy(one)


@pytest.mark.parametrize("B", [385, 512])
def test_second_round_of_long_decisions_in_one_launch(vf, B):
    """16384 ids, more problems than compute units: whole schedules in one launch (from three quarters
    of the second round on) decide what the steps on lists decide, bit for bit."""
    dims, sp = [256, 512, 512, 1], I.mobilenetv2_space()
    pipes = np.stack([I.random_pipeline(3, 40 + b % 7) for b in range(B)])
    ctx = context(vf, pipes, sp, I.model_record(I.MLP, dims, I.BF16), I.mlp_weights(dims, 4, bias_std=0.1))
    vf.vf_set_noise(ctx, 0.2, 9, 0)
    whole, launches = greedy_with_launches(vf, ctx)
    assert launches == 1
    vf.vf_reset_state(ctx)
    for i in range(3):
        vf.vf_argmin_step(ctx, i, True)
    for a, b in zip(whole, vf.vf_greedy_schedule(ctx, first=3)):
        assert np.array_equal(a, b.cpu().numpy())
    vf.vf_destroy(ctx)


@pytest.mark.parametrize("H", [32, 96, 256])
def test_recurrent_batch_equals_single_problems(vf, H):
    """Many candidates run in the forms for throughput, few in those for latency, with the same arithmetic per
    candidate: ids and values of every layer are bit-identical (ragged tiles; noise)."""
    sp, B = I.resnet18_space(256), 14                # 14 * 64 tiles of 64 ids: more than 3 * 256
    pipes = np.stack([I.random_pipeline(5, 90 + b) for b in range(B)])
    w, model = I.lstm_weights(64, H, seed=6, bias_std=0.2), I.model_record(I.LSTM, [64, H, 1], I.BF16)
    many = context(vf, pipes, sp, model, w)
    vf.vf_set_noise(many, 0.1, 3, 0)
    st, cids, vals = (t.cpu().numpy() for t in vf.vf_greedy_schedule(many))
    vf.vf_destroy(many)
    for b in range(B):
        one = context(vf, pipes[b], sp, model, w)
        vf.vf_set_noise(one, 0.1, 3, b)
        s1, c1, v1 = (t.cpu().numpy()[0] for t in vf.vf_greedy_schedule(one))
        assert np.array_equal(c1, cids[b]) and np.array_equal(s1, st[b]) and np.array_equal(v1, vals[b])
        vf.vf_destroy(one)


# the factors make the number of ids of a decision: the search works on lists from 64 tiles of 128 on
@pytest.mark.parametrize("K,fac,const", [(2, [1, 2, 4, 8], True), (33, [1, 2, 4], True), (33, [1, 2, 4], False),
                                         (300, [1, 4], False), (1024, [1, 4], True)])
def test_beam_selection_on_lists(vf, ovf, K, fac, const):
    """The survivors of the layers against the checker.  const: a network whose value is the same
    for every state, so that all scores tie and the survivors are the first (slot, id) pairs."""
    dims = [64, 512, 512, 1]
    pipe = I.random_pipeline(3, 21)
    sp = I.make_space(fac, fac, fac, I.ALL_PERMS[:2 if K > 100 else 6], 2, 2, [I.ROOT, I.L1, I.L2, I.INLINE][:1 if K > 400 else 4],
                      2 if K < 100 else 1, 64)
    assert (I.space_dense_count(sp) + 127) // 128 * K > 64
    w = I.mlp_weights(dims, 5, bias_std=0.1)
    if const:
        w = np.zeros_like(w)
        w[-1] = 0.75
    model = I.model_record(I.MLP, dims, I.BF16)
    ctx = context(vf, np.stack([pipe] * K), sp, model, w)
    st, cids, vals, nb = (t.cpu().numpy() for t in vf.vf_beam_search(ctx))
    vf.vf_destroy(ctx)
    if const:
        ref = ovf.beam(pipe, sp, K, model, w)
        assert nb[0] == ref["n_beams"] > 0
        assert np.array_equal(cids, ref["cids"]) and np.array_equal(vals, ref["values"])
        return
    assert nb[0] == K and len(set(map(tuple, cids))) == K and np.all(np.diff(vals[:, -1]) >= 0)
    # V of every extension of the survivors' prefixes: the values agree and nothing that is clearly
    # better than the last survivor was left out
    kept, worst, tol = set(map(tuple, cids)), vals[:, -1].max(), 2e-2
    scale = np.sqrt(np.mean(vals[:, -1] ** 2))
    for pre in sorted({tuple(r[:2]) for r in cids}):
        s, ok = ovf.decision_scores(pipe, sp, model, w, list(pre) + [0], 2)
        for j in np.flatnonzero((cids[:, :2] == pre).all(axis=1)):
            assert ok[cids[j, 2]] and abs(s[cids[j, 2]] - vals[j, 2]) <= tol * max(abs(s[cids[j, 2]]), scale)
        for c in np.flatnonzero(ok & (s < worst - 2 * tol * max(abs(worst), scale))):
            assert pre + (c,) in kept
