"""GPU parity: beam search guided by V against the CPU checker."""
import numpy as np
import pytest

from paper_2011_14486_amd import inputs as I
from tests.util import TOL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vf():
    import paper_2011_14486_amd as pkg
    return pkg.load()


def layer_scores(ovf, pipe, sp, model, w, pre, i):
    """The checker's V of every candidate state of decision i after prefix `pre`:
    (scores float64 [M], valid [M]) for either kind of value network."""
    M = ovf.dense_count(sp)
    if model[0] == I.LSTM:
        x, valid = ovf.sequences(pipe, sp, list(pre), i)
        sc = np.full(M, np.inf)
        ids = np.flatnonzero(valid)
        if len(ids):
            sc[ids] = ovf.score_lstm(model, w, x[ids])
        return sc, valid.astype(bool)
    feat = ovf.featurize(pipe, sp, list(pre), i)
    return ovf.score_mlp(model, w, feat, M=M).astype(np.float64), feat[16, :M] != 0


def check_beam(ovf, pipe, sp, model, w, run, K, tol, start=()):
    """Layer by layer (run(last) = the GPU search stopped after layer `last`): the checker
    scores every extension of the GPU's survivors of the layer before; the GPU's survivors
    of this layer must be the smallest ones (up to the score tolerance at the cut), in
    order, with matching values and state records.  start: the committed prefix the search
    starts from (decisions that carry no value)."""
    S, n0 = len(pipe), len(start)
    prev, vals_prev = [tuple(start)], [np.zeros(0, np.float32)]
    for i in range(n0, S):
        cids, vals, states, n_beams = run(i)
        items = []
        for b, pre in enumerate(prev):
            sc, valid = layer_scores(ovf, pipe, sp, model, w, pre, i)
            for c in np.flatnonzero(valid):
                if sc[c] < np.inf:
                    items.append((sc[c], b, int(c)))
        items.sort()
        if not items:
            # dead end: the survivors of the layer before are kept as they were
            assert n_beams == len(prev) or (prev == [tuple(start)] and n_beams == 1)
            for j, pre in enumerate(prev):
                assert tuple(int(t) for t in cids[j, :i]) == pre and (cids[j, i:] == -1).all()
            return
        rows = [j for j in range(K) if cids[j, i] >= 0]
        assert rows == list(range(len(rows))) and len(rows) == min(K, len(items)) == n_beams
        score_of = {(b, c): s for s, b, c in items}
        scale = max(float(np.sqrt(np.mean([s * s for s, _, _ in items]))), 1e-30)
        got = []
        for j in rows:
            pre = tuple(int(t) for t in cids[j, :i])
            assert pre in prev, f"layer {i}: row {j} does not extend a survivor of the layer before"
            key = (prev.index(pre), int(cids[j, i]))
            assert key in score_of, f"layer {i}: row {j} is not a valid candidate"
            got.append((score_of[key], key))
            err = abs(float(vals[j, i]) - score_of[key]) / max(abs(score_of[key]), scale)
            assert err <= tol, (i, j, err)
            assert np.array_equal(vals[j, n0:i], vals_prev[key[0]][n0:i])
            rst, _ = ovf.states(pipe, sp, cids[j, :i + 1])
            assert np.array_equal(states[j, :i + 1], rst) and not states[j, i + 1:].any()
        cut = items[len(rows) - 1][0]
        slack = tol * max(abs(cut), scale)
        assert all(s <= cut + slack for s, _ in got), f"layer {i}: a survivor is not among the best"
        chosen = {k for _, k in got}
        assert len(chosen) == len(got), "a survivor appears twice"
        worst = max(s for s, _ in got)
        for s, b, c in items[:len(rows)]:
            assert (b, c) in chosen or s >= worst - slack, f"layer {i}: a better extension was dropped"
        assert (np.diff(vals[rows, i]) >= 0).all(), "survivors are not ordered by score"
        assert (cids[len(rows):] == -1).all() and np.isinf(vals[len(rows):]).all() and not states[len(rows):].any()
        prev = [tuple(int(t) for t in cids[j, :i + 1]) for j in rows]
        vals_prev = [vals[j].copy() for j in rows]


def make_ctx(vf, pipe, sp, model, w, K):
    ctx = vf.vf_create(0)
    vf.vf_set_space(ctx, sp)
    vf.vf_set_pipeline(ctx, np.repeat(pipe[None], K, axis=0))
    vf.vf_set_model(ctx, model, w)

    def run(last):
        vf.vf_reset_state(ctx)
        st, cids, vals, nb = vf.vf_beam_search(ctx, 0, last)
        return cids.cpu().numpy(), vals.cpu().numpy(), st.cpu().numpy(), int(nb.cpu()[0])
    return ctx, run


@pytest.mark.parametrize("K,dims", [(1, [256, 512, 512, 1]), (4, [256, 512, 512, 1]), (16, [256, 512, 512, 1]),
                                    (40, [256, 512, 512, 1]), (3, [256, 512, 512, 512, 512, 1])])
def test_beam_fused_bf16(vf, ovf, K, dims):
    """Lists of valid candidates; (three slots) a network of four hidden layers, whose biases do not fit next to a
    list's tile: the scorer on id ranges and the selection passes."""
    sp = I.make_space([1, 2, 3, 8], [1, 2, 5], [1, 4, 16], [(0, 1, 2), (2, 1, 0), (1, 0, 2)], 2, 2,
                      [I.ROOT, I.L1, I.L2, I.INLINE], 2, 256)
    pipe = I.random_pipeline(4, 41)
    w = I.mlp_weights(dims, 3, bias_std=0.1)
    model = I.model_record(I.MLP, dims, I.BF16)
    ctx, run = make_ctx(vf, pipe, sp, model, w, K)
    check_beam(ovf, pipe, sp, model, w, run, K, TOL[1])
    cids, vals, st, nb = run(len(pipe) - 1)
    if K == 1:
        vf.vf_reset_state(ctx)
        gs, gc, gv = vf.vf_greedy_schedule(ctx)
        assert np.array_equal(gc.cpu().numpy(), cids) and np.array_equal(gv.cpu().numpy(), vals)
        assert np.array_equal(gs.cpu().numpy(), st)
    vf.vf_destroy(ctx)


# the choice on lists: survivors ranked (up to 256 scores below the cut), sorted (more), bisected (more than 1024 parts
# or 2048 scores below it)
@pytest.mark.parametrize("K", [20, 250, 300, 700])
@pytest.mark.parametrize("same", [False, True])
def test_beam_choice_on_lists(vf, ovf, K, same):
    """Many slots; equal scores for all (zero weights), which the order of slots and ids decides."""
    sp = I.make_space([1, 2, 3, 8], [1, 2, 5], [1, 4, 16], [(0, 1, 2), (2, 1, 0)], 2, 1, [I.ROOT, I.L1, I.L2, I.INLINE], 2, 64)
    pipe = I.random_pipeline(3, 41)
    dims = [64, 512, 1]
    w = I.mlp_weights(dims, 3, bias_std=0.1)
    if same:
        w[:] = 0.0
        w[-1] = 0.75   # the output's bias
    model = I.model_record(I.MLP, dims, I.BF16)
    ctx, run = make_ctx(vf, pipe, sp, model, w, K)
    if same:
        cids, vals, st, nb = run(len(pipe) - 1)
        ref = ovf.beam(pipe, sp, K, model, w)
        assert np.array_equal(ref["cids"], cids) and np.array_equal(ref["values"], vals) and ref["n_beams"] == nb
    else:
        check_beam(ovf, pipe, sp, model, w, run, K, TOL[1])
    vf.vf_destroy(ctx)


# decisions of 8 and 96 ids; one slot with more than 512 of them
@pytest.mark.parametrize("K,factors", [(2, [1, 2]), (5, [1, 2, 4]), (1, [1, 2, 3, 8])])
def test_beam_lists_of_short_decisions(vf, ovf, K, factors):
    sp = I.make_space(factors, factors[:2], factors[-2:], [(0, 1, 2), (2, 1, 0)][:len(factors) - 1], 1 if K == 2 else 2, 1,
                      [I.ROOT] if K == 2 else [I.ROOT, I.L1] if K == 5 else [I.ROOT, I.L1, I.L2, I.INLINE], 1 if K > 1 else 3, 64)
    assert ovf.dense_count(sp) == {2: 8, 5: 96, 1: 768}[K]
    pipe = I.random_pipeline(4, 43)
    dims = [64, 512, 512, 1]
    w = I.mlp_weights(dims, 5, bias_std=0.1)
    model = I.model_record(I.MLP, dims, I.BF16)
    ctx, run = make_ctx(vf, pipe, sp, model, w, K)
    check_beam(ovf, pipe, sp, model, w, run, K, TOL[1])
    vf.vf_destroy(ctx)


# one slot with few ids: id ranges
@pytest.mark.parametrize("dims", [[64, 512, 512, 1], [256, 1024, 1]])
def test_beam_of_one_slot_with_short_decisions(vf, ovf, dims):
    sp = I.make_space([1, 2, 4], [1, 2], [1, 4], [(0, 1, 2), (2, 1, 0)], 2, 1, [I.ROOT, I.L1, I.L2, I.INLINE], 2, dims[0])
    assert ovf.dense_count(sp) == 384
    pipe = I.random_pipeline(5, 43)
    w, model = I.mlp_weights(dims, 5, bias_std=0.1), I.model_record(I.MLP, dims, I.BF16)
    ctx, run = make_ctx(vf, pipe, sp, model, w, 1)
    check_beam(ovf, pipe, sp, model, w, run, 1, TOL[1])
    cids, vals, st, nb = run(4)
    vf.vf_reset_state(ctx)
    gs, gc, gv = (t.cpu().numpy() for t in vf.vf_greedy_schedule(ctx))
    assert np.array_equal(gc, cids) and np.array_equal(gv, vals) and np.array_equal(gs, st)
    vf.vf_destroy(ctx)


@pytest.mark.parametrize("K", [2, 9, 300])
def test_beam_on_lists_ends_on_the_way(vf, ovf, K):
    """A layer without a valid candidate: the schedules so far are carried over as they are, by the workgroups that
    copy rows, and the layers behind it change nothing."""
    sp = I.make_space([1, 2, 4], [1, 2], [4, 8], [(0, 1, 2), (2, 1, 0)], 2, 1, [I.ROOT, I.L1], 2, 64)
    pipe = I.random_pipeline(5, 43)
    pipe[:, 3] = np.maximum(pipe[:, 3], 8)
    pipe[2, 3] = 2                                # fewer channels than every channel factor
    dims = [64, 512, 1]
    w, model = I.mlp_weights(dims, 5, bias_std=0.1), I.model_record(I.MLP, dims, I.BF16)
    ctx, run = make_ctx(vf, pipe, sp, model, w, K)
    check_beam(ovf, pipe, sp, model, w, run, K, TOL[1])
    before = run(1)
    assert before[3] == K and (before[0][:, 1] >= 0).all()
    for last in (2, 4):
        for a, b in zip(before, run(last)):
            assert np.array_equal(a, b)
    vf.vf_destroy(ctx)


# 1024 slots with 10 and with 33 parts each: more minima than the bins take in two and in eight rounds, and more than
# they take at all
@pytest.mark.parametrize("n", [588, 2100])
@pytest.mark.parametrize("same", [False, True])
def test_beam_choice_among_many_minima(vf, n, same):
    """Every id is valid.  Equal scores: the first (slot, id) pairs.  Others: against the scores of all extensions of the
    survivors before, which vf_score gives from their features."""
    import torch
    f = lambda k: list(range(1, k + 1))
    nx, ny, nc, nperm, nvec = {588: (7, 7, 4, 3, 1), 2100: (7, 5, 5, 6, 2)}[n]
    sp = I.make_space(f(nx), f(ny), f(nc), I.ALL_PERMS[:nperm], nvec, 1, [I.ROOT], 1, 64)
    assert I.space_dense_count(sp) == n
    K, dims = 1024, [64, 512, 1]
    pipe = I.resnet18_shaped()[:3].copy()
    pipe[:, 1:4] = np.maximum(pipe[:, 1:4], 8)
    w = I.mlp_weights(dims, 3, bias_std=0.1)
    if same:
        w[:] = 0.0
        w[-1] = 0.75
    model = I.model_record(I.MLP, dims, I.BF16)
    ctx, run = make_ctx(vf, pipe, sp, model, w, K)
    cids, vals, st, nb = run(2)
    assert nb == K
    if same:
        rows = [()]
        for _ in range(3):
            rows = [r + (i,) for r in rows[:K // n + 1] for i in range(n)][:K]
        assert cids.tolist() == [list(r) for r in rows] and (vals == 0.75).all()
        vf.vf_destroy(ctx)
        return
    prev, _, _, _ = run(1)
    assert (prev[:, 1] >= 0).all()
    vf.vf_set_state(ctx, np.ascontiguousarray(prev[:, :2]))
    Mp = vf.vf_padded_count(ctx)
    x = vf.vf_featurize(ctx, 2).permute(1, 0, 2).reshape(64, K * Mp).contiguous()
    ref = vf.vf_score(ctx, x, want_min=False)[0].reshape(K, Mp)[:, :n].double().cpu().numpy()
    at = {tuple(r): j for j, r in enumerate(prev[:, :2].tolist())}
    pairs = [(at[tuple(r[:2])], r[2]) for r in cids.tolist()]
    assert len(set(pairs)) == K and (np.diff(vals[:, 2]) >= 0).all()
    scale, tol = np.sqrt(np.mean(ref ** 2)), TOL[1]
    got = np.array([ref[p] for p in pairs])
    assert np.abs(got - vals[:, 2]).max() <= tol * max(np.abs(got).max(), scale)
    better = np.argwhere(ref < vals[:, 2].max() - 2 * tol * max(abs(vals[:, 2].max()), scale))
    assert set(map(tuple, better.tolist())) <= set(pairs)
    vf.vf_destroy(ctx)


@pytest.mark.parametrize("K", [6, 24])
def test_beam_fp32_tiny_config_with_ties(vf, ovf, K):
    """The tiny conv+ReLU config has candidates with identical features, hence exactly
    equal scores: the (score, parent, candidate id) order decides, as in the checker
    (few survivors: rounds of block minima; more: sorted keys)."""
    pipe, sp = I.tiny_conv_relu(), I.tiny_space()
    dims = [64, 128, 128, 1]
    w = I.mlp_weights(dims, 0)
    model = I.model_record(I.MLP, dims, I.FP32)
    ctx, run = make_ctx(vf, pipe, sp, model, w, K)
    check_beam(ovf, pipe, sp, model, w, run, K, TOL[0])
    cids, vals, st, nb = run(1)
    ref = ovf.beam(pipe, sp, K, model, w)
    assert np.array_equal(ref["cids"], cids) and ref["n_beams"] == nb
    vf.vf_destroy(ctx)


@pytest.mark.parametrize("dims", [[64, 96, 32, 1], [64, 160, 32, 1]])
def test_beam_general_widths_and_prefix(vf, ovf, dims):
    """Models outside the fused path - a small one, which generates its candidates itself, and one for
    which the features are materialised and the scores masked afterwards - and a search that starts
    from a committed prefix (the way Algorithm 2 completes schedules)."""
    sp = I.make_space([1, 2, 4], [1, 2], [1, 4], [(0, 1, 2), (2, 1, 0)], 2, 1,
                      [I.ROOT, I.L1, I.L2, I.INLINE], 1, 64)
    pipe = I.random_pipeline(4, 52)
    w = I.mlp_weights(dims, 9, bias_std=0.1)
    model = I.model_record(I.MLP, dims, I.BF16)
    ctx, run = make_ctx(vf, pipe, sp, model, w, 5)
    check_beam(ovf, pipe, sp, model, w, run, 5, TOL[1])
    cids, vals, st, nb = run(3)
    ref = ovf.beam(pipe, sp, 5, model, w)
    if np.array_equal(ref["cids"], cids):                    # no decision inside the tolerance
        assert ref["n_beams"] == nb
    # from the best schedule's first decision onwards
    first = int(cids[0, 0])
    vf.vf_set_state(ctx, np.full((5, 1), first, np.int32))
    st2, c2, v2, nb2 = vf.vf_beam_search(ctx, first=1)
    c2 = c2.cpu().numpy()
    assert (c2[c2[:, 0] >= 0, 0] == first).all()
    if dims[1] == 96:  # (this network's best schedule is found from its first decision as well)
        assert c2[0].tolist() == cids[0].tolist()

    def onwards(last):
        vf.vf_set_state(ctx, np.full((5, 1), first, np.int32))
        st, cids, vals, nb = vf.vf_beam_search(ctx, 1, last)
        return cids.cpu().numpy(), vals.cpu().numpy(), st.cpu().numpy(), int(nb.cpu()[0])
    check_beam(ovf, pipe, sp, model, w, onwards, 5, TOL[1], start=(first,))
    with pytest.raises(vf.VfError):
        vf.vf_beam_search(ctx, first=0)                      # not the next stage
    other = I.random_pipeline(4, 53)
    vf.vf_set_pipeline(ctx, np.stack([pipe, pipe, other, pipe, pipe]))
    with pytest.raises(vf.VfError) as e:
        vf.vf_beam_search(ctx)                               # slots must hold one network
    assert e.value.code == vf.VF_EINVAL
    vf.vf_destroy(ctx)


def test_beam_without_survivors(vf, ovf):
    pipe, sp = I.tiny_conv_relu(), I.tiny_space()
    dims = [64, 32, 1]
    w = I.mlp_weights(dims, 0); w[:] = np.nan
    ctx, run = make_ctx(vf, pipe, sp, I.model_record(I.MLP, dims, I.BF16), w, 3)
    cids, vals, st, nb = run(1)
    assert (cids == -1).all() and np.isinf(vals).all() and not st.any() and nb == 1
    vf.vf_destroy(ctx)
