"""GPU: schedules and beams of a few problems on lists with tiles of 64 candidates."""
import numpy as np
import pytest

from paper_2011_14486_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vf():
    import paper_2011_14486_amd as pkg
    return pkg.load()


def context(vf, pipes, sp, dims, w):
    ctx = vf.vf_create(0)
    vf.vf_set_space(ctx, sp); vf.vf_set_pipeline(ctx, pipes); vf.vf_set_model(ctx, I.model_record(I.MLP, dims, I.BF16), w)
    return ctx


def space(tiles, F):
    """A decision of 64 or 36 tiles of 64 ids."""
    fx = [1, 2, 4, 8] if tiles == 64 else [1, 2, 4]
    sp = I.make_space(fx, fx, [4, 8], I.XC_INNER_PERMS, 2, 2, [I.ROOT, I.L1, I.L2, I.INLINE], 2, F)
    assert I.space_dense_count(sp) == 64 * tiles
    return sp


# the smallest and the largest batch of the range and one problem before and behind it (256 compute
# units), with and without a folded first layer
@pytest.mark.parametrize("tiles,B,lists", [(64, 4, False), (64, 5, True), (64, 8, True), (64, 9, True),
                                           (36, 7, False), (36, 8, True), (36, 14, True)])
@pytest.mark.parametrize("dims", [[256, 512, 512, 1], [64, 512, 512, 512, 1]])
def test_few_problems_equal_single_ones(vf, tiles, B, lists, dims):
    """Ids and values of every layer bit-identical to those of one problem alone, with noise and with a
    problem whose schedule ends early."""
    sp, w = space(tiles, dims[0]), I.mlp_weights(dims, 4, bias_std=0.1)
    pipes = np.stack([I.random_pipeline(5, 40 + b) for b in range(B)])
    pipes[1, 2, 3] = 2
    many = context(vf, pipes, sp, dims, w)
    vf.vf_set_noise(many, 0.2, 9, 0)
    vf.vf_profile_enable(many, True); vf.vf_profile_counts(many)
    whole = [t.cpu().numpy() for t in vf.vf_greedy_schedule(many)]
    scored, valid = vf.vf_profile_counts(many)
    assert valid > 0 and (scored == valid) == lists        # only listed candidates are scored on lists
    for b in range(B):
        one = context(vf, pipes[b], sp, dims, w)
        vf.vf_set_noise(one, 0.2, 9, b)
        st, cids, vals = (t.cpu().numpy()[0] for t in vf.vf_greedy_schedule(one))
        assert np.array_equal(cids, whole[1][b]) and np.array_equal(st, whole[0][b]) and np.array_equal(vals, whole[2][b])
        vf.vf_destroy(one)
    vf.vf_destroy(many)


@pytest.mark.parametrize("tiles,K", [(64, 5), (64, 8), (36, 14)])
@pytest.mark.parametrize("const", [True, False])
def test_beam_of_few_slots(vf, ovf, tiles, K, const):
    """Survivors of a network whose value is the same for every state: the first (slot, id) pairs, exactly.
    Of another network: the best one is what a single problem decides after its prefix, bit for bit."""
    dims = [256, 512, 512, 1]
    sp, w, pipe = space(tiles, 256), I.mlp_weights(dims, 5, bias_std=0.1), I.random_pipeline(3, 21)
    if const:
        w = np.zeros_like(w)
        w[-1] = 0.75
    ctx = context(vf, np.stack([pipe] * K), sp, dims, w)
    st, cids, vals, nb = (t.cpu().numpy() for t in vf.vf_beam_search(ctx))
    vf.vf_destroy(ctx)
    assert nb[0] == K
    if const:
        ref = ovf.beam(pipe, sp, K, I.model_record(I.MLP, dims, I.BF16), w)
        assert np.array_equal(cids, ref["cids"]) and np.array_equal(vals, ref["values"])
        return
    one = context(vf, pipe, sp, dims, w)
    vf.vf_set_state(one, np.ascontiguousarray(cids[:1, :2]))
    best, value = (t.cpu().numpy()[0] for t in vf.vf_argmin_step(one, 2, True))
    vf.vf_destroy(one)
    assert best == cids[0, 2] and value == vals[0, 2]
