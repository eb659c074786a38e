"""GPU parity: candidate enumeration and features, bit-exact against the CPU checker,
through the C ABI."""
import numpy as np
import pytest

from paper_2011_14486_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vf():
    import paper_2011_14486_amd as pkg
    return pkg.load()


def random_prefix(ovf, pipe, space, n, rng):
    pre = []
    for i in range(n):
        _, v, nv = ovf.enumerate_candidates(pipe, space, pre, i)
        pre.append(int(rng.choice(np.flatnonzero(v))))
    return pre


def compare_stage(vf, ovf, ctx, pipes, space, prefixes, stage):
    dec, valid, nv = vf.vf_enumerate(ctx, stage)
    feat = vf.vf_featurize(ctx, stage)
    dec = dec.cpu().numpy().view(np.uint32); valid = valid.cpu().numpy(); nv = nv.cpu().numpy()
    feat = feat.cpu().numpy()
    for b, (pipe, pre) in enumerate(zip(pipes, prefixes)):
        rdec, rvalid, rnv = ovf.enumerate_candidates(pipe, space, pre, stage)
        rfeat = ovf.featurize(pipe, space, pre, stage)
        assert np.array_equal(dec[b], rdec), (b, stage)
        assert np.array_equal(valid[b], rvalid), (b, stage)
        assert nv[b] == rnv
        if not np.array_equal(feat[b], rfeat):
            bad = np.argwhere(feat[b] != rfeat)
            raise AssertionError(f"problem {b} stage {stage}: {len(bad)} feature cells differ, first "
                                 f"(row, cid) {bad[0]}: gpu {feat[b][tuple(bad[0])]} ref {rfeat[tuple(bad[0])]}")


def test_tiny_config_both_orders(vf, ovf):
    sp = I.tiny_space()
    rng = np.random.default_rng(0)
    for order in ("output_first", "input_first"):
        pipe = I.tiny_conv_relu(order)
        ctx = vf.vf_create(0)
        vf.vf_set_space(ctx, sp)
        vf.vf_set_pipeline(ctx, pipe)
        assert vf.vf_dense_count(ctx) == 6000 and vf.vf_padded_count(ctx) == 6144
        compare_stage(vf, ovf, ctx, [pipe], sp, [[]], 0)
        pre = random_prefix(ovf, pipe, sp, 1, rng)
        vf.vf_set_state(ctx, pre)
        assert vf.vf_n_scheduled(ctx) == 1
        compare_stage(vf, ovf, ctx, [pipe], sp, [pre], 1)
        compare_stage(vf, ovf, ctx, [pipe], sp, [pre], 0)   # an earlier stage can be revisited
        vf.vf_destroy(ctx)


@pytest.mark.parametrize("F", [64, 256])
def test_random_pipelines_batched(vf, ovf, F):
    """B different small pipelines with different committed prefixes in one context:
    ragged M (not a multiple of 256), all four compute_at levels, store_at hoists."""
    sp = I.make_space([1, 2, 3, 8], [1, 2, 5], [1, 4, 16], [(0, 1, 2), (2, 1, 0), (1, 0, 2)], 2, 2,
                      [I.ROOT, I.L1, I.L2, I.INLINE], 3, F)
    rng = np.random.default_rng(F)
    S, B = 6, 7
    pipes = [I.random_pipeline(S, 100 + b) for b in range(B)]
    ctx = vf.vf_create(0)
    vf.vf_set_space(ctx, sp)
    vf.vf_set_pipeline(ctx, np.stack(pipes))
    full = [random_prefix(ovf, p, sp, S - 1, rng) for p in pipes]
    for n in (0, 1, 3, 5):
        pres = [f[:n] for f in full]
        vf.vf_set_state(ctx, np.array(pres, np.int32).reshape(B, n))
        compare_stage(vf, ovf, ctx, pipes, sp, pres, n)
    # committed state records agree as well
    vf.vf_set_model(ctx, I.model_record(I.MLP, [F, 8, 1], I.FP32), I.mlp_weights([F, 8, 1], 0))
    vf.vf_set_state(ctx, np.array(full, np.int32))
    st, cids, vals = vf.vf_greedy_schedule(ctx, first=S - 1, last=S - 2)  # empty range: just read back
    st = st.cpu().numpy(); cids = cids.cpu().numpy()
    for b in range(B):
        rst, _ = ovf.states(pipes[b], sp, full[b])
        assert np.array_equal(st[b, :S - 1], rst) and not st[b, S - 1].any()
        assert cids[b, :S - 1].tolist() == full[b] and cids[b, S - 1] == -1
    vf.vf_destroy(ctx)


def test_resnet_and_mobilenet_shapes(vf, ovf):
    rng = np.random.default_rng(11)
    for pipe, sp, stages in ((I.resnet18_shaped(), I.resnet18_space(), (0, 1, 4, 5, 12, 19)),
                             (I.mobilenetv2_shaped(), I.mobilenetv2_space(), (0, 3, 50, 99))):
        pre = random_prefix(ovf, pipe, sp, max(stages), rng)
        ctx = vf.vf_create(0)
        vf.vf_set_space(ctx, sp)
        vf.vf_set_pipeline(ctx, pipe)
        for s in stages:
            vf.vf_set_state(ctx, pre[:s])
            compare_stage(vf, ovf, ctx, [pipe], sp, [pre[:s]], s)
        vf.vf_destroy(ctx)


def test_saturating_features(vf, ovf):
    sp = I.make_space([1, 2], [1], [1], [(0, 1, 2)], 1, 1, [I.ROOT], 1, 64)
    pipe = np.array([I.stage_record(I.CONV, 60000, 60000, 8, RC=64, KH=7, KW=7, anchor=-1)], np.int32)
    ctx = vf.vf_create(0)
    vf.vf_set_space(ctx, sp); vf.vf_set_pipeline(ctx, pipe)
    compare_stage(vf, ovf, ctx, [pipe], sp, [[]], 0)
    vf.vf_destroy(ctx)


def test_error_codes(vf, ovf):
    sp = I.tiny_space()
    pipe = I.tiny_conv_relu()
    ctx = vf.vf_create(0)
    with pytest.raises(vf.VfError) as e:
        vf.vf_set_pipeline(ctx, pipe)           # no space yet
    assert e.value.code == vf.VF_ESTATE
    bad = sp.copy(); bad[64] = 100
    with pytest.raises(vf.VfError) as e:
        vf.vf_set_space(ctx, bad)
    assert e.value.code == vf.VF_EINVAL
    vf.vf_set_space(ctx, sp)
    wrong = pipe.copy(); wrong[1, 8] = 1        # anchor not listed earlier
    with pytest.raises(vf.VfError) as e:
        vf.vf_set_pipeline(ctx, wrong)
    assert e.value.code == vf.VF_EINVAL
    vf.vf_set_pipeline(ctx, pipe)
    with pytest.raises(vf.VfError) as e:
        vf.vf_featurize(ctx, 1)                  # stage 0 is not committed yet
    assert e.value.code == vf.VF_ESTATE
    with pytest.raises(vf.VfError) as e:
        vf.vf_featurize(ctx, 2)
    assert e.value.code == vf.VF_EINVAL
    _, v0, _ = ovf.enumerate_candidates(pipe, sp, [], 0)
    with pytest.raises(vf.VfError) as e:
        vf.vf_set_state(ctx, [int(np.flatnonzero(v0 == 0)[0])])   # invalid candidate as prefix
    assert e.value.code == vf.VF_ESTATE and vf.vf_n_scheduled(ctx) == 0
    with pytest.raises(vf.VfError) as e:
        vf.vf_argmin_step(ctx, 0)                # no model
    assert e.value.code == vf.VF_ESTATE
    assert vf.lib().vf_strerror(-2).decode().startswith("call out of order")
    vf.vf_destroy(ctx)


def test_features_of_more_problems_than_a_launch_takes(vf):
    """90,000 problems of 256 rows: 193 workgroups each are more than 2^32 work-items, so that the last
    problems come from a second launch.  All problems are the same one."""
    import torch
    B, sp = 90000, I.make_space([1, 2], [1, 2], [1, 2], [(0, 1, 2)], 1, 1, [I.ROOT], 1, 256)
    ctx = vf.vf_create(0)
    vf.vf_set_space(ctx, sp)
    vf.vf_set_pipeline(ctx, np.stack([I.random_pipeline(2, 3)] * B))
    feat = vf.vf_featurize(ctx, 0)
    first = feat[0].clone()
    assert int(first[16].sum()) > 0 and int(first[208:224].sum()) > 0
    for b in range(0, B, 10000):
        assert bool((feat[b:b + 10000] == first).all()), b
    vf.vf_destroy(ctx)
