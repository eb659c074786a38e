"""GPU: schedules of a few problems in one launch (vf_chain.hip, vf_small.hip) against the launches layer by layer, bit for bit."""
import numpy as np
import pytest

from paper_2011_14486_amd import inputs as I
from tests.test_gpu_greedy import greedy_with_launches

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vf():
    import paper_2011_14486_amd as pkg
    return pkg.load()


def space(shape, F):
    """Decisions of whole tiles of 32 or 64 ids, of a last tile that is nearly empty or nearly full, of one tile."""
    perms = [(0, 1, 2), (2, 1, 0)]
    if shape == "whole":
        return I.make_space([1, 2, 4], [1, 4], [4, 8], perms, 2, 2, [I.ROOT, I.L1, I.L2, I.INLINE], 2, F)   # 768
    if shape == "odd":
        return I.make_space([1, 2, 4], [1, 2, 4, 7, 14], [1, 4, 8], perms[:1], 1, 1, [I.ROOT, I.L1, I.L2], 3, F)   # 405
    if shape == "full":
        return I.make_space([1, 2, 4], [1, 2, 4], [1, 4, 8, 16, 32, 64, 128], perms[:1], 1, 1, [I.ROOT], 1, F)   # 63
    return I.make_space([1, 2], [1], [4], perms, 1, 1, [I.ROOT, I.L2], 1, F)                                  # 8


def context(vf, pipes, sp, dims, dtype=I.BF16):
    ctx = vf.vf_create(0)
    vf.vf_set_space(ctx, sp); vf.vf_set_pipeline(ctx, pipes)
    vf.vf_set_model(ctx, I.model_record(I.MLP, dims, dtype), I.mlp_weights(dims, 3, bias_std=0.1))
    return ctx


def layer_by_layer(vf, ctx):
    vf.vf_reset_state(ctx)
    S = len(vf.vf_greedy_schedule(ctx, last=-1)[1][0])
    for i in range(S):
        vf.vf_argmin_step(ctx, i, True)
    return [t.cpu().numpy() for t in vf.vf_greedy_schedule(ctx, first=S)]


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


# 768 ids: tiles of 32 up to 10 problems (256 compute units), of 64 behind that; wait 0: every minimum that is not
# there at once is worked out by the workgroup that misses it
@pytest.mark.parametrize("dims", [[256, 512, 512, 1], [64, 512, 512, 1], [256, 512, 1], [256, 512, 512, 512, 1]])
@pytest.mark.parametrize("shape,B", [("whole", 1), ("whole", 11), ("odd", 3), ("odd", 23), ("full", 2), ("one", 1)])
@pytest.mark.parametrize("wait", [1 << 22, 0])
def test_chain_equals_layer_by_layer(vf, dims, shape, B, wait):
    pipes = np.stack([I.random_pipeline(7, 70 + b, max_hw=60, max_c=160) for b in range(B)])
    pipes[B // 2, 2, 3] = 2                       # fewer channels than every channel factor of the first space
    ctx = context(vf, pipes, space(shape, dims[0]), dims)
    vf.vf_set_wait_limit(ctx, wait)
    for eps in (0.0, 0.1):
        vf.vf_set_noise(ctx, eps, 11, 2)
        whole, launches = greedy_with_launches(vf, ctx)
        assert launches == 1
        assert same(whole, layer_by_layer(vf, ctx))
    vf.vf_sync_status(ctx)
    vf.vf_destroy(ctx)


def test_chain_of_one_layer_and_of_many(vf):
    """One stage; 300 stages, in two pieces and without the caller's tables in between."""
    dims, sp = [256, 512, 512, 1], space("whole", 256)
    for S, cut in ((1, None), (300, 123)):
        ctx = context(vf, I.random_pipeline(S, 8), sp, dims)
        ref = layer_by_layer(vf, ctx)
        whole, launches = greedy_with_launches(vf, ctx)
        assert launches == 1 and same(whole, ref)
        if cut:
            vf.vf_reset_state(ctx)
            vf.vf_greedy_schedule(ctx, last=cut)
            best, value = (t.cpu().numpy() for t in vf.vf_argmin_step(ctx, cut + 1, True))   # from the context left behind
            assert best[0] == ref[1][0, cut + 1] and value[0] == ref[2][0, cut + 1]
            assert same([t.cpu().numpy() for t in vf.vf_greedy_schedule(ctx, first=cut + 2)], ref)
        vf.vf_destroy(ctx)


def test_chain_in_a_graph(vf):
    """Captured and replayed, with the context's own calls in between: the launch leaves its words as it found them."""
    import torch
    dims, s = [256, 512, 512, 1], torch.cuda.Stream()
    with torch.cuda.stream(s):
        ctx = vf.vf_create(0, s)
        vf.vf_set_space(ctx, space("whole", 256)); vf.vf_set_pipeline(ctx, I.resnet18_batch(2, seed=5))
        vf.vf_set_model(ctx, I.model_record(I.MLP, dims, I.BF16), I.mlp_weights(dims, 3, bias_std=0.1))
        S = 20
        out = (ctx.empty((2, S, 16), torch.int32), ctx.empty((2, S), torch.int32), ctx.empty((2, S), torch.float32))
        vf.vf_greedy_schedule(ctx, out=out)
        s.synchronize()
        ref = [t.cpu().numpy() for t in out]
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            vf.vf_reset_state(ctx)
            vf.vf_greedy_schedule(ctx, out=out)
        for k in range(4):
            for t in out:
                t.zero_()
            g.replay()
            s.synchronize()
            assert same([t.cpu().numpy() for t in out], ref)
            vf.vf_reset_state(ctx)
            assert same([t.cpu().numpy() for t in vf.vf_greedy_schedule(ctx, last=9 + k)][1][:, :10 + k], ref[1][:, :10 + k])
        vf.vf_destroy(ctx)


@pytest.mark.parametrize("dims,dtype", [([256, 512, 512, 1], I.BF16), ([64, 128, 128, 1], I.FP32)])
def test_first_schedule_of_a_context_in_a_graph(vf, dims, dtype):
    """Captured before the context has made its words, and called before the graph has run."""
    import torch
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        pipes = I.resnet18_batch(2, seed=5)[:, :6]
        ref = context(vf, pipes, space("whole", dims[0]), dims, dtype)
        want = [t.cpu().numpy() for t in vf.vf_greedy_schedule(ref)]
        vf.vf_destroy(ref)
        ctx = vf.vf_create(0, s)
        vf.vf_set_space(ctx, space("whole", dims[0])); vf.vf_set_pipeline(ctx, pipes)
        vf.vf_set_model(ctx, I.model_record(I.MLP, dims, dtype), I.mlp_weights(dims, 3, bias_std=0.1))
        out = (ctx.empty((2, 6, 16), torch.int32), ctx.empty((2, 6), torch.int32), ctx.empty((2, 6), torch.float32))
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s, capture_error_mode="relaxed"):
            vf.vf_reset_state(ctx)
            vf.vf_greedy_schedule(ctx, out=out)
        for k in range(3):
            vf.vf_reset_state(ctx)
            assert same([t.cpu().numpy() for t in vf.vf_greedy_schedule(ctx)], want)
            for t in out:
                t.zero_()
            g.replay()
            s.synchronize()
            assert same([t.cpu().numpy() for t in out], want)
        vf.vf_destroy(ctx)


# small networks: one, four or eight waves of a workgroup have a sub-tile (32 ids in bf16, 16 in fp32), the last ones
# none or part of one; 768 ids: 12 tiles of 64 in fp32 up to 21 problems, of 128 behind that
@pytest.mark.parametrize("dims,dtype", [([64, 128, 128, 1], I.FP32), ([256, 40, 24, 1], I.FP32), ([64, 96, 32, 1], I.BF16),
                                        ([256, 64, 1], I.BF16)])
@pytest.mark.parametrize("shape,B", [("whole", 1), ("whole", 22), ("odd", 3), ("full", 2), ("one", 40)])
@pytest.mark.parametrize("wait", [1 << 22, 0])
def test_small_chain_equals_layer_by_layer(vf, dims, dtype, shape, B, wait):
    pipes = np.stack([I.random_pipeline(7, 70 + b, max_hw=60, max_c=160) for b in range(B)])
    pipes[B // 2, 2, 3] = 2
    ctx = context(vf, pipes, space(shape, dims[0]), dims, dtype)
    vf.vf_set_wait_limit(ctx, wait)
    for eps in (0.0, 0.1):
        vf.vf_set_noise(ctx, eps, 11, 2)
        whole, launches = greedy_with_launches(vf, ctx)
        assert launches == 1
        assert same(whole, layer_by_layer(vf, ctx))
    vf.vf_reset_state(ctx)
    vf.vf_greedy_schedule(ctx, last=2)
    best, value = (t.cpu().numpy() for t in vf.vf_argmin_step(ctx, 3, True))
    assert np.array_equal(best, whole[1][:, 3]) and np.array_equal(value, whole[2][:, 3])
    vf.vf_destroy(ctx)
