"""GPU parity of the recurrent search at every width that the network can have: the forms that hold the
recurrent weights in registers and LDS (one, two or several workgroups per compute unit, with and without
a stream for what does not fit), tiles of 32 and of 64 candidates, lists that end inside and at the end of a
tile, problems without candidates in between."""
import numpy as np
import pytest

from paper_2011_14486_amd import inputs as I
from tests.test_gpu_lstm_search import compare_schedule, setup
from tests.util import TOL, score_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vf():
    import paper_2011_14486_amd as pkg
    return pkg.load()


@pytest.mark.parametrize("H", range(32, 257, 32))
def test_every_width(vf, ovf, H):
    """One problem (tiles of 32) and 70 (768 tiles of 64 ids or more: the forms for throughput) of
    different lists: ids, values and states of the batch are those of single problems, bit for bit, and the
    checker's (the same tolerance as everywhere for bf16)."""
    sp = I.make_space([1, 2, 4], [1, 3, 4], [1, 2, 8], I.ALL_PERMS[:2], 2, 2, [I.ROOT, I.L1, I.L2, I.INLINE], 2, 64)
    B = 70
    assert (I.space_dense_count(sp) + 63) // 64 * B >= 3 * 256
    pipes = np.stack([I.random_pipeline(4, 60 + b % 9) for b in range(B)])
    ctx, model, w = setup(vf, pipes, sp, H)
    st, cids, vals = [t.cpu().numpy() for t in vf.vf_greedy_schedule(ctx)]
    vf.vf_destroy(ctx)
    for b in (0, 4, 8):
        compare_schedule(ovf, pipes[b], sp, model, w, cids[b], vals[b], st[b], TOL[1])
    for b in range(9):
        one, _, _ = setup(vf, pipes[b], sp, H)
        s1, c1, v1 = [t.cpu().numpy()[0] for t in vf.vf_greedy_schedule(one)]
        vf.vf_destroy(one)
        for k in range(b, B, 9):
            assert np.array_equal(c1, cids[k]) and np.array_equal(v1, vals[k]) and np.array_equal(s1, st[k])


@pytest.mark.parametrize("H", [32, 128, 192, 256])
@pytest.mark.parametrize("fx,fy,fc", [([1], [1], [1]), ([1, 2, 4, 8], [1, 2, 4, 8], [1, 2]), ([1, 2, 4], [1, 2, 3, 4], [1, 2, 4]),
                                      ([1, 2, 4, 8], [1, 2, 4, 8], [1, 2, 3, 4]), ([1, 2, 3, 4, 5], [1, 2, 3, 4, 5], [1, 2, 3])])
def test_ends_of_tiles(vf, ovf, H, fx, fy, fc):
    """Lists of 1, 32, 36, 64 and 75 entries."""
    sp = I.make_space(fx, fy, fc, I.ALL_PERMS[:1], 1, 1, [I.ROOT], 1, 64)
    pipe = I.random_pipeline(3, 13)
    assert (pipe[:, 1:4] >= [max(fx), max(fy), max(fc)]).all()  # (every candidate is valid)
    ctx, model, w = setup(vf, pipe, sp, H)
    st, cids, vals = [t.cpu().numpy()[0] for t in vf.vf_greedy_schedule(ctx)]
    vf.vf_destroy(ctx)
    compare_schedule(ovf, pipe, sp, model, w, cids, vals, st, TOL[1])


@pytest.mark.parametrize("F,H", [(F, H) for F in range(32, 257, 32) for H in range(32, 193, 32)])
def test_sequences(vf, ovf, F, H):
    """Sequences through the networks that a workgroup holds and the smallest ones that it does not (F = 96 with
    H = 160, 256 with 128): one tile, ragged tiles, minima per group."""
    import torch
    w, model = I.lstm_weights(F, H, seed=4, bias_std=0.2), I.model_record(I.LSTM, [F, H, 1], I.BF16)
    ctx = vf.vf_create(0)
    vf.vf_set_model(ctx, model, w)
    for M, T, group in ((1, 3, 0), (32, 1, 0), (300, 2, 128), (33, 6, 0)):
        rng = np.random.default_rng([F, H, M])
        x = torch.from_numpy((rng.random((M, T, F)) * 20).astype(np.float32)).to(torch.bfloat16)
        s, bi, bv = vf.vf_score(ctx, x.cuda(), vf.VF_X_SEQ_BF16, group=group)
        s, bi, bv = s.cpu().numpy(), bi.cpu().numpy(), bv.cpu().numpy()
        assert score_err(s, ovf.score_lstm(model, w, x.view(torch.int16).numpy().view(np.uint16))) <= TOL[1]
        g = group or M
        for k in range(len(bi)):
            part = s[k * g:(k + 1) * g]
            assert bi[k] == k * g + int(np.argmin(part)) and bv[k] == part.min()
    vf.vf_destroy(ctx)


def test_more_sequences_than_minima(vf):
    """Above 32 * 65536 sequences a minimum covers two tiles: the scores are those of a small call."""
    import torch
    F, H, M = 32, 32, 32 * 65536 + 65
    w, model = I.lstm_weights(F, H, seed=4, bias_std=0.2), I.model_record(I.LSTM, [F, H, 1], I.BF16)
    ctx = vf.vf_create(0)
    vf.vf_set_model(ctx, model, w)
    x = (torch.rand((M, 1, F), device="cuda", generator=torch.Generator(device="cuda").manual_seed(1)) * 20).to(torch.bfloat16)
    s, bi, bv = vf.vf_score(ctx, x, vf.VF_X_SEQ_BF16)
    tail, _, _ = vf.vf_score(ctx, x[-1000:].contiguous(), vf.VF_X_SEQ_BF16)
    assert torch.equal(s[-1000:], tail)
    assert float(bv[0]) == float(s.min()) and int(bi[0]) == int((s == s.min()).to(torch.int8).argmax())
    s2, bi2, bv2 = vf.vf_score(ctx, x, vf.VF_X_SEQ_BF16, group=128)
    want = torch.nn.functional.pad(s, (0, -M % 128), value=float("inf")).reshape(-1, 128)
    assert torch.equal(s2, s) and torch.equal(bv2, want.min(dim=1).values)
    vf.vf_destroy(ctx)


@pytest.mark.parametrize("K", [3, 20])
def test_searches_one_behind_the_other(vf, K):
    """The prefix's step goes along with the opening of a call's next decision, the last one at the call's end: a
    beam, a greedy schedule and single steps on top of each other decide what they decide on the same prefix set by hand, bit for bit."""
    sp = I.make_space([1, 2, 4], [1, 3], [1, 2, 8], I.ALL_PERMS[:2], 2, 2, [I.ROOT, I.L1, I.L2, I.INLINE], 1, 64)
    pipes = np.stack([I.random_pipeline(6, 77)] * K)

    def context():
        return setup(vf, pipes, sp, 64)[0]

    def host(ts):
        return [t.cpu().numpy() for t in ts]

    def on_prefix(cids, n, what):
        c = context()
        vf.vf_set_state(c, np.ascontiguousarray(cids[:, :n]))
        out = host(what(c))
        vf.vf_destroy(c)
        return out
    ctx = context()
    first = host(vf.vf_beam_search(ctx, 0, 1))[1]
    got = host(vf.vf_greedy_schedule(ctx, 2, 3))                    # every slot goes on by itself
    for a, b in zip(on_prefix(first, 2, lambda c: vf.vf_greedy_schedule(c, 2, 3)), got):
        assert np.array_equal(a[:, 2:4], b[:, 2:4])
    got = host(vf.vf_beam_search(ctx, 4, 4))                        # from slot 0's schedule
    mixed = np.repeat(got[1][:1], K, axis=0)
    want = on_prefix(mixed, 4, lambda c: vf.vf_beam_search(c, 4, 4))
    assert np.array_equal(want[1], got[1]) and np.array_equal(want[2][:, 4], got[2][:, 4])
    nb = int(got[3][0])
    again = host(vf.vf_beam_search(ctx, 5, 5))                      # and from the best of those
    want = on_prefix(np.repeat(got[1][:1], K, axis=0), 5, lambda c: vf.vf_beam_search(c, 5, 5))
    assert nb == K and np.array_equal(want[1], again[1]) and np.array_equal(want[2][:, 5], again[2][:, 5])
    vf.vf_reset_state(ctx)
    for i in range(2):
        vf.vf_argmin_step(ctx, i, True)
    vf.vf_reset_state(ctx)                                          # (nothing of it outlives its state)
    a, b = host(vf.vf_greedy_schedule(ctx)), on_prefix(first[:, :0], 0, vf.vf_greedy_schedule)
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
    vf.vf_destroy(ctx)


def test_spaces_one_behind_the_other(vf, ovf):
    """A larger and a smaller space on the same context: each search as on a context of its own."""
    pipe = I.random_pipeline(4, 61)
    spaces = [I.make_space([1, 2], [1, 2], [1, 2], I.ALL_PERMS[:1], 1, 1, [I.ROOT], 1, 64),
              I.make_space([1, 2, 4], [1, 2, 4], [1, 2, 4], I.ALL_PERMS, 2, 2, [I.ROOT, I.L1], 1, 64)]
    ctx, model, w = setup(vf, np.stack([pipe] * 3), spaces[0], 64)
    for sp in (spaces[0], spaces[1], spaces[0]):
        vf.vf_set_space(ctx, sp)
        st, cids, vals = [t.cpu().numpy() for t in vf.vf_greedy_schedule(ctx)]
        for b in range(3):
            compare_schedule(ovf, pipe, sp, model, w, cids[b], vals[b], st[b], TOL[1])
    vf.vf_destroy(ctx)
