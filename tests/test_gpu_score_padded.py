"""GPU parity of vf_score for MLPs whose hidden layers are filled up to a multiple of 256 units."""
import numpy as np
import pytest

from paper_2011_14486_amd import inputs as I
from tests.util import TOL, check_argmin, score_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vf():
    import paper_2011_14486_amd as pkg
    return pkg.load()


def score(vf, dims, w, raw, group=0):
    import torch
    ctx = vf.vf_create(0)
    vf.vf_set_model(ctx, I.model_record(I.MLP, dims, I.BF16), w)
    s, bi, bv = vf.vf_score(ctx, torch.from_numpy(raw).cuda(), vf.VF_X_RAW_I32, group=group)
    s, bi, bv = s.cpu().numpy(), bi.cpu().numpy(), bv.cpu().numpy()
    vf.vf_destroy(ctx)
    return s, bi, bv


# one, two and four row tiles per wave; a filled-up layer in front of a full one and behind it; the widest
# input of the smallest form; eight times the products and just above (the kernel for any width)
@pytest.mark.parametrize("dims", [[256, 256, 128, 1], [64, 32, 256, 1], [512, 160, 224, 1], [256, 288, 1], [192, 512, 480, 32, 1],
                                  [256, 544, 1024, 1], [64, 992, 1024, 1], [1024, 608, 1], [64, 160, 96, 1], [64, 288, 32, 1],
                                  [96, 256, 1], [1024, 256, 1]])
@pytest.mark.parametrize("M,group", [(1, 0), (64, 0), (200, 128), (1025, 0)])
def test_widths(vf, ovf, dims, M, group):
    rng = np.random.default_rng(dims + [M])
    raw = np.floor(2.0 ** (rng.random((dims[0], M)) * 20)).astype(np.int32)
    w, model = I.mlp_weights(dims, 3, bias_std=0.1), I.model_record(I.MLP, dims, I.BF16)
    s, bi, bv = score(vf, dims, w, raw, group)
    ref = ovf.score_mlp(model, w, raw)
    assert score_err(s, ref) <= TOL[1]
    g = group or M
    for k in range(len(bi)):
        check_argmin(int(bi[k]), float(bv[k]), ref[k * g:(k + 1) * g], None, TOL[1], k * g)
        assert bv[k] == s[k * g:(k + 1) * g].min()


def test_infinite_activations_and_sizes(vf, ovf):
    """An infinite hidden value meets the zero weights of the units that fill the next layer up: they stay 0.
    Scores do not depend on the size of the call (tiles of 64, and of 128 above 64 * 65536 vectors)."""
    import torch
    dims, M = [64, 160, 96, 1], 64 * 65536 + 7
    w, model = I.mlp_weights(dims, 3, bias_std=0.1), I.model_record(I.MLP, dims, I.BF16)
    inf = w.copy()
    inf[64 * 160 + 5] = np.inf                                # bias of hidden unit 5
    raw = np.arange(64 * 300, dtype=np.int32).reshape(64, 300)
    s, _, _ = score(vf, dims, inf, raw)
    ref = ovf.score_mlp(model, inf, raw)
    assert not np.isfinite(ref).all() and score_err(s, ref) <= TOL[1]
    ctx = vf.vf_create(0)
    vf.vf_set_model(ctx, model, w)
    x = torch.randint(0, 1 << 20, (64, M), dtype=torch.int32, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))
    s, bi, bv = vf.vf_score(ctx, x, vf.VF_X_RAW_I32)
    tail, _, _ = vf.vf_score(ctx, x[:, -1000:].contiguous(), vf.VF_X_RAW_I32)
    assert torch.equal(s[-1000:], tail) and float(bv[0]) == float(s.min())
    vf.vf_destroy(ctx)
