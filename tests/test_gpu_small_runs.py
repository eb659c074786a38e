"""GPU: vf_score of small networks, whose sub-tiles are dealt out to the XCDs in runs."""
import numpy as np
import pytest

from paper_2011_14486_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vf():
    import paper_2011_14486_amd as pkg
    return pkg.load()


# 7, 8 and 9 sub-tiles (runs from eight workgroups on, where their number divides), one per compute unit and one
# more, one per wave, the first size with two columns per lane, odd sizes with several rounds of waves, sub-tiles in
# groups (more than 32768 of them)
@pytest.mark.parametrize("M", [224, 256, 288, 8192, 8193, 65536, 65537, 131073, 200003, 2097217])
@pytest.mark.parametrize("dims,dtype", [([64, 128, 128, 1], I.BF16), ([64, 32, 1], I.BF16), ([64, 128, 128, 1], I.FP32)])
def test_sizes(vf, M, dims, dtype):
    """Every score is the one that the same vector has in a call of fewer vectors (two parts, the second of which
    begins at an odd column, and calls of 48), and the minima are those of the scores."""
    import torch
    w = I.mlp_weights(dims, 3, bias_std=0.1)
    ctx = vf.vf_create(0)
    vf.vf_set_model(ctx, I.model_record(I.MLP, dims, dtype), w)
    x = torch.randint(0, 1 << 20, (dims[0], M), dtype=torch.int32, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(M))
    s, bi, bv = vf.vf_score(ctx, x, vf.VF_X_RAW_I32)
    first = int(torch.nonzero(s == s.min())[0])
    assert int(bi[0]) == first and float(bv[0]) == float(s.min())
    half = M // 2 | 1
    for lo, hi in [(0, half), (half, M)] + [(k, min(k + 48, M)) for k in {0, 31, M // 3, M - 48}]:
        part, _, _ = vf.vf_score(ctx, x[:, lo:hi].contiguous(), vf.VF_X_RAW_I32)
        assert torch.equal(part, s[lo:hi])
    group = max(M // 640, 1) * 128
    _, gi, gv = vf.vf_score(ctx, x, vf.VF_X_RAW_I32, group=group)
    sn = s.cpu().numpy()
    for k in range(len(gi)):
        of = sn[k * group:(k + 1) * group]
        assert int(gi[k]) - k * group == int(np.argmin(of)) and float(gv[k]) == of.min()
    vf.vf_destroy(ctx)
