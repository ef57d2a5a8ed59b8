"""Non-finite inputs of the split weight gradient (needs a GPU): an Inf or NaN
reaches the taps that it reaches in the unsplit kernel, and no others."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# images that end inside a tile in both directions, in one direction, and whole tiles
@pytest.mark.parametrize("H,Wd,dil", [(5, 33, 1), (9, 70, 4), (8, 37, 2), (6, 64, 1), (8, 64, 2)])
def test_nonfinite_pixels_at_the_image_edge(H, Wd, dil):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_31347_amd import warmstart as W
    B, Cin, Cout = 8, 7, 32
    rng = np.random.default_rng(H)
    x = rng.standard_normal((B, Cin, H, Wd)).astype(np.float32)
    dz = rng.standard_normal((B, Cout, H, Wd)).astype(np.float32)
    x[0, 1, 0, Wd - 1] = np.inf
    x[1, 3, H - 1, 2] = np.nan
    x[1, 5, H - 1, Wd - 1] = -np.inf
    xg, dzg = W.to_bf16(torch.from_numpy(x).cuda()), torch.from_numpy(dz).cuda()
    n = W._L.slbm_conv3x3_backward_weight_workspace(B, Cin, H, Wd, dil)
    assert n > 0
    out = []
    for nbytes in (0, n):                               # unsplit, split
        ws = torch.empty(max(nbytes, 1), dtype=torch.uint8, device="cuda")
        gw = torch.zeros((Cout, Cin * 9), dtype=torch.float32, device="cuda")
        gb = torch.zeros(Cout, dtype=torch.float32, device="cuda")
        W._chk(W._L.slbm_conv3x3_backward_weight_ws(W._p(dzg), W._p(xg), W._p(gw), W._p(gb), B, Cin, Cout, H, Wd,
                                                    dil, W._p(ws), nbytes, W._stream()), "bww")
        out.append((gw.cpu().numpy(), gb.cpu().numpy()))
    (a, ab), (b, bb) = out
    ok = np.isfinite(a)
    assert ok.any() and not ok.all()
    assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isinf(a), np.isinf(b))
    # FP32 sums of at most 2^13 terms of random sign in two orders, against the largest element
    assert np.abs(a[ok] - b[ok]).max() <= 1e-5 * np.abs(a[ok]).max()
    assert np.abs(ab - bb).max() <= 1e-5 * np.abs(ab).max()
