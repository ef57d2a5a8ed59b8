"""Weight gradient split over the pixels, and the tiled forward convolution at
the edges of their tiles (needs a GPU): against the float64 reference with the
same rounding points."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# a single pixel; one tile exactly; one pixel more than a tile in each direction; several tiles per workgroup
# (300 tiles and more on 256 compute units); a dilation wider than the image; odd and single channels; 33 and 56
# input channels (16 column blocks); a dilation whose region does not fit (no workspace, the unsplit kernel)
@pytest.mark.parametrize("B,Cin,Cout,H,Wd,dil", [(1, 32, 32, 1, 1, 1), (2, 32, 32, 4, 32, 2), (2, 7, 32, 5, 33, 1),
                                                 (40, 3, 5, 13, 65, 1), (33, 32, 2, 9, 70, 8), (1, 1, 1, 39, 64, 4),
                                                 (2, 32, 32, 6, 10, 12), (2, 56, 32, 9, 40, 1), (2, 57, 32, 9, 40, 1),
                                                 (1, 32, 32, 9, 40, 30)])
def test_split_weight_gradient_and_forward(B, Cin, Cout, H, Wd, dil):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import convnet as C
    from paper_2609_31347_amd import warmstart as W
    rng = np.random.default_rng(Cin * 100 + H)
    x = rng.standard_normal((B, Cin, H, Wd)).astype(np.float32)
    dz = rng.standard_normal((B, Cout, H, Wd)).astype(np.float32)
    xg, dzg = W.to_bf16(torch.from_numpy(x).cuda()), torch.from_numpy(dz).cuda()
    n = W._L.slbm_conv3x3_backward_weight_workspace(B, Cin, H, Wd, dil)
    assert (n > 0) == (Cin <= 56 and dil < 30)
    # FP32 sums of at most 2^15 terms of random sign, a lane adding at most 2^12 of them in a row:
    # sqrt(2^12) 2^-24 of the root-sum-square, against a largest element of several root-sum-squares
    tol = 1e-5
    # the reference wants images larger than the dilation: the same images with a zero rim
    rim = ((0, 0), (0, 0), (0, dil), (0, dil))
    xr = np.pad(C.bf16(x), rim)
    rw, rb = C.conv3x3_grad_w(np.pad(dz, rim), xr, dil)
    for nbytes in {n, 0}:
        ws = torch.empty(max(nbytes, 1), dtype=torch.uint8, device="cuda")
        gw = torch.full((Cout, Cin * 9), float("nan"), dtype=torch.float32, device="cuda")
        gb = torch.full((Cout,), float("nan"), dtype=torch.float32, device="cuda")
        out = []
        for _ in range(2):
            W._chk(W._L.slbm_conv3x3_backward_weight_ws(W._p(dzg), W._p(xg), W._p(gw), W._p(gb), B, Cin, Cout, H, Wd,
                                                        dil, W._p(ws), nbytes, W._stream()), "bww")
            out.append((gw.clone(), gb.clone()))
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])      # deterministic
        assert np.abs(gw.cpu().numpy().reshape(rw.shape) - rw).max() <= tol * np.abs(rw).max()
        assert np.abs(gb.cpu().numpy() - rb).max() <= tol * np.abs(rb).max()
    if Cin > 32:
        return
    w = (rng.standard_normal((Cout, Cin, 3, 3)) * 0.3).astype(np.float32)
    w32 = torch.from_numpy(w.reshape(Cout, Cin * 9)).cuda()
    k = 32 * W._kp(Cin * 9)
    store = torch.zeros(k + 1, dtype=torch.bfloat16, device="cuda")
    for wp in (store[:k], store[1:]):                   # 16-byte aligned weights and misaligned ones
        W._chk(W._L.slbm_pack_weights(W._p(w32), W._p(wp), None, Cin, Cout, W._stream()), "pack")
        y = torch.empty((B, Cout, H, Wd), dtype=torch.float32, device="cuda")
        W._chk(W._L.slbm_conv3x3_forward(W._p(xg), W._p(wp), None, W._p(y), None, B, Cin, Cout, H, Wd, 0, dil,
                                         W._stream()), "fwd")
        ref = C.conv3x3(xr, C.bf16(w), np.zeros(Cout, np.float32), dil)[:, :, :H, :Wd]
        # 9 Cin products in FP32: 288 x 2^-24 of the sum of absolute terms
        assert np.abs(y.cpu().numpy() - ref).max() <= 1e-5 * np.abs(ref).max()
