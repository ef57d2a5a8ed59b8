"""The two forms of the forward convolution (needs a GPU): from a staged region
and from memory, at sizes on both sides of the line between them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# from memory: more tiles than run at once and regions of many times the pixels (columns, wide dilation), the last 128
# pixels of an image cut short, a single pixel; staged: the same layers with fewer images
@pytest.mark.parametrize("B,Cin,Cout,H,Wd,dil", [(70, 32, 32, 65, 1, 1), (2, 32, 32, 65, 1, 1), (300, 5, 2, 37, 3, 4),
                                                 (40, 32, 32, 10, 64, 8), (25, 32, 32, 10, 64, 8),
                                                 (600, 3, 7, 1, 1, 1), (2100, 9, 32, 3, 3, 1)])
def test_both_forms_match_the_reference(B, Cin, Cout, H, Wd, dil):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import convnet as C
    from paper_2609_31347_amd import warmstart as W
    rng = np.random.default_rng(B)
    x = rng.standard_normal((B, Cin, H, Wd)).astype(np.float32)
    w = (rng.standard_normal((Cout, Cin, 3, 3)) * 0.3).astype(np.float32)
    b = rng.standard_normal(Cout).astype(np.float32)
    xg, bg = W.to_bf16(torch.from_numpy(x).cuda()), torch.from_numpy(b).cuda()
    w32 = torch.from_numpy(w.reshape(Cout, Cin * 9)).cuda()
    wp = torch.zeros(32 * W._kp(Cin * 9), dtype=torch.bfloat16, device="cuda")
    W._chk(W._L.slbm_pack_weights(W._p(w32), W._p(wp), None, Cin, Cout, W._stream()), "pack")
    y = torch.full((B, Cout, H, Wd), float("nan"), dtype=torch.float32, device="cuda")
    W._chk(W._L.slbm_conv3x3_forward(W._p(xg), W._p(wp), W._p(bg), W._p(y), None, B, Cin, Cout, H, Wd, 0, dil,
                                     W._stream()), "fwd")
    # the reference wants images larger than the dilation: the same images with a zero rim
    xr = np.pad(C.bf16(x), ((0, 0), (0, 0), (0, dil), (0, dil)))
    ref = C.conv3x3(xr, C.bf16(w), b, dil)[:, :, :H, :Wd]
    # 9 Cin products in FP32: 288 x 2^-24 of the sum of absolute terms
    assert np.abs(y.cpu().numpy() - ref).max() <= 1e-5 * np.abs(ref).max()

