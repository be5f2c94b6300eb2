"""Tall tiles add the same products in the same order as tiles of 128 and 256: every result to the bit, where no 64 tile (which sums in another order) is on either side."""
import pytest
import torch

import paper_2602_06183_amd as sffn

pytestmark = pytest.mark.gpu

# T, D, F, segments of experts; forms of the launches of eqs. (3), (5), (4), of (5), (4) and of (7), (8), then of the last two with float32 sums (None: launches of their own, the gradients' on tall tiles)
EXACT = [
    (1920, 1920, 5632, None, (7, 6, 3, 6, 3)),
    (1728, 1856, 4928, None, (3, 2, 3, 2, 1)),
    (1984, 1600, 5248, None, (1, 2, 1, 2, 1)),
    (2304, 1664, 5312, [0, 1344, 2304, 2304, 2304], (7, 6, 3, 6, 3)),
    (1920, 1280, 4096, [0, 0, 832, 832, 1920], (3, 6, 3, 6, 3)),
    (3648, 1216, 2944, [0, 1472, 2432, 3648], (7, 2, 3, 2, 3)),
    (4928, 1920, 5248, [0, 1536, 2816, 3648, 4928], (None,) * 5),
]


@pytest.mark.parametrize("T,D,F,seg,forms", EXACT)
def test_every_result_to_the_bit(T, D, F, seg, forms):
    gen = torch.Generator(device="cuda").manual_seed(73)
    lead = (len(seg) - 1,) if seg else ()
    rand = lambda scale, *shape: (torch.randn(shape, device="cuda", generator=gen) * scale).to(torch.bfloat16)  # noqa: E731
    X, dY, W1, W2 = rand(1, T, D), rand(1, T, D), rand(0.02, *lead, F, D), rand(0.02, *lead, D, F)
    b1 = torch.randn((*lead, F), device="cuda", generator=gen) * 0.1
    make = lambda **kw: sffn.FfnStepGrouped(seg, D, F, sffn.MODE_SOFT, **kw) if seg else sffn.FfnStep(T, D, F, sffn.MODE_SOFT, **kw)  # noqa: E731
    step = make()
    Y3, dX, dW1, dW2 = step(X, W1, W2, b1, dY)
    two = make(lean=True, dw_fp32=True)
    two.dW1.zero_(), two.dW2.zero_()
    assert torch.equal(two.forward(X, W1, W2, b1), Y3) and torch.equal(two.backward(W1, dY)[0], dX)
    assert torch.equal(two.dW1.to(torch.bfloat16), dW1) and torch.equal(two.dW2.to(torch.bfloat16), dW2)
    if not seg:
        s = step.saved()
        y2, dy1 = [s[k] for k in ("y2_vals", "y2_meta", "colidx")], [s[k] for k in ("dy1_vals", "y2_meta", "colidx")]
        y1 = sffn.spmm24_fwd(X, s["w1_vals"], s["w1_meta"], b1)
        assert all(torch.equal(a, b) for a, b in zip(y2, sffn.sqrelu_vnm_compress(y1)))
        assert torch.equal(dy1[0], sffn.dsqrelu_vnm(sffn.spmm24_dgrad(dY, s["w2t_vals"], s["w2t_meta"]), y1, *y2[1:]))
        assert torch.equal(Y3, sffn.vnm_spmm(*y2, W2, 0)) and torch.equal(dX, sffn.vnm_spmm(*dy1, W1, 1))
        assert torch.equal(dW2, sffn.vnm_wgrad(*y2, dY, False)) and torch.equal(dW1, sffn.vnm_wgrad(*dy1, X, True))
        return
    for e, (a, b) in enumerate(zip(seg, seg[1:])):
        if a == b:
            assert not dW1[e].any() and not dW2[e].any()
            continue
        alone = sffn.FfnStep(b - a, D, F, sffn.MODE_SOFT, lean=True)(X[a:b].contiguous(), W1[e], W2[e], b1[e], dY[a:b].contiguous())
        for got, want in zip((Y3[a:b], dX[a:b], dW1[e], dW2[e]), alone):
            assert torch.equal(got, want)
