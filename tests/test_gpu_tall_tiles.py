"""Shared launches with contractions on 256 x 128 tiles, remainders in every dimension: against the same contractions as separate operations, or the oracle."""
import pytest
import torch

import paper_2602_06183_amd as sffn
from tests.test_gpu_fp8 import _check_fp8_step_against_oracle, _fp8_step_scales
from tests.util import to_bits, to_dev
from workload import make_ffn_inputs

pytestmark = pytest.mark.gpu

# T, D, F; bits 0, 1, 2: eqs. (3) / (7), (5) / (8), (4) on tall tiles in the launches of eqs. (3), (5), (4), of (5), (4) and of (7), (8)
PLAIN = [
    (1664, 960, 832, (1, 0, 1)),
    (1152, 1088, 3072, (3, 0, 2)),
    (1472, 1408, 2880, (3, 2, 3)),
    (1728, 1280, 4224, (7, 6, 3)),
    (1728, 1088, 4160, (7, 6, 0)),
    (3328, 512, 1344, (1, 0, 1)),       # beside 64 tiles of eq. (8)
    (128, 1472, 3136, (2, 2, 2)),       # beside 64 tiles of eqs. (3), (7), which sum in another order
    (768, 1536, 1984, (3, 2, 0)),
]
WIDE = [(16, 1472, 1536, 3840, (6, 6, 0)), (32, 1600, 1472, 5120, (6, 6, 2)), (64, 128, 1024, 4096, (2, 2, 0))]
FP8 = [(8, 1344, 1408, 3968, (7, 6, 3)), (16, 896, 1024, 6144, (6, 6, 2))]


def same(a, b):
    """The same bits, or (64 tiles, alone or in the step, sum in another order) as many elements a last place of bf16 apart as float32 sums put there: 2e-4 of the whole where it was measured; a
    wrong row of the largest of these outputs would be 1.5e-2."""
    return torch.equal(a, b) or float((a.float() - b.float()).norm()) <= 1e-3 * float(b.float().norm())


@pytest.mark.parametrize("T,D,F,forms", PLAIN)
def test_step(T, D, F, forms):
    """The step in one call, its two calls with float32 sums of the weight gradients, and its contractions one by one."""
    inp = make_ffn_inputs(T, D, F, seed=61)
    X, W1, W2, b1, dY = (to_dev(inp[k]) for k in ("X", "W1", "W2", "b1", "dY"))
    step = sffn.FfnStep(T, D, F, sffn.MODE_SOFT)
    Y3, dX, dW1, dW2 = step(X, W1, W2, b1, dY)
    s = step.saved()
    y2, dy1 = [s[k] for k in ("y2_vals", "y2_meta", "colidx")], [s[k] for k in ("dy1_vals", "y2_meta", "colidx")]
    y1 = sffn.spmm24_fwd(X, s["w1_vals"], s["w1_meta"], b1)
    for got, want in zip(y2, sffn.sqrelu_vnm_compress(y1)):
        assert torch.equal(got, want)
    assert torch.equal(dy1[0], sffn.dsqrelu_vnm(sffn.spmm24_dgrad(dY, s["w2t_vals"], s["w2t_meta"]), y1, *y2[1:]))
    assert same(Y3, sffn.vnm_spmm(*y2, W2, 0)) and same(dX, sffn.vnm_spmm(*dy1, W1, 1))
    assert same(dW2, sffn.vnm_wgrad(*y2, dY, False)) and same(dW1, sffn.vnm_wgrad(*dy1, X, True))
    two = sffn.FfnStep(T, D, F, sffn.MODE_SOFT, lean=True, dw_fp32=True)
    assert same(two.forward(X, W1, W2, b1), Y3)
    assert torch.equal(two.backward(W1, dY)[0], dX)
    assert torch.equal(two.dW1.to(torch.bfloat16), dW1) and torch.equal(two.dW2.to(torch.bfloat16), dW2)


# T, D, F whose epilogues store past the caches, on tiles of 64, 128, 256
STREAMED = [(64, 8192, 8128), (704, 5760, 10944), (1344, 5120, 11264)]


@pytest.mark.parametrize("T,D,F", STREAMED)
def test_step_that_stores_past_the_caches(T, D, F):
    test_step(T, D, F, None)


@pytest.mark.parametrize("M,T,D,F,forms", WIDE)
def test_step_of_wide_blocks(M, T, D, F, forms):
    inp = make_ffn_inputs(T, D, F, seed=62)
    dev = [to_dev(inp[k]) for k in ("X", "W1", "W2", "b1", "dY")]
    for a, b in zip(sffn.FfnStep(T, D, F, M=M, lean=True)(*dev), sffn.FfnStep(T, D, F, M=M, unfused=True)(*dev)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("M,T,D,F,forms", FP8)
def test_step_on_codes(M, T, D, F, forms):
    inp = make_ffn_inputs(T, D, F, seed=63)
    sc = _fp8_step_scales(inp)
    dev = [to_dev(inp[k]) for k in ("X", "W1", "W2", "b1", "dY")]
    step = sffn.FfnStepFp8(T, D, F, sc, sffn.MODE_HARD, keep_dense=True, wgrad_fp8=True, M=M)
    outs = step(*dev)
    s = {k: to_bits(v) if v.dtype == torch.bfloat16 else v.cpu().numpy() for k, v in step.saved().items()}
    _check_fp8_step_against_oracle(inp, sc, s, {k: to_bits(v) for k, v in zip(("Y3", "dX", "dW1", "dW2"), outs)}, sffn.MODE_HARD, True, M)


def test_experts():
    """Experts whose segments end anywhere in their last tile, one of them empty: each one's results are those of a step on its tokens alone."""
    seg, D, F = [0, 704, 704, 1600, 2496], 1088, 3072
    inp = [make_ffn_inputs(seg[-1], D, F, seed=64 + e) for e in range(4)]
    X, dY = to_dev(inp[0]["X"]), to_dev(inp[0]["dY"])
    W1, W2, b1 = (torch.stack([to_dev(i[k]) for i in inp]) for k in ("W1", "W2", "b1"))
    step = sffn.FfnStepGrouped(seg, D, F, lean=True)
    Y3, dX, dW1, dW2 = step(X, W1, W2, b1, dY)
    for e, (a, b) in enumerate(zip(seg, seg[1:])):
        if a == b:
            assert not dW1[e].any() and not dW2[e].any()
            continue
        alone = sffn.FfnStep(b - a, D, F, lean=True)(X[a:b].contiguous(), W1[e], W2[e], b1[e], dY[a:b].contiguous())
        for got, want in ((Y3[a:b], alone[0]), (dX[a:b], alone[1]), (dW1[e], alone[2]), (dW2[e], alone[3])):
            assert same(got, want)


# fp8, T, N, F: launches of their own, on tall tiles instead of 256 or 128
ALONE_ACTIVATION = [(0, 2496, 2944, 256), (0, 1600, 3456, 960), (1, 2624, 2624, 1664), (1, 3776, 3328, 512)]
ALONE_GRADIENT = [(0, 448, 1856, 8256), (0, 704, 2624, 9408)]


def compressed(T, F, seed):
    X = to_dev(make_ffn_inputs(T, 64, 64, seed=seed)["X"])
    return X.repeat(1, F // 64) * torch.linspace(0.5, 2.0, F, device="cuda").to(torch.bfloat16)


@pytest.mark.parametrize("fp8,T,N,F", ALONE_ACTIVATION)
def test_activation_contraction_alone(fp8, T, N, F):
    """As on the tokens in three pieces, which take other tiles."""
    y1, W = compressed(T, F, 65), to_dev(make_ffn_inputs(64, N, F, seed=66)["W2"])
    if fp8:
        y2, Wq = sffn.sqrelu_vnm_compress_fp8(y1, 0.05), sffn.quantize_fp8(W, 1e-3)
        spmm = lambda *v: sffn.vnm_spmm_fp8(*v, 0.05, Wq, 1e-3, 0)  # noqa: E731
    else:
        y2 = sffn.sqrelu_vnm_compress(y1)
        spmm = lambda *v: sffn.vnm_spmm(*v, W, 0)  # noqa: E731
    whole = spmm(*y2)
    assert float(whole.float().abs().max()) > 0
    for a, b in ((0, 448), (448, 1024), (1024, T)):
        assert same(whole[a:b], spmm(*(t[a // d:b // d].contiguous() for t, d in zip(y2, (1, 1, 64)))))


@pytest.mark.parametrize("fp8,T,N,F", ALONE_GRADIENT)
@pytest.mark.parametrize("f_major", [False, True])
def test_gradient_contraction_alone(fp8, T, N, F, f_major):
    """As on the columns of the dense operand in three pieces, which take other tiles."""
    y2, G = sffn.sqrelu_vnm_compress(compressed(T, F, 67)), to_dev(make_ffn_inputs(T, N, 64, seed=68)["X"])
    whole = sffn.vnm_wgrad(*y2, G, f_major)
    assert float(whole.float().abs().max()) > 0
    for a, b in ((0, 320), (320, 1024), (1024, N)):
        piece = sffn.vnm_wgrad(*y2, G[:, a:b].contiguous(), f_major)
        assert same(whole[:, a:b] if f_major else whole[a:b], piece)
