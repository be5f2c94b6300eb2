"""Eq. (1) on W1 itself, pruned as it is read (unpacked weights, K <= 448): bit for bit what it gives on the packed weight that the same launch writes for later calls."""
import pytest
import torch

import paper_2602_06183_amd as sffn
from tests.util import to_dev
from workload import make_ffn_inputs

pytestmark = pytest.mark.gpu


def inputs(T, D, F, seed):
    """W1 with groups of four that hold equal magnitudes of either sign, zeros and subnormals."""
    X, W1, W2, b1, dY = (to_dev(make_ffn_inputs(T, D, F, seed=seed)[k]) for k in ("X", "W1", "W2", "b1", "dY"))
    W1[: F // 4] = (W1[: F // 4] * 50).round() / 64
    W1[F // 4: F // 4 + 3, ::2] = 0
    W1[F // 4 + 3: F // 4 + 6] *= 1e-37
    return X, W1, W2, b1, dY


@pytest.mark.parametrize("mode", [sffn.MODE_HARD, sffn.MODE_SOFT])
@pytest.mark.parametrize("T,D,F,M", [(64, 64, 128, 8), (192, 128, 896, 8), (320, 192, 320, 8), (512, 256, 1024, 8), (64, 256, 192, 8), (192, 320, 576, 8), (128, 384, 512, 8), (64, 448, 1600, 8), (192, 192, 512, 16), (256, 256, 1024, 32), (64, 448, 512, 16)])
def test_step(T, D, F, M, mode):
    x = inputs(T, D, F, 71)
    step = sffn.FfnStep(T, D, F, mode, M=M)
    first = [t.clone() for t in step(*x)]
    saved = {k: v.clone() for k, v in step.saved().items()}
    vals, meta = sffn.prune24_compress(x[1], mode=mode)
    assert torch.equal(saved["w1_vals"].view(torch.int16), vals.view(torch.int16)) and torch.equal(saved["w1_meta"], meta)
    again = step(*x, weights_packed=True)
    for a, b in zip(first, again):
        assert torch.equal(a, b)
    for k, v in step.saved().items():
        assert torch.equal(saved[k].view(torch.uint8), v.view(torch.uint8)), k
    halves = sffn.FfnStep(T, D, F, mode, M=M, lean=True)
    assert torch.equal(halves.forward(*x[:4]), first[0]) and torch.equal(halves.forward(*x[:4], weights_packed=True), first[0])
    for a, b in zip(first[1:], halves.backward(x[1], x[4])):
        assert torch.equal(a, b)


@pytest.mark.parametrize("M,D", [(8, 192), (16, 192), (8, 320)])
def test_experts(M, D):
    seg, F = [0, 64, 64, 256, 384], 256
    per = [inputs(seg[-1], D, F, 72 + e) for e in range(4)]
    X, dY = per[0][0], per[0][4]
    W1, W2, b1 = (torch.stack([p[i] for p in per]) for i in (1, 2, 3))
    step = sffn.FfnStepGrouped(seg, D, F, lean=True, M=M)
    first = [t.clone() for t in step(X, W1, W2, b1, dY)]
    for a, b in zip(first, step(X, W1, W2, b1, dY, weights_packed=True)):
        assert torch.equal(a, b)
    for e, (a, b) in enumerate(zip(seg, seg[1:])):
        if a < b:
            assert torch.equal(first[0][a:b], sffn.FfnStep(b - a, D, F, lean=True, M=M)(X[a:b].contiguous(), W1[e], W2[e], b1[e], dY[a:b].contiguous())[0])
