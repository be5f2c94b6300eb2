"""Y3 and dX of 16 MiB and more leave past the caches: the same bits as those of a step on the first tokens, which do not."""
import pytest
import torch

import paper_2602_06183_amd as sffn

pytestmark = pytest.mark.gpu

T, FEW, D = 4160, 2048, 2112          # 16.8 and 8.3 MiB; remainders on tiles of 512, 256 and 128 tokens and of 256 and 128 columns
STEPS = [(0, 8, D, 1536), (0, 8, D, 4096), (0, 16, D, 2048), (0, 32, D, 2048), (0, 64, D, 2048), (1, 8, 2176, 2048), (1, 16, 2176, 2048)]       # fp8, M, d_model, d_ff


@pytest.mark.parametrize("fp8,M,D,F", STEPS)
def test_results(fp8, M, D, F):
    gen = torch.Generator(device="cuda").manual_seed(79)
    rand = lambda scale, *shape: (torch.randn(shape, device="cuda", generator=gen) * scale).to(torch.bfloat16)  # noqa: E731
    X, dY, W1, W2 = rand(1, T, D), rand(1, T, D), rand(0.02, F, D), rand(0.02, D, F)
    b1 = torch.randn((F,), device="cuda", generator=gen) * 0.1
    scales = dict(x=0.012, w1=2e-4, w2=2e-4, y2=0.05, dy=0.012, dy1=0.05)
    make = lambda n: sffn.FfnStepFp8(n, D, F, scales, wgrad_fp8=True, lean=True, M=M) if fp8 else sffn.FfnStep(n, D, F, lean=True, M=M)  # noqa: E731
    Y3, dX = make(T)(X, W1, W2, b1, dY)[:2]
    few = make(FEW)(X[:FEW].contiguous(), W1, W2, b1, dY[:FEW].contiguous())
    last = make(T - FEW)(X[FEW:].contiguous(), W1, W2, b1, dY[FEW:].contiguous())
    assert float(Y3.float().abs().max()) > 0 and float(dX.float().abs().max()) > 0
    for whole, a, b in ((Y3, few[0], last[0]), (dX, few[1], last[1])):
        assert torch.equal(whole[:FEW], a) and torch.equal(whole[FEW:], b)
