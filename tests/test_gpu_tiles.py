"""The tile sizes of the contractions at sizes where each is chosen (256 x 256, 128 x 128, and 64 x 64 with the contraction split over the tile's
wavefronts), with remainders in every dimension; stage by stage against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_06183_amd as sffn
from tests.test_gpu_full_size import sampled_router_step_check
from tests.test_gpu_fp8 import _check_fp8_step_against_oracle, _fp8_step_scales
from tests.test_gpu_kernels import _check_wide_step_against_oracle, _teacher_forced_step_check
from tests.util import assert_gemm_close, to_bits, to_dev
from workload import bf16_bits_from_f32, make_ffn_inputs, make_router_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,D,F", [
    (64, 1088, 2112),       # few tiles, long contractions: 64 tiles in eqs. (1), (3), (7), trip counts that four wavefronts do not share evenly
    (832, 320, 576),        # 64 tiles in the weight gradients (13 token blocks)
    (1088, 1152, 4160),     # 128 tiles with a half-empty last row and column
    (2112, 2112, 4160),     # 256 tiles in eq. (1), shared launches of 128 tiles behind it
])
def test_step_on_every_tile_size(T, D, F):
    _teacher_forced_step_check(T, D, F, sffn.MODE_SOFT, seed=21)


@pytest.mark.parametrize("M,T,D,F", [(16, 64, 1088, 2048), (64, 64, 1088, 3072), (64, 832, 320, 2048), (32, 832, 320, 1024)])
def test_wide_step_on_small_tiles(M, T, D, F):
    inp = make_ffn_inputs(T, D, F, seed=22)
    dev = {k: to_dev(v) for k, v in inp.items()}
    (Y3, dX, dW1, dW2), step = sffn.ffn_sparse_step(dev["X"], dev["W1"], dev["W2"], dev["b1"], dev["dY"], sffn.MODE_HARD, M=M)
    s = {k: to_bits(v) for k, v in step.saved().items()}
    _check_wide_step_against_oracle(inp, s, dict(Y3=to_bits(Y3), dX=to_bits(dX), dW1=to_bits(dW1), dW2=to_bits(dW2)), sffn.MODE_HARD, M)


@pytest.mark.parametrize("M,T,D,F", [(8, 64, 2304, 1152), (8, 832, 384, 640), (8, 832, 384, 1664), (64, 64, 2304, 2048), (16, 832, 384, 1024)])
def test_fp8_step_on_small_tiles(M, T, D, F):
    inp = make_ffn_inputs(T, D, F, seed=23)
    sc = _fp8_step_scales(inp)
    dev = {k: to_dev(v) for k, v in inp.items()}
    step = sffn.FfnStepFp8(T, D, F, sc, sffn.MODE_HARD, keep_dense=True, wgrad_fp8=True, M=M)
    outs = step(dev["X"], dev["W1"], dev["W2"], dev["b1"], dev["dY"])
    torch.cuda.synchronize()
    s = {k: to_bits(v) if v.dtype == torch.bfloat16 else v.cpu().numpy() for k, v in step.saved().items()}
    _check_fp8_step_against_oracle(inp, sc, s, {k: to_bits(v) for k, v in zip(("Y3", "dX", "dW1", "dW2"), outs)}, sffn.MODE_HARD, True, M)


@pytest.mark.parametrize("M,T,D,F", [
    (32, 2112, 1088, 6656),     # kept rows only (the outputs fill the chip): a half-empty last tile in both dimensions, 33 token blocks
    (64, 2048, 1344, 7168),
    (64, 768, 1344, 7168),
    (64, 320, 1344, 7168),      # the fewest tokens of this form
])
def test_wide_weight_gradients_on_kept_rows(M, T, D, F):
    """Eqs. (5), (8) on the kept rows only: the same bits as the unfused path, which multiplies the rows of zeros too, in bf16 and as float32
    accumulators."""
    inp = make_ffn_inputs(T, D, F, seed=24)
    dev = [to_dev(inp[k]) for k in ("X", "W1", "W2", "b1", "dY")]
    plain = [t.clone() for t in sffn.FfnStep(T, D, F, M=M, lean=True)(*dev)]
    for a, b in zip(plain, sffn.FfnStep(T, D, F, M=M, unfused=True)(*dev)):
        assert torch.equal(a, b)
    acc = sffn.FfnStep(T, D, F, M=M, lean=True, dw_fp32=True)
    acc(*dev)
    assert torch.equal(acc.dW1.to(torch.bfloat16), plain[2]) and torch.equal(acc.dW2.to(torch.bfloat16), plain[3])


@pytest.mark.parametrize("M", [32, 64])
def test_wide_weight_gradients_of_experts_on_kept_rows(M):
    """Experts with 1, 0, 24 and 23 token blocks: each one's weight gradients are those of a step on its tokens alone (bit for bit, except where
    64 tokens alone are contracted by several wavefronts)."""
    seg, D, F = [0, 64, 64, 1600, 3072], 1344, 7168
    inp = [make_ffn_inputs(seg[-1], D, F, seed=25 + e) for e in range(4)]
    X, dY = to_dev(inp[0]["X"]), to_dev(inp[0]["dY"])
    W1, W2, b1 = (torch.stack([to_dev(i[k]) for i in inp]) for k in ("W1", "W2", "b1"))
    step = sffn.FfnStepGrouped(seg, D, F, M=M, lean=True)
    step(X, W1, W2, b1, dY)
    for e, (a, b) in enumerate(zip(seg, seg[1:])):
        if a == b:
            assert not step.dW1[e].any() and not step.dW2[e].any()
            continue
        alone = sffn.FfnStep(b - a, D, F, M=M, unfused=True)(X[a:b].contiguous(), W1[e], W2[e], b1[e], dY[a:b].contiguous())
        for got, want in ((step.dW1[e], alone[2]), (step.dW2[e], alone[3])):
            assert torch.equal(got, want) or (b - a == 64 and (got.float() - want.float()).norm() < 2e-2 * want.float().norm())


@pytest.mark.parametrize("M,T,N,F", [
    (8, 64, 64, 64), (8, 192, 320, 832), (16, 128, 192, 320), (32, 832, 64, 320), (64, 64, 64, 128),      # compacted rows: edges of the 256-unit pieces
    (32, 768, 128, 768), (64, 832, 64, 1536),                                                             # kept rows only: half-empty last pieces
])
def test_standalone_weight_gradients(M, T, N, F):
    rng = np.random.default_rng(31)
    y1 = bf16_bits_from_f32(rng.standard_normal((T, F)).astype(np.float32))
    G = bf16_bits_from_f32(rng.standard_normal((T, N)).astype(np.float32))
    a = sffn.sqrelu_vnm_compress(to_dev(y1), 64, M)
    bits = [to_bits(t) for t in a]
    for f_major in (0, 1):
        assert_gemm_close(to_bits(sffn.vnm_wgrad(*a, to_dev(G), f_major, 64, M)), oracle.vnm_wgrad(*bits, G, f_major, 64, M), "wgrad")
    if M == 8:
        W = bf16_bits_from_f32(rng.standard_normal((N, F)).astype(np.float32))
        assert_gemm_close(to_bits(sffn.vnm_spmm(*a, to_dev(W), 0, 64, M)), oracle.vnm_spmm(*bits, W, 0, 64, M), "spmm")


@pytest.mark.parametrize("T,M", [(1023, 8), (1024, 64), (1025, 16), (32768, 32), (32769, 32)])
def test_grouping_at_the_edges_of_its_blocks(T, M):
    inp = make_router_inputs(T, 64, 256, M, seed=T)
    r = sffn.venom_route(to_dev(inp["X"]), to_dev(inp["means"]), M)
    perm, seg = oracle.expert_permutation(to_bits(r["expert"]), M // 4)
    assert r["seg"] == [int(v) for v in seg] and np.array_equal(to_bits(r["perm"]), perm)
    assert np.array_equal(perm[to_bits(r["row_of_token"])], np.arange(T))


@pytest.mark.parametrize("M,T,D,F", [
    (8, 64, 3968, 8192),
    (8, 192, 2048, 8256),       # several token blocks; 129 stages (the step shares launches, so that only the stand-alone call is split)
    (8, 128, 576, 13120),       # two token blocks, 11 workgroups a tile, which do not share 205 stages evenly
    (16, 64, 3968, 8192),       # gathered rows
    (16, 128, 576, 13312),
])
def test_split_activation_contractions(M, T, D, F):
    """Eqs. (3), (7) shared by several workgroups per tile: twice in a row (the counters are left as they were found), alone and in the step."""
    inp = make_ffn_inputs(T, D, F, seed=33)
    dev = [to_dev(inp[k]) for k in ("X", "W1", "W2", "b1", "dY")]
    step = sffn.FfnStep(T, D, F, M=M)
    first = [t.clone() for t in step(*dev)]
    for a, b in zip(first, step(*dev)):
        assert torch.equal(a, b)
    y2 = [to_bits(step.saved()[k]) for k in ("y2_vals", "y2_meta", "colidx")]
    assert_gemm_close(to_bits(first[0]), oracle.vnm_spmm(*y2, inp["W2"], 0, 64, M), "y3")
    assert_gemm_close(to_bits(first[1]), oracle.vnm_spmm(to_bits(step.saved()["dy1_vals"]), *y2[1:], inp["W1"], 1, 64, M), "dX")
    alone = sffn.vnm_spmm(*[step.saved()[k] for k in ("y2_vals", "y2_meta", "colidx")], dev[2], 0, 64, M)
    assert_gemm_close(to_bits(alone), to_bits(first[0]), "y3 alone")


@pytest.mark.parametrize("M,T,N,F", [(8, 64, 192, 16384), (8, 512, 1024, 16384), (16, 64, 64, 65536)])
def test_most_splits_and_most_tiles(M, T, N, F):
    """16 workgroups a tile; 128 tiles, whose counters share lines.  Over and over: every call finds its counters as it needs them."""
    rng = np.random.default_rng(36)
    y1 = bf16_bits_from_f32(rng.standard_normal((T, F)).astype(np.float32))
    W = bf16_bits_from_f32(rng.standard_normal((N, F)).astype(np.float32) * np.float32(0.02))
    a = sffn.sqrelu_vnm_compress(to_dev(y1), 64, M)
    first = sffn.vnm_spmm(*a, to_dev(W), 0, 64, M)
    assert_gemm_close(to_bits(first), oracle.vnm_spmm(*[to_bits(t) for t in a], W, 0, 64, M), "spmm")
    for _ in range(20):
        assert torch.equal(first, sffn.vnm_spmm(*a, to_dev(W), 0, 64, M))


@pytest.mark.parametrize("wgrad_fp8,dw_fp32", [(False, False), (True, True)])
def test_split_activation_contractions_of_the_fp8_step(wgrad_fp8, dw_fp32):
    """The same on codes, in the steps that do not share launches: against the oracle, and twice in a row."""
    T, D, F = 64, 1024, 8192
    inp = make_ffn_inputs(T, D, F, seed=34)
    sc = _fp8_step_scales(inp)
    dev = [to_dev(inp[k]) for k in ("X", "W1", "W2", "b1", "dY")]
    step = sffn.FfnStepFp8(T, D, F, sc, sffn.MODE_HARD, keep_dense=True, wgrad_fp8=wgrad_fp8, dw_fp32=dw_fp32)
    first = [t.clone() for t in step(*dev)]
    s = {k: to_bits(v) if v.dtype == torch.bfloat16 else v.cpu().numpy() for k, v in step.saved().items()}
    outs = {k: to_bits(v.to(torch.bfloat16)) for k, v in zip(("Y3", "dX", "dW1", "dW2"), first)}
    _check_fp8_step_against_oracle(inp, sc, s, outs, sffn.MODE_HARD, wgrad_fp8, 8)
    second = step(*dev)
    assert torch.equal(first[0], second[0]) and torch.equal(first[1], second[1])


@pytest.mark.parametrize("fp8,M,D,F,seg", [
    (False, 8, 2240, 9664, [0, 128, 128, 448, 640]),         # shared launches
    (False, 8, 2240, 9664, [0, 512, 512, 1216, 1792]),
    (False, 64, 2240, 9216, [0, 512, 512, 1216, 1792]),      # 256 tiles (experts of fewer tokens by themselves: eqs. (1), (4) on 64 tiles, whose sums can choose other columns)
    (True, 8, 2304, 9728, [0, 128, 128, 448, 640]),          # on codes
])
def test_grouped_step_on_tiles_chosen_by_the_segments(fp8, M, D, F, seg):
    """Experts with 0 and odd numbers of 64-token blocks: packed metadata and weight gradients are the bits of a step on the expert's tokens alone, whose tiles
    are others (128 and 256 tiles sum in the same order); Y3 and dX are the same sums in another order where 64 tiles are among them: 2^-8, a bf16's last place."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(41)
    randn = lambda *shape: torch.randn(shape, dtype=torch.bfloat16, device="cuda", generator=gen)  # noqa: E731
    E, T = len(seg) - 1, seg[-1]
    X, dY, W1, W2 = randn(T, D), randn(T, D), randn(E, F, D).mul_(0.02), randn(E, D, F).mul_(0.02)
    b1 = torch.full((E, F), -0.5 * 0.02 * D ** 0.5, device="cuda")
    sc = dict(x=5 / 448, w1=0.1 / 448, w2=0.1 / 448, y2=0.05, dy=5 / 448, dy1=0.05)
    step = sffn.FfnStepFp8Grouped(seg, D, F, sc, M=M, wgrad_fp8=True) if fp8 else sffn.FfnStepGrouped(seg, D, F, M=M)
    Y3, dX, dW1, dW2 = step(X, W1, W2, b1, dY)
    for e, (a, b) in enumerate(zip(seg, seg[1:])):
        if a == b:
            assert not dW1[e].any() and not dW2[e].any()
            continue
        alone = sffn.FfnStepFp8(b - a, D, F, sc, M=M, wgrad_fp8=True) if fp8 else sffn.FfnStep(b - a, D, F, M=M)
        want = alone(X[a:b].contiguous(), W1[e], W2[e], b1[e], dY[a:b].contiguous())
        assert torch.equal(dW1[e], want[2]) and torch.equal(dW2[e], want[3])
        assert torch.equal(step.saved()["y2_meta"][a:b], alone.saved()["y2_meta"])
        for got, ref in ((Y3[a:b], want[0]), (dX[a:b], want[1])):
            assert (got.float() - ref.float()).norm() <= 2.0 ** -8 * ref.float().norm()


def test_step_on_large_tiles():
    """Every contraction in a launch of its own on its large tile (eqs. (3), (7): 512 x 128), with remainders in all dimensions."""
    _teacher_forced_step_check(2752, 4800, 3136, sffn.MODE_HARD, seed=26)


@pytest.mark.parametrize("fp8,T,D,F", [(False, 1344, 5952, 64), (False, 2112, 3904, 512), (True, 1472, 5504, 128), (True, 2112, 3968, 512)])
def test_forward_call_on_large_tiles_of_a_step_that_shares_launches(fp8, T, D, F):
    """Eq. (3) on 128 tiles in the step's shared launch, on 512 x 128 in the forward call: the same bits, and the oracle's sums (bf16)."""
    inp = make_ffn_inputs(T, D, F, seed=27)
    dev = [to_dev(inp[k]) for k in ("X", "W1", "W2", "b1", "dY")]
    sc = _fp8_step_scales(inp) if fp8 else None
    new = (lambda: sffn.FfnStepFp8(T, D, F, sc, sffn.MODE_HARD, wgrad_fp8=True)) if fp8 else (lambda: sffn.FfnStep(T, D, F, sffn.MODE_HARD))  # noqa: E731
    one, two = new(), new()
    Y3, dX, dW1, dW2 = one(*dev)
    assert torch.equal(two.forward(*dev[:4]), Y3)
    for got, want in zip(two.backward(dev[4]) if fp8 else two.backward(dev[1], dev[4]), (dX, dW1, dW2)):
        assert torch.equal(got, want)
    if not fp8:
        y2 = [to_bits(one.saved()[k]) for k in ("y2_vals", "y2_meta", "colidx")]
        assert_gemm_close(to_bits(Y3), oracle.vnm_spmm(*y2, inp["W2"], 0, 64, 8), "y3")


@pytest.mark.parametrize("fp8,T,D,F", [(False, 1984, 1344, 4160), (True, 3520, 640, 2560)])
def test_step_in_shared_launches_of_128_tiles(fp8, T, D, F):
    """Launches are shared although a contraction by itself would take the large tile: against the oracle."""
    if not fp8:
        _teacher_forced_step_check(T, D, F, sffn.MODE_SOFT, seed=28)
        return
    inp = make_ffn_inputs(T, D, F, seed=28)
    sc = _fp8_step_scales(inp)
    step = sffn.FfnStepFp8(T, D, F, sc, sffn.MODE_SOFT, keep_dense=True, wgrad_fp8=True)
    outs = step(*[to_dev(inp[k]) for k in ("X", "W1", "W2", "b1", "dY")])
    s = {k: to_bits(v) if v.dtype == torch.bfloat16 else v.cpu().numpy() for k, v in step.saved().items()}
    _check_fp8_step_against_oracle(inp, sc, s, {k: to_bits(v) for k, v in zip(("Y3", "dX", "dW1", "dW2"), outs)}, sffn.MODE_SOFT, True, 8)


@pytest.mark.parametrize("fp8,D,F", [(False, 3904, 8256), (True, 3968, 8320)])
def test_grouped_step_on_tiles_of_512_tokens(fp8, D, F):
    """Experts of 2, 0, 10 and 23 token blocks (F: eq. (1) of an expert alone takes no 64 tile, which would sum in another order)."""
    test_grouped_step_on_tiles_chosen_by_the_segments(fp8, 8, D, F, [0, 128, 128, 768, 2240])


# (M, T, D, F, segments of experts; eq. (1): its tile, does it read X as it is on packed weights, does it on others; are the preparing passes one launch)
FORWARD_CALLS = [
    (8, 64, 64, 64, None, 64, 1, 1, 1),             # the smallest: one stage for four wavefronts
    (8, 64, 1088, 1088, None, 64, 1, 1, 1),         # 64 tiles, a half-empty stage round of their four wavefronts
    (8, 832, 320, 576, None, 64, 1, 1, 1), (8, 832, 320, 1344, None, 128, 1, 1, 1),         # 128 tiles, half-empty in both dimensions
    (8, 576, 320, 640, [0, 64, 64, 256, 576], 64, 1, 1, 1), (8, 576, 320, 1600, [0, 64, 64, 256, 576], 128, 1, 1, 1),
    (16, 64, 1088, 1024, None, 64, 1, 1, 1), (16, 832, 320, 1024, None, 128, 1, 1, 1),
    (32, 64, 1088, 1024, None, 64, 1, 1, 1), (32, 832, 320, 1024, None, 128, 1, 1, 1),
    (64, 64, 1088, 3072, None, 64, 1, 1, 1), (64, 832, 320, 2048, None, 128, 1, 1, 1),      # tiles of 128 and 256 hidden units
    (64, 576, 320, 2048, [0, 64, 64, 256, 576], 128, 1, 1, 1),
    # larger weights: the call that packs them copies X into blocks
    (8, 64, 1088, 2112, None, 64, 1, 0, 1), (8, 64, 1088, 4160, None, 64, 1, 0, 1), (8, 832, 1344, 4160, None, 128, 1, 0, 1), (8, 576, 1088, 8256, [0, 64, 64, 256, 576], 128, 1, 0, 1),
    (16, 64, 1088, 2048, None, 64, 1, 0, 1), (32, 64, 2048, 1024, None, 64, 1, 0, 1), (64, 64, 3072, 6144, None, 64, 1, 0, 1),
    (16, 64, 1088, 4096, None, 64, 1, 0, 1), (16, 832, 1344, 4096, None, 128, 1, 0, 1),
    (32, 64, 1088, 4096, None, 64, 1, 0, 1), (32, 832, 1344, 4096, None, 128, 1, 0, 1),
    (64, 64, 3584, 6144, None, 64, 1, 0, 1), (64, 320, 576, 12288, None, 128, 1, 0, 1), (64, 832, 576, 3072, [0, 128, 128, 512, 832], 128, 1, 0, 1),
    (8, 4032, 1152, 2112, None, 256, 0, 0, 1),      # 256 tiles: both copy X
    (8, 4032, 640, 2112, None, 128, 1, 1, 1),       # ... which saves less here than reading X as it is
    # ... and nothing but X.T is prepared in the call on packed weights, behind the tiles of eq. (1)
    (8, 64, 2112, 12352, None, 64, 1, 0, 0), (8, 192, 2112, 12288, None, 128, 1, 0, 0), (16, 64, 2112, 12288, None, 64, 1, 0, 0),
    (16, 192, 2112, 12288, None, 128, 1, 0, 0), (32, 128, 1600, 18432, None, 128, 1, 0, 0), (64, 64, 2112, 14336, None, 64, 1, 0, 0), (64, 320, 2112, 12288, None, 128, 1, 0, 0),
    (64, 576, 1088, 8192, [0, 64, 64, 256, 576], 128, 1, 0, 0),
]


@pytest.mark.parametrize("M,T,D,F,seg,tile,packed_reads,reads,together", FORWARD_CALLS)
def test_forward_call_on_packed_weights_reads_x_as_it_is(M, T, D, F, seg, tile, packed_reads, reads, together):
    """The same bits as the call that packs the weights, in Y3 and, through the backward call, in all gradients (X.T); where that call does not copy X into blocks
    either, both against the oracle."""
    experts = len(seg) - 1 if seg else 1
    parts = [make_ffn_inputs(T, D, F, seed=51 + e) for e in range(experts)]
    inp = {k: np.stack([p[k] for p in parts]) if seg and k in ("W1", "W2", "b1") else parts[0][k] for k in parts[0]}
    dev = {k: to_dev(inp[k]) for k in ("X", "W1", "W2", "b1", "dY")}
    weights = [dev[k] for k in ("W1", "W2", "b1")]
    new = (lambda **kw: sffn.FfnStepGrouped(seg, D, F, M=M, **kw)) if seg else (lambda **kw: sffn.FfnStep(T, D, F, M=M, **kw))  # noqa: E731
    a, b = new(), new(keep_dense=bool(reads))
    want = [a.forward(dev["X"], *weights), *a.backward(dev["W1"], dev["dY"])]
    b.forward(dev["dY"], *weights)          # packs the weights; another X
    got = [b.forward(dev["X"], *weights, weights_packed=True), *b.backward(dev["W1"], dev["dY"])]
    for g, w in zip(got, want):
        assert torch.equal(g, w)
    if not reads:
        return
    s = {k: to_bits(v) for k, v in b.saved().items()}
    outs = {k: to_bits(v) for k, v in zip(("Y3", "dX", "dW1", "dW2"), got)}
    if not seg:
        _check_wide_step_against_oracle(inp, s, outs, sffn.MODE_HARD, M)
    for e in range(experts if seg else 0):
        lo, hi = seg[e], seg[e + 1]
        if lo == hi:
            continue
        one = dict(X=inp["X"][lo:hi], dY=inp["dY"][lo:hi], W1=inp["W1"][e], W2=inp["W2"][e], b1=inp["b1"][e])
        se = {k: s[k][e] for k in ("w1_vals", "w1_meta", "w2t_vals", "w2t_meta")}
        se.update({k: s[k][lo:hi] for k in ("y1", "y2_vals", "y2_meta", "dy2", "dy1_vals")}, colidx=s["colidx"][lo // 64:hi // 64],
                  y1_kept=s["y1_kept"].reshape(-1)[lo * 2 * F // M:hi * 2 * F // M])
        _check_wide_step_against_oracle(one, se, dict(Y3=outs["Y3"][lo:hi], dX=outs["dX"][lo:hi], dW1=outs["dW1"][e], dW2=outs["dW2"][e]), sffn.MODE_HARD, M)


# (M, T, D, F, are the preparing passes one launch): the router's step shares launches in all of them
ROUTER_CALLS = [(8, 700, 2048, 12288, 0), (16, 700, 2048, 12288, 0), (32, 300, 2048, 12288, 0), (64, 700, 2048, 12288, 0), (16, 576, 448, 1280, 1)]


@pytest.mark.parametrize("mode", [sffn.MODE_HARD, sffn.MODE_SOFT])
@pytest.mark.parametrize("M,T,D,F,together", ROUTER_CALLS)
def test_router_step_in_shared_launches(M, T, D, F, together, mode):
    """Preparing passes behind the tiles of eq. (1) (not in the last, smallest case), eqs. (3) and (4) in one launch, the transpose of dW2 behind eq. (7): every stage on
    sampled rows and hidden units against the oracle.  The forward and backward calls, whose eqs. (3), (4) have launches of their own, and calls on weights that are
    packed already: the same bits."""
    inp = make_router_inputs(T, D, F, M, seed=61)
    dev = {k: to_dev(v) for k, v in inp.items()}
    route = sffn.venom_route(dev["X"], dev["means"], M)
    one, two = sffn.FfnRouterStep(T, D, F, M, mode), sffn.FfnRouterStep(T, D, F, M, mode)
    want = [t.clone() for t in one(route, dev["X"], dev["W1"], dev["W2"], dev["b1"], dev["dY"])]
    got = [two.forward(route, dev["X"], dev["W1"], dev["W2"], dev["b1"]), *two.backward(route, dev["dY"])]
    for g, w in zip(got, want):
        assert torch.equal(g, w)
    for packed in (True, False):
        for g, w in zip(one(route, dev["X"], dev["W1"], dev["W2"], dev["b1"], dev["dY"], weights_packed=packed), want):
            assert torch.equal(g, w)
    for g, w in zip(sampled_router_step_check(inp, dev, M, mode), want):
        assert np.array_equal(g, to_bits(w))
    if mode == sffn.MODE_HARD and F <= 1280:       # (5 %: the oracle's own run, in which near ties of the 2:4 choice may fall the other way)
        ref = oracle.ffn_router_step_ref(inp["X"], inp["W1"], inp["W2"], inp["b1"], inp["dY"], inp["means"], M)
        for name, g in zip(("y3", "dX", "dW1", "dW2"), want):
            a, b = oracle.bits_to_f64(to_bits(g)), oracle.bits_to_f64(ref[name])
            assert np.linalg.norm(a - b) <= 0.05 * np.linalg.norm(b), name


@pytest.mark.parametrize("T,N,K", [(2112, 4160, 256), (2112, 4160, 512), (2112, 4160, 768), (2112, 4160, 1344), (1984, 2240, 256), (1984, 2240, 768), (576, 3008, 2048)])
def test_standalone_24_contractions_on_large_tiles(T, N, K):
    """256 and (the last three) 128 tiles with remainders in both dimensions; metadata fetched for four stages at a time (one, two, three and eight groups), and
    stage by stage (K = 1344)."""
    rng = np.random.default_rng(71)
    X, W = (bf16_bits_from_f32(rng.standard_normal((n, K)).astype(np.float32)) for n in (T, N))
    b1 = rng.standard_normal(N).astype(np.float32)
    vals, meta = sffn.prune24_compress(to_dev(W), False, sffn.MODE_HARD)
    rv, rm = oracle.prune24_compress(W, sffn.MODE_HARD)
    assert np.array_equal(to_bits(vals), rv) and np.array_equal(to_bits(meta), rm)
    assert_gemm_close(to_bits(sffn.spmm24_fwd(to_dev(X), vals, meta, to_dev(b1))), oracle.spmm24(X, rv, rm, b1), "fwd")
    assert_gemm_close(to_bits(sffn.spmm24_dgrad(to_dev(X), vals, meta)), oracle.spmm24(X, rv, rm, None), "dgrad")


@pytest.mark.parametrize("M,T,F", [(8, 64, 64), (8, 128, 320), (16, 64, 64), (16, 128, 448), (32, 64, 64), (32, 128, 704), (64, 64, 128), (64, 128, 640)])
def test_compressor_choices_among_equal_and_special_values(M, T, F):
    """The stand-alone compressor, bit for bit: a workgroup of one to four wavefronts of 64 columns, activations of few distinct values (ties of column scores
    and of survivors everywhere), NaN (counts as 0), infinities, squares that overflow or vanish."""
    rng = np.random.default_rng(M * F)
    y1 = bf16_bits_from_f32(rng.integers(-3, 4, (T, F)).astype(np.float32) / 2)
    y1[rng.random((T, F)) < 0.02] = 0x7FC0
    y1[rng.random((T, F)) < 0.02] = 0xFF81
    y1[rng.random((T, F)) < 0.001] = 0x7F80
    y1[rng.random((T, F)) < 0.02] = 0x0001
    y1[rng.random((T, F)) < 0.001] = 0x7F7F
    v, m, c = sffn.sqrelu_vnm_compress(to_dev(y1), 64, M)
    clean = np.where((y1 & 0x7FFF) > 0x7F80, 0, y1).astype(np.uint16)
    rv, rm, rc = oracle.sqrelu_vnm_compress(clean, 64, M)
    assert np.array_equal(to_bits(c), rc) and np.array_equal(to_bits(m), rm) and np.array_equal(to_bits(v), rv)


@pytest.mark.parametrize("M", [32, 64])
@pytest.mark.parametrize("blocks", [1, 2, 3, 4, 5, 6, 7, 8, 9])
def test_kept_row_weight_gradients_over_few_token_blocks(M, blocks):
    """Up to four token blocks the compacted operand is multiplied as a whole.  From five on the kept rows only, on 512 x 32 tiles: every place in the four
    blocks in flight (the two sets of LDS addresses alternate), N that no tile divides.  (Fewer blocks on kept rows: experts, below.)"""
    T, F, N = 64 * blocks, 16 * M, 192
    rng = np.random.default_rng(M + blocks)
    y1 = bf16_bits_from_f32(rng.standard_normal((T, F)).astype(np.float32) - np.float32(0.5))
    G = bf16_bits_from_f32(rng.standard_normal((T, N)).astype(np.float32))
    packed = oracle.sqrelu_vnm_compress(y1, 64, M)
    dev = [to_dev(x) for x in packed]
    for f_major in (True, False):
        assert_gemm_close(to_bits(sffn.vnm_wgrad(*dev, to_dev(G), f_major, 64, M)), oracle.vnm_wgrad(*packed, G, f_major, 64, M), "wgrad")


@pytest.mark.parametrize("M", [32, 64])
@pytest.mark.parametrize("blocks", [5, 6, 7, 10, 11, 12, 13])
def test_kept_row_weight_gradients_on_large_tiles(M, blocks):
    """512 x 64 tiles (17 x 17 of them, at M = 32 the last row half full) at every place in the six token blocks that are in flight, from the fewest
    tokens of this form on.  Small integers: every sum is exact in float32, so the results are equal to the bit."""
    T, F, N = 64 * blocks, 8704 - 256 * (M == 32), 1088
    rng = np.random.default_rng(M + blocks)
    y1 = bf16_bits_from_f32(rng.integers(-3, 4, (T, F)).astype(np.float32))
    G = bf16_bits_from_f32(rng.integers(-2, 3, (T, N)).astype(np.float32))
    packed = oracle.sqrelu_vnm_compress(y1, 64, M)
    dense, g = to_dev(oracle.vnm_decompress(*packed, 64, M)).float(), to_dev(G).float()
    dev = [to_dev(x) for x in packed]
    want = (dense.t().contiguous() @ g).bfloat16()
    assert torch.equal(sffn.vnm_wgrad(*dev, to_dev(G), True, 64, M), want)
    assert torch.equal(sffn.vnm_wgrad(*dev, to_dev(G), False, 64, M), want.t())


# (M, D, F, token blocks of the experts): eqs. (5), (8) on the kept rows in launches of their own, on 512 x 32 and 512 x 64 tiles
KEPT_EXPERTS = [(M, D, F, blocks) for M in (32, 64) for D, F, blocks in ((384, 3072, (2, 3, 4, 5, 6, 7, 96)), (960, 7168, (7, 2, 6, 3, 24, 5, 4)))]


@pytest.mark.parametrize("M,D,F,blocks", KEPT_EXPERTS)
def test_kept_row_weight_gradients_of_experts_with_few_token_blocks(M, D, F, blocks):
    """Fewer token blocks than are in flight (four; six on the large tile at M = 32), as many and more: the weight gradients of every expert have the bits of the unfused step on its tokens
    alone, which multiplies the rows of zeros too."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(43)
    randn = lambda *shape: torch.randn(shape, dtype=torch.bfloat16, device="cuda", generator=gen)  # noqa: E731
    seg = [64 * sum(blocks[:e]) for e in range(len(blocks) + 1)]
    E, T = len(blocks), seg[-1]
    X, dY, W1, W2 = randn(T, D), randn(T, D), randn(E, F, D).mul_(0.02), randn(E, D, F).mul_(0.02)
    b1 = torch.full((E, F), -0.5 * 0.02 * D ** 0.5, device="cuda")
    _, _, dW1, dW2 = sffn.FfnStepGrouped(seg, D, F, M=M, lean=True)(X, W1, W2, b1, dY)
    for e, (a, b) in enumerate(zip(seg, seg[1:])):
        want = sffn.FfnStep(b - a, D, F, M=M, unfused=True)(X[a:b].contiguous(), W1[e], W2[e], b1[e], dY[a:b].contiguous())
        assert torch.equal(dW1[e], want[2]) and torch.equal(dW2[e], want[3]), (e, b - a)


# (T, N, F) of weight gradients on 128 tiles, three workgroups a CU
THREE_A_CU = [
    (64, 2560, 2624), (128, 2560, 2624), (192, 2560, 2624),     # one stage, as many as the ring has, one more; 420 tiles, the last row half full
    (320, 4032, 4160),          # 1056 tiles: a second round of three workgroups a CU, both edges half full
    (1280, 3008, 3136),         # 600 tiles of many stages
]


@pytest.mark.parametrize("T,N,F", THREE_A_CU + [(320, 1088, 12352)])      # (the last on 256 tiles)
def test_weight_gradients_with_three_workgroups_a_cu(T, N, F):
    """Small integers: every sum is exact in float32, so the results are equal to the bit; added to float32 gradients in a backward call."""
    rng = np.random.default_rng(T + N)
    y1 = bf16_bits_from_f32(rng.integers(-3, 4, (T, F)).astype(np.float32))
    G = bf16_bits_from_f32(rng.integers(-2, 3, (T, N)).astype(np.float32))
    packed = oracle.sqrelu_vnm_compress(y1, 64, 8)
    dense, g = to_dev(oracle.vnm_decompress(*packed, 64, 8)).float(), to_dev(G).float()
    dev = [to_dev(x) for x in packed]
    want = (dense.t().contiguous() @ g).bfloat16()
    assert torch.equal(sffn.vnm_wgrad(*dev, to_dev(G), True, 64, 8), want)
    assert torch.equal(sffn.vnm_wgrad(*dev, to_dev(G), False, 64, 8), want.t())


THREE_A_CU_FP32 = (192, 6592, 19008)


@pytest.mark.parametrize("T,D,F", [(192, 4544, 11264), THREE_A_CU_FP32])
def test_float32_weight_gradients_with_three_workgroups_a_cu(T, D, F):
    """A backward call into float32 (the second: eqs. (5), (8) in launches of their own; several rounds of tiles, both edges half full) rounds to the bits of the bf16 step."""
    inp = make_ffn_inputs(T, D, F, seed=31)
    dev = [to_dev(inp[k]) for k in ("X", "W1", "W2", "b1", "dY")]
    plain = [t.clone() for t in sffn.FfnStep(T, D, F, lean=True)(*dev)]
    step = sffn.FfnStep(T, D, F, lean=True, dw_fp32=True)
    step.dW1.zero_(), step.dW2.zero_()
    step.forward(*dev[:4])
    step.backward(dev[1], dev[4])
    for a, b in zip(plain[2:], (step.dW1, step.dW2)):
        assert torch.equal(a, b.bfloat16())


# (fp8, T, N, F) of eqs. (3), (7) on 64 tiles: as many stages as the fewest that take them, two a wavefront where the ring has three; one wavefront with a stage more; rings that are just full,
# and one stage more for some of the wavefronts; three token blocks with selections of their own; contractions shared by workgroups
KEPT_CALLS = [(fp8, T, N, F << fp8) for fp8 in (False, True) for T, N, F in ((64, 64, 512), (64, 128, 576), (64, 128, 768), (64, 64, 832), (64, 64, 1024), (64, 64, 1152), (192, 320, 2176), (64, 64, 9216))]


@pytest.mark.parametrize("fp8,T,N,F", KEPT_CALLS + [(fp8, 64, N, F) for fp8 in (False, True) for N, F in ((64, 128), (192, 384))])
def test_activation_contractions_on_kept_rows(fp8, T, N, F):
    """Eqs. (3), (7) on 64 tiles (the last four, too short for them, on 128).  Small integers (codes: with scales of 1): every sum is exact in float32, so the results are equal to the bit."""
    rng = np.random.default_rng(T + N + F)
    y1 = bf16_bits_from_f32(rng.integers(-2, 3, (T, F)).astype(np.float32))
    W = bf16_bits_from_f32(rng.integers(-2, 3, (N, F)).astype(np.float32))
    packed = oracle.sqrelu_vnm_compress(y1, 64, 8)
    want = (to_dev(oracle.vnm_decompress(*packed, 64, 8)).float() @ to_dev(W).float().t()).bfloat16()
    if fp8:
        codes = sffn.sqrelu_vnm_compress_fp8(to_dev(y1), 1.0, 64, 8)
        assert torch.equal(sffn.vnm_spmm_fp8(*codes, 1.0, sffn.quantize_fp8(to_dev(np.ascontiguousarray(W.T)), 1.0), 1.0, 1, 64, 8), want)
        return
    dev = [to_dev(x) for x in packed]
    assert torch.equal(sffn.vnm_spmm(*dev, to_dev(W), 0, 64, 8), want)
    assert torch.equal(sffn.vnm_spmm(*dev, to_dev(np.ascontiguousarray(W.T)), 1, 64, 8), want)
