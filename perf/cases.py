"""The work that users of this package have it do, as a list of cases that can be timed.

Every case is one pass through the public entry points at one shape.  `listed()` gives the fixed ones, `draw(rng)` more of the same ranges:
d_model 256 to 8192, d_ff 2.5 to 4.5 times that (Table 1 of the paper has 4, a 70B-scale layer 3.5), 64 to 16384 tokens in a call (an
evaluation call: up to 2048), every size a multiple of 64 as the entry points want it (fp8: d_model and d_ff of 128; blocks of M >= 16
columns: d_ff of 16 M), and no call larger than the 70B-scale layer on 8192 tokens.
"""
import math

import torch

import paper_2602_06183_amd as sffn

MODES = {"hard": sffn.MODE_HARD, "soft": sffn.MODE_SOFT}
# standard-normal quantiles of the wanted fraction of zero SquaredReLU outputs (the paper reports more than 0.9 in training, about 0.5 at its start)
QUANTILE = {0.5: 0.0, 0.75: 0.6744897501960817, 0.9: 1.2815515655446004, 0.95: 1.6448536269514722}


def listed():
    return [
        # one small layer, the whole training step in one call, as a first-time user builds it: launches and host time count
        dict(name="step_tiny", kind="step", T=512, D=256, F=1024, M=8, mode="soft", lean=False, zero=0.9),
        # no dimension fits the tiles: odd multiples of 64 tokens, hidden units and model dimensions
        dict(name="step_ragged", kind="step", T=1984, D=1344, F=4160, M=8, mode="hard", lean=True, zero=0.75),
        # the FFN of a Llama-1B layer on 4 sequences of 2048 tokens
        dict(name="step_1b", kind="step", T=8192, D=2048, F=8192, M=8, mode="soft", lean=True, zero=0.9),
        # the 70B-scale layer: the largest call
        dict(name="step_70b", kind="step", T=8192, D=8192, F=28672, M=8, mode="hard", lean=True, zero=0.9),
        # wider V:N:M blocks (64:2:32) at the Llama-7B shape
        dict(name="step_wide_7b", kind="step", T=16384, D=4096, F=16384, M=32, mode="soft", lean=True, zero=0.9),
        # evaluation of one short sequence on weights packed earlier: forward only, the fewest tokens a call can have
        dict(name="eval_1b", kind="eval", T=64, D=2048, F=8192, M=8, mode="soft", lean=True, zero=0.9),
        # an optimizer step of a training loop: two micro-batches through Alg. 1 and Alg. 2 as separate calls on one scratch buffer, the second
        # on the first one's packed weights, weight gradients summed in float32
        dict(name="micro_7b", kind="micro", T=8192, D=4096, F=16384, M=8, mode="soft", lean=True, zero=0.9),
        # a mixture-of-experts layer: 8 experts, 16384 tokens routed top-2, uneven segments
        dict(name="moe_8x", kind="moe", tokens=16384, experts=8, D=4096, F=14336, M=8, mode="soft", lean=True, zero=0.9),
        # the 70B-scale layer with fp8 operands in all six contractions, delayed scaling
        dict(name="fp8_70b", kind="fp8", T=8192, D=8192, F=28672, M=8, mode="hard", lean=True, zero=0.9),
        # the neuron-level router's training step with the routing inside the call: 4 experts of hidden units
        dict(name="router_1b", kind="router", T=8192, D=2048, F=8192, M=16, mode="soft", zero=0.9),
        # the sparsifiers as separate operations, for users who bring their own contractions: both weights, the activation, eq. (6)
        dict(name="pack_7b", kind="pack", T=16384, D=4096, F=16384, M=8, mode="soft", zero=0.9),
        # the six contractions of the layer as separate operations on packed tensors
        dict(name="gemm_1b", kind="gemm", T=8192, D=2048, F=8192, M=8, mode="soft", zero=0.9),
    ]


#: The most multiply-adds of one dense contraction (T D F) that a drawn case of a kind has.
MOST = {"step": 1.92e12, "eval": 4.8e11, "micro": 5.5e11, "moe": 1.5e12, "fp8": 1.92e12, "router": 1.1e12, "pack": 1.1e12, "gemm": 6e11}


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "eval", "micro", "moe", "fp8", "fp8", "router", "pack", "gemm"])
    M = {"step": rng.choice([8, 8, 16, 32, 64]), "fp8": rng.choice([8, 8, 16]), "router": rng.choice([8, 16, 32, 64]),
         "pack": rng.choice([8, 8, 16, 32]), "gemm": rng.choice([8, 8, 16, 32])}.get(kind, 8)
    spread = lambda lo, hi: math.exp(rng.uniform(math.log(lo), math.log(hi)))  # noqa: E731
    unit_d, unit_f = (128, max(128, 32 * M if M > 8 else 0)) if kind == "fp8" else (64, 16 * M if M > 8 or kind == "router" else 64)
    top = {"moe": 4096, "gemm": 4096}.get(kind, 8192)
    D = unit_d * max(1, round(spread(256, top) / unit_d))
    F = min(28672, unit_f * max(1, round(D * rng.uniform(2.5, 4.5) / unit_f)))
    most = min(2048 if kind == "eval" else 16384, MOST[kind] / (D * F))
    case = dict(kind=kind, D=D, F=F, M=M, mode=rng.choice(["hard", "soft"]), zero=rng.choice([0.5, 0.75, 0.9, 0.9, 0.95]))
    if kind == "moe":
        case.update(experts=rng.choice([4, 8]), tokens=max(256, int(spread(256, most / 2))), lean=True)
    else:
        case["T"] = 64 * max(1, int(spread(64, most)) // 64)
        if kind not in ("router", "pack", "gemm"):
            case["lean"] = rng.choice([True, True, False])
    return case


def _rows(case):
    """Token rows of one call; mixture of experts: two slots a token and room for rounding every segment up to 64 rows."""
    if case["kind"] != "moe":
        return case["T"]
    return -(-2 * case["tokens"] // 64) * 64 + 64 * case["experts"]


def _bias(W1, zero):
    """-z times each neuron's standard deviation under X ~ N(0, 1) once the two smallest of every four weights are dropped."""
    out = torch.empty(W1.shape[:-1], dtype=torch.float32, device=W1.device)
    flat, rows = out.view(-1), W1.view(-1, W1.shape[-1])
    step = max(64, (1 << 26) // W1.shape[-1])
    for r in range(0, rows.shape[0], step):
        q = rows[r:r + step].float().square_().view(-1, W1.shape[-1] // 4, 4)
        a, b = torch.maximum(q[..., 0], q[..., 1]), torch.minimum(q[..., 0], q[..., 1])
        c, d = torch.maximum(q[..., 2], q[..., 3]), torch.minimum(q[..., 2], q[..., 3])
        second = torch.maximum(torch.minimum(a, c), torch.maximum(b, d))
        flat[r:r + step] = (torch.maximum(a, c) + second).sum(1).sqrt_().mul_(-QUANTILE[zero])
    return out


def _segments(case, gen):
    """Row offsets of the experts for tokens routed top-2 by normal logits: the last segment takes the rows that rounding left over."""
    E = case["experts"]
    logits = torch.randn((case["tokens"], E), device="cuda", generator=gen)
    counts = torch.bincount(logits.topk(2, dim=1).indices.reshape(-1), minlength=E).tolist()
    seg = [0]
    for c in counts:
        seg.append(seg[-1] + -(-c // 64) * 64)
    seg[-1] = _rows(case)
    return seg, counts


def prepare(case, seed):
    kind, D, F, M, mode = case["kind"], case["D"], case["F"], case["M"], MODES[case["mode"]]
    T, lead = _rows(case), (case["experts"],) if kind == "moe" else ()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    randn = lambda *shape: torch.randn(shape, dtype=torch.bfloat16, device="cuda", generator=gen)  # noqa: E731
    X, dY = randn(T, D), randn(T, D)
    W1, W2 = randn(*lead, F, D).mul_(0.02), randn(*lead, D, F).mul_(0.02)
    s = dict(kind=kind, M=M, mode=mode, X=X, dY=dY, W1=W1, W2=W2, b1=_bias(W1, case["zero"]))
    if kind in ("step", "eval"):
        s["step"] = sffn.FfnStep(T, D, F, mode, M=M, lean=case["lean"])
        if kind == "eval":
            s["step"].forward(X, W1, W2, s["b1"])
    elif kind == "micro":
        size = sffn.buffer_sizes(T, D, F, mode, M=M, lean=case["lean"])
        scratch = torch.empty((size["scratch"],), dtype=torch.uint8, device="cuda")
        first = sffn.FfnStep(T, D, F, mode, M=M, lean=case["lean"], scratch=scratch, dw_fp32=True)
        second = sffn.FfnStep(T, D, F, mode, M=M, lean=case["lean"], scratch=scratch, weights_of=first, dw_fp32=True)
        second.dW1, second.dW2 = first.dW1, first.dW2
        s.update(first=first, second=second, X2=randn(T, D), dY2=randn(T, D))
    elif kind == "moe":
        seg, counts = _segments(case, gen)
        for e, c in enumerate(counts):      # a segment's rows past its tokens are padding
            X[seg[e] + c:seg[e + 1]] = 0
            dY[seg[e] + c:seg[e + 1]] = 0
        s["step"] = sffn.FfnStepGrouped(seg, D, F, mode, M=M, lean=case["lean"])
    elif kind == "fp8":
        top = lambda t: max(float(t.abs().max()), 1e-12) / 448  # noqa: E731
        step = sffn.FfnStepFp8(T, D, F, dict(x=top(X), w1=top(W1), w2=top(W2), y2=1.0, dy=top(dY), dy1=1.0), mode, wgrad_fp8=True,
                               lean=case["lean"], M=M)
        step(X, W1, W2, s["b1"], dY)        # delayed scaling: the maxima of the call before make the scales
        step.set_scales({k: max(v, 1e-12) / 448 for k, v in step.amax_dict().items()})
        s["step"] = step
    elif kind == "router":
        # unit-length expert means: the average of the expert's rows of W1 plus a random direction of comparable length
        E = M // 4
        mean = W1.view(F // M, E, 4, D).float().mean((0, 2))
        mean += torch.randn((E, D), device="cuda", generator=gen) * mean.norm(dim=1, keepdim=True) / math.sqrt(D)
        s["means"] = (mean / mean.norm(dim=1, keepdim=True)).to(torch.bfloat16)
        s["step"] = sffn.FfnRouterStep(T, D, F, M, mode)
    elif kind == "pack":
        s["y1"], s["dy2"] = randn(T, F).sub_(QUANTILE[case["zero"]]), randn(T, F)
    elif kind == "gemm":
        s["w1"], s["w2t"] = sffn.prune24_compress(W1, False, mode), sffn.prune24_compress(W2, True, mode)
        s["y2"] = sffn.sqrelu_vnm_compress(randn(T, F).sub_(QUANTILE[case["zero"]]), 64, M)
    return s


def run(s):
    kind, M, X, dY, W1, W2, b1 = s["kind"], s["M"], s["X"], s["dY"], s["W1"], s["W2"], s["b1"]
    if kind in ("step", "moe"):
        return s["step"](X, W1, W2, b1, dY)
    if kind == "eval":
        return s["step"].forward(X, W1, W2, b1, weights_packed=True)
    if kind == "micro":
        first, second = s["first"], s["second"]
        first.dW1.zero_()
        first.dW2.zero_()
        ya = first.forward(X, W1, W2, b1)
        yb = second.forward(s["X2"], W1, W2, b1, weights_packed=True)
        dxb = second.backward(W1, s["dY2"])[0]
        dxa = first.backward(W1, dY)[0]
        return ya, yb, dxa, dxb, first.dW1, first.dW2
    if kind == "fp8":
        return (*s["step"](X, W1, W2, b1, dY), s["step"].amax[:6])
    if kind == "router":
        return s["step"].full(s["means"], X, W1, W2, b1, dY)
    if kind == "pack":
        y2 = sffn.sqrelu_vnm_compress(s["y1"], 64, M)
        return (sffn.prune24_compress(W1, False, s["mode"]), sffn.prune24_compress(W2, True, s["mode"]), y2,
                sffn.dsqrelu_vnm(s["dy2"], s["y1"], y2[1], y2[2], 64, M))
    y2 = s["y2"]
    return (sffn.spmm24_fwd(X, *s["w1"], b1), sffn.vnm_spmm(*y2, W2, 0, 64, M), sffn.spmm24_dgrad(dY, *s["w2t"]),
            sffn.vnm_wgrad(*y2, dY, False, 64, M), sffn.vnm_spmm(*y2, W1, 1, 64, M), sffn.vnm_wgrad(*y2, X, True, 64, M))


def work(case):
    """Every input read once and every output written once; the non-zero multiply-adds of the method, times two."""
    kind, D, F, M = case["kind"], case["D"], case["F"], case["M"]
    T, E = _rows(case), case.get("experts", 1)
    packed24, packed_vnm = 1.125 * F * D, (4 + 0.5 + 1 / 16) / M * T * F      # bytes of a packed weight / of a packed activation
    sparse_w, sparse_a = 1.0 * T * D * F, 4.0 * T * D * F / M                 # flop of a contraction with 2:4 weights / with V:2:M activations
    if kind == "eval":
        return dict(bytes=4 * T * D + packed24 + 2 * D * F + 4 * F, flops=sparse_w + sparse_a)
    if kind == "pack":
        return dict(bytes=4 * D * F + 2 * packed24 + 2 * T * F + packed_vnm + 2 * 4 / M * T * F, flops=0)
    if kind == "gemm":
        return dict(bytes=4 * T * D + 8 * D * F + 2 * packed24 + packed_vnm + 4 * T * F + 4 * T * D + 4 * F, flops=2 * sparse_w + 4 * sparse_a)
    if kind == "router":        # eqs. (1), (4) at the routed hidden units only: 4 of every M
        return dict(bytes=8 * T * D + 8 * D * F + 4 * F, flops=8.0 * T * D * F / M + 4 * sparse_a)
    flops = 2 * sparse_w + 4 * sparse_a
    if kind == "micro":
        return dict(bytes=2 * 8 * T * D + 4 * D * F + 8 * D * F + 4 * F, flops=2 * flops)
    return dict(bytes=8 * T * D + E * (8 * D * F + 4 * F), flops=flops)


def tolerance(case):
    """The packed tensors are defined to the bit; bf16 results of contractions (and, fp8, of code products) to their last places."""
    return "exact" if case["kind"] == "pack" else {"rel": 1e-2}
