"""Which kernels the built library launches for a call (tests/launches.cpp stands in for the HIP runtime)."""
import os
import re
import subprocess

import pytest

import paper_2602_06183_amd as sffn

HERE = os.path.dirname(os.path.abspath(__file__))
FORWARD, HEAD, TAIL = 0, 1, 2          # launches of eqs. (3), (5), (4), of (5), (4) and of (7), (8)


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """calls (lines for launches.cpp) -> the kernels of each"""
    exe = str(tmp_path_factory.mktemp("launches") / "launches")
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", os.path.join(HERE, "launches.cpp"), "-o", exe, "-ldl"], check=True)

    def run(calls):
        out = subprocess.run([exe, sffn.lib_path()], input="\n".join(calls), capture_output=True, text=True, check=True).stdout.strip().split("\n")
        assert len(out) == len(calls) and not any(line.startswith("refused") for line in out), out
        return [line.split(" ; ") for line in out]
    return run


def step(call, M, T, D, F, fp8=0, seg=None, flags=sffn.FLAG_LEAN):
    return "step %s %d %d %d %d %d %d %d %s" % (call, fp8, M, T, D, F, flags | (sffn.FLAG_FP8_WGRAD if fp8 else 0), len(seg) - 1 if seg else 0, " ".join(map(str, seg or [])))


GRADIENT = {"1, 1, 64, 3, 4": 64, "2, 2, 64, 2, 1": 3, "2, 2, 64, 3, 1": 128, "2, 2, 128, 2, 1": "tall", "2, 4, 128, 3, 1": 256}
ACTIVATION = {"1, 1, 2, 3, 4": 64, "2, 2, 2, 3, 1": 128, "4, 1, 4, 3, 1": "tall", "4, 2, 4, 3, 1": 256, "8, 1, 4, 3, 1": 512}
WEIGHT = {"1, 1, 64, 1, 4": 64, "1, 1, 64, 2, 4": 64, "1, 1, 64, 3, 4": 64, "1, 1, 128, 2, 4": 64, "2, 2, 64, 3, 1": 128, "2, 2, 128, 2, 1": "tall", "2, 4, 128, 3, 1": 256}


def tiles(kernel):
    """The tiles of a launch's contractions: activation (eqs. (3), (7)), gradient (eqs. (5), (8)), weight (eqs. (1), (4)); gathered rows: 0"""
    found = {}
    for kind, known, pattern in (("activation", ACTIVATION, r"Vnm8Unit<\w+, sffn::VTile<([^>]*)>"), ("gradient", GRADIENT, r"WgradUnit<[^:]*sffn::WTile<([^>]*)>"), ("weight", WEIGHT, r"GemmV2Unit<true, true, [^:]*sffn::Tile<([^>]*)>")):
        m = re.search(pattern, kernel)
        if m:
            found[kind] = known[m.group(1)]
    if "Gather" in kernel:
        found["activation"] = 0
    return found


def form(kernels, what, M=8):
    """Bits 0, 1, 2: eqs. (3) / (7), (5) / (8), (4) on tall tiles where 128 would do; None: the call shares no such launch"""
    want = {FORWARD: ["activation", "gradient", "weight"], HEAD: ["gradient", "weight"], TAIL: ["activation", "gradient"]}[what]
    for k in kernels:
        t = tiles(k)
        if sorted(t) == sorted(want):
            return sum(bit for kind, bit in (("activation", 1), ("gradient", 2), ("weight", 4)) if t.get(kind) == "tall" and not (kind == "weight" and M == 64))
    return None


def test_shared_launches_of_the_gpu_tests(launches):
    from tests.test_gpu_tall_tiles import FP8, PLAIN, WIDE
    cases = [(0, 8, *c) for c in PLAIN] + [(0, *c) for c in WIDE] + [(1, *c) for c in FP8]
    calls = [step(call, M, T, D, F, fp8) for fp8, M, T, D, F, _ in cases for call in ("step", "backward")]
    got = launches(calls)
    for (fp8, M, T, D, F, want), whole, back in zip(cases, got[::2], got[1::2]):
        assert (form(whole, FORWARD, M), form(back, HEAD, M), form(whole, TAIL, M)) == want, (fp8, M, T, D, F)
        assert form(back, TAIL, M) == want[2]


def test_launches_of_their_own_of_the_gpu_tests(launches):
    from tests.test_gpu_tall_tiles import ALONE_ACTIVATION, ALONE_GRADIENT
    for call, kernels in zip(ALONE_ACTIVATION, launches(["spmm %d 8 %d %d %d" % c for c in ALONE_ACTIVATION])):
        assert tiles(kernels[-1]) == {"activation": "tall"}, call
    for major in (0, 1):
        for call, kernels in zip(ALONE_GRADIENT, launches(["wgrad %d 8 %d %d %d" % (major, T, F, N) for _, T, N, F in ALONE_GRADIENT])):
            assert tiles(kernels[-1]) == {"gradient": "tall"}, call


def test_tall_tiles_beside_float32_sums(launches):
    """Against backward calls that were timed on every form: chosen, they take no longer than tiles of 128 do, and less on average."""
    rows = [line.split(" | ") for line in open(os.path.join(HERE, "golden", "sums_times.txt")) if not line.startswith("#")]
    cases = [([int(v) for v in c.split()[:4]], [int(v) for v in c.split()[4].split(",")] if "," in c else None, list(map(float, h.split())), list(map(float, t.split()))) for c, h, t in rows]
    got = launches([step("backward", *shape, seg=seg, flags=sffn.FLAG_LEAN | sffn.FLAG_DW_FP32_ACCUMULATE) for shape, seg, _, _ in cases])
    ratios = []
    for (shape, seg, head, tail), kernels in zip(cases, got):
        h, t = form(kernels, HEAD, shape[0]), form(kernels, TAIL, shape[0])
        ratios += [(head[{0: 0, 2: 1, 6: 2}[h]] / head[0], shape, seg, h), (tail[t] / tail[0], shape, seg, t)]
    assert max(ratios)[0] <= 1.04, max(ratios)
    assert sum(r[0] for r in ratios) / len(ratios) <= 0.985


def test_tall_tiles_beside_few_tokens(launches):
    """The same for steps of few tokens: eq. (5) beside 64 tiles of eq. (3)."""
    rows = [line.split(" | ") for line in open(os.path.join(HERE, "golden", "few_tokens_times.txt")) if not line.startswith("#")]
    cases = [(list(map(int, c.split())), list(map(float, t.split()))) for c, t in rows]
    ratios = [(t[form(kernels, FORWARD) // 2] / t[0], shape) for (shape, t), kernels in zip(cases, launches([step("step", 8, *shape) for shape, _ in cases]))]
    assert max(ratios)[0] <= 1.03, max(ratios)
    assert sum(r[0] for r in ratios) / len(ratios) <= 0.97


PRUNES = re.compile(r"GemmV2Unit<true, true, (\d+), true, false, sffn::Tile<[^>]*>, true, false, [12]>")


def test_eq_1_prunes_what_it_reads_in_the_gpu_tests(launches):
    """The shapes of test_gpu_prune_in_place.py at M = 8, experts too, and no others; every such kernel of the library is one of those."""
    import tests.test_gpu_prune_in_place as t
    shapes = next(m.args[1] for m in t.test_step.pytestmark if m.name == "parametrize" and m.args[0].startswith("T"))
    calls = [step(call, M, T, D, F, flags=flags) for T, D, F, M in shapes for call in ("step", "forward") for flags in (0, sffn.FLAG_WEIGHTS_PACKED)]
    experts = [(M, D) for M, D in next(m.args[1] for m in t.test_experts.pytestmark if m.name == "parametrize")]
    calls += [step("step", M, 384, D, 256, seg=[0, 64, 64, 256, 384]) for M, D in experts]
    seen = set()
    for call, kernels in zip(calls, launches(calls)):
        found = PRUNES.findall(" ".join(kernels))
        assert bool(found) == (call.split()[3] == "8" and not int(call.split()[7]) & sffn.FLAG_WEIGHTS_PACKED), call
        assert not found or "PrologueUnit" not in kernels[0].split("GemmV2Unit")[0], call          # nothing in front of it
        seen |= {k for k in kernels if PRUNES.search(k)}
    built = {k for k in launches(["kernels"])[0] if PRUNES.search(k)}
    # (soft pruning: the same calls in the other mode)
    assert {k.replace("false, 2>", "false, 1>").replace("<true> ", "<false> ") for k in built} == seen, (built, seen)


def test_no_kernel_for_a_form_that_is_never_chosen(launches):
    """Eq. (4) on tall tiles only beside eqs. (5) and, at M = 8, (3) on tall ones."""
    shared = [k for k in launches(["kernels"])[0] if sorted(tiles(k)) == ["activation", "gradient", "weight"]]
    assert len(shared) >= 40
    for k in shared:
        t = tiles(k)
        assert t["weight"] == 128 or t["gradient"] == "tall" and t["activation"] in (0, "tall") or ", 38, " in k, k


def test_launches_of_the_exact_gpu_tests(launches):
    """The forms that test_gpu_tall_tiles_exact.py names, experts and float32 sums among them, and no 64 tile of an activation or a gradient on either side of its comparisons."""
    from tests.test_gpu_tall_tiles_exact import EXACT
    for T, D, F, seg, want in EXACT:
        sums = sffn.FLAG_LEAN | sffn.FLAG_DW_FP32_ACCUMULATE
        calls = [step("step", 8, T, D, F, seg=seg, flags=0), step("backward", 8, T, D, F, seg=seg), step("backward", 8, T, D, F, seg=seg, flags=sums), step("forward", 8, T, D, F, seg=seg, flags=sums)]
        other = [step("step", 8, b - a, D, F) for a, b in zip(seg, seg[1:]) if b > a] if seg else ["spmm 0 8 %d %d %d" % (T, D, F)] + ["wgrad %d 8 %d %d %d" % (m, T, F, D) for m in (0, 1)]
        got = launches(calls + other)
        whole, back, back_sums = got[:3]
        assert (form(whole, FORWARD), form(back, HEAD), form(whole, TAIL), form(back_sums, HEAD), form(back_sums, TAIL)) == want, (T, D, F, seg)
        assert all(t.get(kind) != 64 for kernels in got for t in map(tiles, kernels) for kind in ("activation", "gradient")), (T, D, F, seg)
        if want[0] is None:
            assert all({"gradient": "tall"} in list(map(tiles, kernels)) for kernels in (whole, back, back_sums))


def test_launches_of_the_gpu_tests_of_results_past_the_caches(launches):
    """No 64 tile of eqs. (3), (7), which would sum in another order, on either side."""
    from tests.test_gpu_results_past import FEW, STEPS, T
    for fp8, M, D, F in STEPS:
        assert 2 * T * D >= 16 << 20 > 2 * FEW * D and 2 * (T - FEW) * D < 16 << 20
        for kernels in launches([step("step", M, n, D, F, fp8) for n in (T, FEW, T - FEW)]):
            units = " ".join(kernels)
            assert ("Vnm8Unit" in units) == (M == 8) and "GTile<1, 3, 4>" not in units and all(t.get("activation") != 64 for t in map(tiles, kernels)), (fp8, M, D, F)
