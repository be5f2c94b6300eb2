"""The host-side rules that choose a contraction's output tile (kernels.hpp), against measured times of every tile (tests/golden/tile_times.txt): over
the calls of a group, what the rules choose takes at most 4 % longer than the best tile of each call (where not said otherwise), and no call a third longer.
The rules that have a step's contractions share launches, against whole steps timed both ways (tests/golden/step_times.txt, router_times.txt)."""
import math
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
TILES = (256, 128, 64)


def golden(name):
    return [line.strip().split(" | ") for line in open(os.path.join(HERE, "golden", name)) if not line.startswith("#")]


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    """calls -> the lines that the rules print for them"""
    exe = str(tmp_path_factory.mktemp("tiles") / "tile_rules")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", os.path.join(HERE, "tile_rules.cpp"), "-o", exe], check=True)
    return lambda calls: subprocess.run([exe], input="\n".join(calls), capture_output=True, text=True, check=True).stdout.split("\n")


@pytest.fixture(scope="module")
def chosen(rules):
    """[(call, its measured times, what the rules print for it)]"""
    calls = golden("tile_times.txt")
    out = rules([c[0] for c in calls])
    times = [{int(t.split(":")[0]): float(t.split(":")[1]) for t in c[1].split()} if c[0].startswith("split") else
             dict(zip((1, 0), map(float, c[1].split()))) if c[0].startswith("rowx") else
             {t.split()[0]: {e: float(v) for e, v in zip(TILES, t.split()[1:]) if v != "-"} for t in c[1:]} for c in calls]
    return [(c[0].split(), t, [int(v) for v in o.split()]) for c, t, o in zip(calls, times, out)]


def check(rows, most=1.34, total=1.04):
    """rows: (times by tile, tile chosen)"""
    assert len(rows) >= 2
    for times, tile in rows:
        assert times[tile] <= most * min(times.values()), (times, tile)
    assert sum(times[tile] for times, tile in rows) <= total * sum(min(times.values()) for times, _ in rows), rows


def steps(chosen, fp8, grouped, tall=False):
    """Calls of the step; the tiles are those of launches of their own, also where the rules have the step's contractions share launches."""
    return [(t, o) for c, t, o in chosen if c[0] == "step" and c[1] == str(int(fp8)) and (c[5] != "1") == grouped and (c[2] == "64") == tall]


@pytest.mark.parametrize("tall", [False, True])
def test_tiles_of_the_epilogue_contractions(chosen, tall):
    rows = steps(chosen, False, False, tall)
    check([(t["eq1"], o[0]) for t, o in rows])
    check([(t["eq4"], o[1]) for t, o in rows if "eq4" in t])


@pytest.mark.parametrize("M", [(8,), (16, 32), (64,)])
@pytest.mark.parametrize("fp8", [False, True])
def test_tiles_of_the_epilogue_contractions_by_type_and_width(chosen, fp8, M):
    """Eqs. (1), (4) on tiles of 256 and 128 (M = 64: 256 x 128): no call more than 5 % above the better one, 2 % in total (two runs of one tile differ by 1 - 2 %)."""
    rows = [(t, o) for c, t, o in chosen if c[0] == "step" and c[1] == str(int(fp8)) and int(c[2]) in M and c[5] == "1"]
    big = lambda t: {e: t[e] for e in (256, 128) if e in t}
    check([(big(t["eq1"]), o[0]) for t, o in rows if o[0] != 64], 1.05, 1.02)
    check([(big(t["eq4"]), o[1]) for t, o in rows if "eq4" in t and o[1] != 64], 1.05, 1.02)


def test_tiles_of_the_plain_contractions(chosen):
    rows = [(t["bf16"], o[0]) for c, t, o in chosen if c[0] == "plain"]
    check([(t, tile) for t, tile in rows if tile in t], 1.2)


@pytest.mark.parametrize("fp8", [False, True])
def test_tiles_of_grouped_steps(chosen, fp8):
    rows = steps(chosen, fp8, True)
    check([(t["eq1"], o[0]) for t, o in rows])
    check([(t["eq4"], o[1]) for t, o in rows])
    # (one call of the list has experts whose weights do not stay in a cache for a second round of small tiles: 396 us for 320)
    for v in (2, 5):
        check([(t["eq3"], o[v]) for t, o in rows if "eq3" in t and o[v] != 64], total=1.04)


@pytest.mark.parametrize("fp8", [False, True])
def test_tiles_of_the_activation_contractions(chosen, fp8):
    """Eqs. (3), (7) at M = 8 in launches of their own, where the step's contractions have such launches and in the forward call of a step whose contractions share them."""
    for v in (2, 5):
        check([(t["eq3"], o[v]) for c, t, o in chosen if c[0] == "step" and c[1] == str(int(fp8)) and "eq3" in t and o[v] in t["eq3"]], 1.3, 1.06)


def test_tiles_of_the_routers_contractions(chosen):
    rows = [(t, o[0]) for c, t, o in chosen if c[0] == "router"]
    check([(t["eq1"], tile) for t, tile in rows])
    check([(t["eq4"], tile) for t, tile in rows])


def test_forward_calls_read_x_as_it_is(chosen):
    """Eq. (1) on row-major X where that is faster than a copy in blocks: no call 4 % above the better form, 1 % in total."""
    check([(t, o[0]) for c, t, o in chosen if c[0] == "rowx" and o[0] >= 0], 1.04, 1.01)


def test_splits_of_the_activation_contractions(chosen):
    """No slower than undivided, and all of them together 5 % faster."""
    rows = [(t, min(t, key=lambda n: abs(n - o[0]))) for c, t, o in chosen if c[0] == "split"]       # (the nearest number that was measured)
    assert len(rows) >= 8 and all(t[n] <= 1.04 * t[1] for t, n in rows), rows
    assert sum(t[n] for t, n in rows) <= 0.95 * sum(t[1] for t, _ in rows), rows


def test_shared_launches_of_the_routers_step(rules):
    """Where the router's step shares launches it is faster, by 5 % and more over all calls, and no call 4 % slower."""
    calls = golden("router_times.txt")
    rows = [tuple(map(float, t.split())) for (c, t), line in zip(calls, rules(["shares " + c for c, _ in calls])) if line.split()[0] == "1"]
    assert len(rows) >= 30 and all(shared <= 1.04 * apart for shared, apart in rows), rows
    assert sum(math.log(shared / apart) for shared, apart in rows) <= -0.05 * len(rows), rows


def test_routes_of_the_gpu_tests(rules):
    """tests/test_gpu_tiles.py compares the routes that it means to: a call that reads X as it is with one that copies it, or with the oracle; the router's shared launches."""
    from tests.test_gpu_tiles import FORWARD_CALLS, ROUTER_CALLS
    offsets = [seg or [0, T] for _, T, _, _, seg, *_ in FORWARD_CALLS]
    lines = rules(["forward %d %d %d %d %s" % (M, D, F, len(o) - 1, " ".join(map(str, o))) for (M, _, D, F, *_), o in zip(FORWARD_CALLS, offsets)])
    for call, line in zip(FORWARD_CALLS, lines):
        assert line.split() == [str(v) for v in call[5:]], (call, line)
    for call, line in zip(ROUTER_CALLS, rules(["shares %d %d %d %d" % (M, D, F, T) for M, T, D, F, _ in ROUTER_CALLS])):
        assert line.split() == ["1", str(call[4])], (call, line)


@pytest.mark.parametrize("what,mean,most", [("step", 0.0025, 0.15), ("calls", 0.0025, 0.08), ("forward", 0.0075, 0.20)])
def test_shared_launches_of_the_step(rules, what, mean, most):
    """The form that is chosen takes 0.25 % longer than the better one on average, for the whole step as for its calls of one pass each (two runs of one form differ by
    1 - 2 %), no more than 1 % in any group of calls, and 4 % in one call of 40; a forward call that loses a split (StepTiles) up to a fifth."""
    calls = golden("step_times.txt")
    assert len(calls) >= 480
    losses = {}
    for (call, *times), share in zip(calls, rules(["share " + c[0] for c in calls])):
        shared, apart = next(map(float, t.split()[1:]) for t in times if t.split()[0] == what)
        losses.setdefault(tuple(call.split()[:2]) + (call.split()[4] != "1",), []).append(math.log((shared if share == "1" else apart) / min(shared, apart)))
    every = [x for group in losses.values() for x in group]
    assert sum(every) <= mean * len(every) and max(every) <= most and sum(x > 0.04 for x in every) <= len(every) / 40, (sum(every) / len(every), max(every))
    assert what == "forward" or all(sum(group) <= 0.01 * len(group) for group in losses.values()), {k: sum(v) / len(v) for k, v in losses.items()}
