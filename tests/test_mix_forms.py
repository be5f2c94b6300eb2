"""The rule that puts contractions of a shared launch on tall tiles (mix_plan.hpp)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("forms") / "mix_forms")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", os.path.join(HERE, "mix_forms.cpp"), "-o", exe], check=True)
    return lambda calls: [line.split() for line in subprocess.run([exe], input="\n".join(calls), capture_output=True, text=True, check=True).stdout.strip().split("\n")]


def test_a_launch_played_through(forms):
    """64 slots on 32 CUs: 32 tiles alone; 64 side by side; 65 in two rounds, the last one alone; classes in their order."""
    got = [float(r[0]) for r in forms(["play 64 32 10 0.5 0 1 1 0 1 1", "play 64 64 10 0.5 0 1 1 0 1 1", "play 64 65 10 0.5 0 1 1 0 1 1", "play 64 64 10 1 64 4 1 64 1 1", "play 32 33 8 1 0 1 1 0 1 1"])]
    assert got == pytest.approx([5.0, 10.0, 15.0, 15.0, 16.0], rel=1e-3)


def test_forms_of_the_gpu_tests(forms):
    from tests.test_gpu_tall_tiles import FP8, PLAIN, WIDE
    calls = [(0, 8, *c) for c in PLAIN] + [(0, *c) for c in WIDE] + [(1, *c) for c in FP8]
    for (fp8, M, T, D, F, want), line in zip(calls, forms(["%d %d %d %d %d" % (fp8, M, D, F, T) for fp8, M, T, D, F, _ in calls])):
        assert line == ["1"] + [str(v) for v in want], (fp8, M, T, D, F, line)


def test_every_form_is_one_that_is_built(forms):
    """Eq. (4) on tall tiles only with the others; nothing where every tile has a CU, all that there is past 16 rounds."""
    calls = [(fp8, M, D, F, T) for fp8 in (0, 1) for M in (8, 16, 64) for T in (64, 320, 1088, 2240, 9024) for D in (384, 1152, 2304, 4608) for F in (2048, 4096, 14336)]
    for call, line in zip(calls, forms(["%d %d %d %d %d" % c for c in calls])):
        mix, *f = map(int, line)
        fwd, head, tail = f
        assert not (fwd & 4) or fwd == (7 if call[1] == 8 else 6), (call, line)
        assert head in (0, 2, 6) and tail in ((0, 1, 2, 3) if call[1] == 8 else (0, 2)), (call, line)
        assert call[1] != 64 or not (fwd | head) & 4, (call, line)


def test_launches_of_their_own_of_the_gpu_tests(forms):
    from tests.test_gpu_tall_tiles import ALONE_ACTIVATION, ALONE_GRADIENT
    for call, line in zip(ALONE_ACTIVATION, forms(["alone %d %d %d %d" % c for c in ALONE_ACTIVATION])):
        assert line[0] in ("128", "256") and line[1] == "1", (call, line)
    for call, line in zip(ALONE_GRADIENT, forms(["alone %d %d %d %d" % c for c in ALONE_GRADIENT])):
        assert line[2] in ("128", "256") and line[3] == "1", (call, line)
    # codes: gradients never; no activation contraction whose tiles all have a CU
    small = [(fp8, T, 512, F) for fp8 in (0, 1) for T in (64, 512, 2048) for F in (512, 4096)]
    assert all(line[1] == "0" and line[3] == "0" for line in forms(["alone %d %d %d %d" % c for c in small]))


def test_streamed_steps_of_the_gpu_tests(forms):
    from tests.test_gpu_tall_tiles import STREAMED
    assert [r[0] for r in forms(["streams %d %d %d" % c for c in STREAMED])] == ["1"] * len(STREAMED)
    assert [r[0] for r in forms(["streams 4096 1024 4096", "streams 8192 8192 28672"])] == ["0", "1"]
