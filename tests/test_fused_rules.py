"""The rules that pick fused launches, against what is compiled: a rule about speed may never name
a launch that no kernel stands behind, and such a launch fails instead of leaving the state as it
was while the step count goes on.  Host code of the built library, called from a small C++
program; every launch tried here is refused before it reaches the device."""
import subprocess

import pytest

import fused_rules


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    return fused_rules.build(tmp_path_factory.mktemp("rules"))


def test_rules_name_compiled_launches(driver):
    r = subprocess.run([driver], capture_output=True, text=True)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
    seen, fused, _, _ = map(int, r.stdout.split("\n")[-2].split())
    assert seen > 5000 and fused > seen // 4


F64, F32, F16 = 0, 1, 2
AB, AA, TILED, LIST = 0, 1, 2, 3
# (nx, ny, type, layout, force, drag, open, collision (1 TRT, 2 MRT), fluid fraction), whether
# fused launches were the faster side, by 5 % or more, of discs with a force
MEASURED = [
    ((704, 688, F64, AB, 1, 0, 0, 0, 0.1), False), ((704, 688, F64, AB, 1, 0, 0, 0, 0.25), True),
    ((704, 688, F64, AB, 1, 0, 0, 2, 0.1), False), ((704, 688, F64, AB, 1, 0, 0, 2, 0.4), True),
    ((4096, 4096, F64, AB, 1, 0, 0, 2, 0.1), False), ((4096, 4096, F64, AB, 1, 0, 0, 0, 0.25), True),
    ((704, 688, F32, AB, 1, 0, 0, 0, 0.1), True), ((704, 688, F32, AB, 1, 0, 0, 2, 0.1), False),
    ((1504, 1504, F32, AB, 1, 0, 0, 2, 0.1), False), ((1504, 1504, F32, AB, 1, 0, 0, 2, 0.4), True),
    ((1504, 1504, F16, AB, 1, 0, 0, 0, 0.1), False), ((1504, 1504, F16, AB, 1, 0, 0, 0, 0.25), True),
    ((704, 688, F64, AA, 1, 0, 0, 0, 0.1), False), ((4096, 4096, F64, AA, 1, 0, 0, 0, 0.1), False),
    ((4096, 4096, F64, AA, 1, 0, 0, 0, 0.25), True), ((4096, 4096, F64, AA, 1, 0, 0, 2, 0.1), False),
    ((4096, 4096, F64, AA, 1, 0, 0, 2, 0.4), True), ((4096, 4096, F32, AA, 1, 0, 0, 0, 0.1), False),
    ((4096, 4096, F32, AA, 1, 0, 0, 0, 0.25), True), ((4096, 4096, F32, AA, 1, 0, 0, 2, 0.1), False),
    ((1504, 1504, F32, AA, 1, 0, 0, 2, 0.7), True), ((1504, 1504, F16, AA, 1, 0, 0, 0, 0.25), False),
    ((4096, 4096, F16, AA, 1, 0, 0, 0, 0.1), False), ((4096, 4096, F16, AA, 1, 0, 0, 0, 0.4), True),
    ((704, 688, F64, LIST, 1, 0, 0, 2, 0.55), False), ((704, 688, F64, LIST, 1, 0, 0, 2, 0.7), True),
    ((1504, 1504, F64, LIST, 1, 0, 0, 2, 0.4), False), ((1504, 1504, F64, LIST, 1, 0, 0, 0, 0.4), True),
    ((512, 480, F64, LIST, 1, 0, 0, 1, 0.3), False), ((512, 480, F64, LIST, 1, 1, 0, 0, 0.3), False),
    ((512, 480, F64, LIST, 1, 0, 0, 2, 0.6), False), ((512, 480, F64, LIST, 1, 0, 0, 1, 0.6), True),
    ((4096, 4096, F64, TILED, 1, 0, 0, 0, 0.25), False), ((4096, 4096, F64, TILED, 1, 0, 0, 0, 0.4), True),
]


# the same with the steps to go, and the steps of the next launch: two or three steps a launch where
# single steps were faster
TAILS = [
    ((4096, 4096, F32, TILED, 1, 0, 0, 0, 0.97, 2), 1), ((4096, 4096, F64, TILED, 1, 0, 0, 0, 0.4, 3), 1),
    ((704, 688, F32, TILED, 1, 0, 0, 0, 0.7, 10), 4), ((704, 688, F32, TILED, 1, 0, 0, 0, 0.7, 2), 1),
    ((1504, 1504, F64, LIST, 1, 0, 0, 0, 0.4, 3), 1), ((4096, 4096, F64, LIST, 1, 0, 0, 0, 0.7, 2), 2),
    ((4096, 4096, F16, AB, 1, 0, 0, 0, 0.97, 2), 1), ((4096, 4096, F64, AB, 1, 0, 0, 0, 0.25, 5), 4),
    ((4096, 4096, F64, AB, 0, 0, 0, 0, 1.0, 5), 5), ((4096, 4096, F64, AB, 0, 0, 0, 0, 1.0, 2), 2),
    ((4096, 4096, F32, AB, 1, 0, 0, 0, 0.1, 2), 1), ((256, 64, F32, LIST, 1, 0, 0, 0, 0.97, 2), 2),
    ((4096, 4096, F32, AB, 1, 0, 0, 0, 0.97, 100), 8),
    ((240, 160, F64, AB, 0, 0, 1, 0, 1.0, 2), 1), ((240, 160, F64, LIST, 0, 0, 1, 2, 1.0, 3), 1),
    ((2048, 1536, F32, LIST, 1, 1, 0, 2, 0.9, 5), 1), ((4096, 2048, F16, AB, 0, 0, 0, 2, 1.0, 5), 1),
    ((4096, 2048, F16, TILED, 0, 0, 1, 0, 1.0, 5), 1), ((512, 480, F32, AB, 0, 0, 1, 2, 1.0, 2), 1),
    ((2048, 2048, F16, AB, 0, 0, 0, 0, 1.0, 2), 2),
]


# D3Q19: (nx, ny, nz, type, AA, force, fluid fraction), whether pairs were the faster side
PAIRS = [
    ((96, 80, 64, F32, 0, 1, 0.1), 0), ((96, 80, 64, F32, 0, 1, 0.6), 1),
    ((96, 80, 64, F64, 0, 1, 0.1), 1), ((128, 128, 128, F32, 0, 1, 0.1), 1),
    ((96, 80, 64, F64, 1, 1, 0.1), 0), ((96, 80, 64, F32, 1, 1, 0.6), 0),
    ((128, 128, 128, F64, 1, 1, 0.3), 0), ((128, 128, 128, F64, 1, 1, 0.6), 1),
    ((128, 128, 128, F32, 1, 1, 0.1), 0), ((256, 256, 128, F64, 1, 1, 0.1), 0),
    ((256, 256, 128, F32, 1, 1, 0.1), 0), ((256, 256, 128, F32, 1, 1, 0.6), 1),
    ((256, 256, 256, F32, 0, 0, 1.0), 1), ((96, 80, 64, F32, 1, 0, 1.0), 1),
]


def test_faster_side_is_taken(driver):
    got = fused_rules.ask(driver, [(*c, 100) for c, _ in MEASURED])
    wrong = [(c, steps) for (c, fused), (steps, *_) in zip(MEASURED, got) if (steps > 1) != fused]
    assert not wrong


def test_short_rests_take_the_faster_side(driver):
    got = fused_rules.ask(driver, [c for c, _ in TAILS])
    assert [(c, g[1]) for (c, _), g in zip(TAILS, got)] == TAILS


def test_pairs_take_the_faster_side(driver):
    got = fused_rules.ask(driver, [c for c, _ in PAIRS], "3")
    assert [(c, g[0]) for (c, _), g in zip(PAIRS, got)] == PAIRS


def test_reverse_steps_take_the_faster_side(driver):
    """(nx, ny, type, fluid fraction): whether squares were faster than single reverse steps."""
    cases = [((200, 60, F64, 0.2), True), ((400, 150, F32, 0.2), True), ((1024, 256, F32, 0.2), True),
             ((1024, 256, F64, 1.0), True), ((1024, 256, F64, 0.2), False), ((900, 900, F32, 1.0), True),
             ((900, 900, F32, 0.6), False), ((900, 900, F32, 0.2), False), ((900, 900, F64, 1.0), False)]
    got = fused_rules.ask(driver, [c for c, _ in cases], "adjoint")
    assert [(c, g[0] > 1) for (c, _), g in zip(cases, got)] == cases
