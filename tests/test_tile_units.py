"""The numbering of the persistent FFN kernels' units (csrc/rules.hpp, compiled here with g++ and walked as the kernels walk
them): every block of output columns of every item and slice has one workgroup, whatever the numbers are."""
import os
import random
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def units(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("units") / "units")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", os.path.join(HERE, "units_main.cpp"), "-o", exe], check=True)

    def run(cases):
        text = "".join(" ".join(map(str, c)) + "\n" for c in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        return [tuple(int(v) for v in line.split()) for line in out if line]
    return run


def draw(rng, f32):
    items = rng.choice([1, 2, 3, 7, 8, 31, 32, 33, 64, rng.randint(1, 700)])
    longs = rng.choice([0, items, min(items, 32), rng.randint(0, items)]) if f32 else 0
    return (f32, rng.randint(0, 1), items, longs, rng.choice([1, 2, 3, 5, 8, 11, 16, 32]), 1 if f32 else rng.choice([1, 1, 2, 3]),
            rng.randint(1, 20), rng.randint(0, 1))


def test_every_unit_has_one_workgroup(units):
    rng = random.Random(7)
    cases = [draw(rng, f32) for f32 in (0, 1) for _ in range(1500)]
    cut = uncut = 0
    for case, (wrong, whole, halves, most, *_) in zip(cases, units(cases)):
        f32, gate_up, items, _, blocks, ksplit, steps, tail = case
        total = items * blocks * ksplit
        assert wrong == 0 and most <= 1, case
        if f32 or tail:
            assert 2 * whole + halves == 2 * total, case
        cut += halves > 0
        uncut += halves == 0 and not f32
    assert cut > 300 and uncut > 300


def test_halves_behind_whole_units_only_where_they_pay(units):
    """A remainder of up to half of an XCD's workgroups; gate/up from five k steps on, down always.  With no whole units
    before, always."""
    for rest in range(1, 32):
        for rounds in (0, 1, 3):
            items = 8 * (32 * rounds + rest)
            cases = [(0, gate_up, items, 0, 1, 1, steps, 1) for gate_up in (0, 1) for steps in (1, 3, 4, 5, 30)]
            for case, (_, whole, halves, *_) in zip(cases, units(cases)):
                pays = rest <= 16 and (rounds == 0 or case[1] == 0 or case[6] >= 5)
                assert (whole, halves) == ((256 * rounds, 16 * rest) if pays else (items, 0)), case


def test_workgroups_with_a_long_unit_get_a_further_one_last(units):
    """Every XCD has an eighth of the long units and of the others; the first round takes the long ones and the second goes the other
    way round the workgroups."""
    cases = [(1, 1, 8 * (longs + others), 8 * longs, 1, 1, 8, 1) for longs in range(1, 33) for others in (32 - longs, 48 - longs, 64 - longs)]
    for case, (wrong, whole, _, _, both) in zip(cases, units(cases)):
        longs, second = case[3] // 8, case[2] // 8 - 32
        assert (wrong, whole) == (0, case[2])
        if longs < 32:
            assert both == 8 * max(0, longs + second - 32), case
