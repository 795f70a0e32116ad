"""The numbering of the persistent FFN kernels' units (csrc/rules.hpp, compiled here with g++ and walked as the kernels walk
them): every block of output columns of every item and slice has one workgroup, whatever the numbers are."""
import os
import random
import subprocess

import pytest

from paper_2602_07616_amd import binding as B
from . import test_gpu_f32_units as gpu_f32, test_gpu_tile_halves as gpu

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


@pytest.fixture(scope="module")
def launches(tmp_path_factory, units):
    """(plan, {launch: (kernel, whole units, halves)}) of bf16 calls whose experts all have all tokens."""
    exe = str(tmp_path_factory.mktemp("plan") / "plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", os.path.join(HERE, "plan_main.cpp"), "-o", exe], check=True)

    def run(cases):
        text = "".join(f"{B.SERE_BF16} {T} {dh} {M} {M} {dm} {sh} {M} 0.0 1\n" for T, dh, M, dm, sh in cases)
        out = subprocess.run([exe, "call"], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        plans = [tuple(int(v) for v in line.split()) for line in out if line]
        which, asked, results = [], [], [(plan, {}) for plan in plans]
        for i, ((T, dh, M, dm, sh), (rows, tile_gu, tile_dn, ksplit, wide)) in enumerate(zip(cases, plans)):
            items, short = (M + sh) * -(-T // rows), rows >= 192 and not wide
            assert not (wide and tile_gu), "not cut"
            if tile_gu:
                out = 64 if short else 128
                asked.append((0, 1, items, 0, -(-dm // out), 1, dh // 64, int(not 0 < dm % out <= out // 2)))
                which.append((i, "gate_up", ("gate_up", rows, 0)))
            if tile_dn:
                two = int(dm >= 4096)
                out = 128 if short or (two and rows == 128) else 256
                asked.append((0, 0, items, 0, -(-dh // out), ksplit, -(-(dm // 64) // ksplit), int(not 0 < dh % out <= out // 2)))
                which.append((i, "down", ("down", rows, two)))
        for (i, launch, kernel), (_, whole, halves, *_) in zip(which, units(asked)):
            results[i][1][launch] = kernel, whole, halves
        return results
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


def test_gpu_cases_have_the_units_that_they_are_there_for(launches):
    reached = set()
    for (case, (rows, *want)), (plan, got) in zip(gpu.CASES.items(), launches(list(gpu.CASES))):
        assert plan[0] == rows, case
        assert [got[l][1:] if l in got else None for l in ("gate_up", "down")] == want, case
        # more units than workgroups and halves: at least an XCD's workgroups have both
        reached |= {kernel for kernel, whole, halves in got.values() if whole >= 256 and halves > 0}
    assert reached == {("gate_up", r, 0) for r in (32, 64, 96, 128, 160, 192, 256)} | {("down", r, 0) for r in (32, 64, 96, 128, 160, 192, 256)} | \
        {("down", r, 1) for r in (32, 64, 128)}


def test_gpu_pairs_are_cut_and_not_cut(launches):
    for (dh, M, dm, sh), (launch, cut, whole) in gpu.PAIRS.items():
        (p, a), (q, b) = launches([(T, dh, M, dm, sh) for T in (cut, whole)])
        assert p[1:] == q[1:], (dh, M, dm, sh)               # the same kernels and slices; other item sizes
        assert a[launch][1] >= 256 and a[launch][2] > 0 and b[launch][1] > 0 and b[launch][2] == 0, (dh, M, dm, sh)


def test_gpu_cases_of_fp32_layers_have_their_items():
    """Items, those of more than 16 rows, and whether these come first: more than a round of gate/up units."""
    import oracle
    from paper_2602_07616_amd import workloads as wk
    from . import pins
    for case, want in gpu_f32.CASES.items():
        T, dh, M, K, dm, n_sh, S, rho = case
        seed = gpu_f32.seed(case)
        wl = wk.make_workload(wk.custom_spec("units", wk.F32, dh, M, K, dm, n_sh, T, seed, weight_std=0.02, calib_batches=1, calib_tokens=4))
        ref = oracle.route(wl.hidden, wl.router_w, wk.F32, K, pins.rand_sim(seed, M), S, rho)
        counts = [int(n) for n in ref.count_after if n] + [T] * n_sh
        items = [min(32, n - 32 * j) for n in counts for j in range(-(-n // 32))]
        assert (len(items), sum(n > 16 for n in items), len(items) * -(-dm // 64) > 256) == want, case
