"""The host's plan of a similarity estimation (csrc/similarity_plan.hpp, compiled here with g++): a call checks its
workspace against the largest group of batches that it launches, so the layouts of all smaller groups, the last one of
a call among them, have to fit into the same bytes."""
import math
import os
import random
import subprocess

import pytest

from paper_2602_07616_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))
METRICS = (0, B.SERE_FLAG_SIM_COSINE, B.SERE_FLAG_SIM_CKA_LINEAR)


@pytest.fixture(scope="module")
def layouts(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("simplan") / "plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", os.path.join(HERE, "similarity_plan_main.cpp"), "-o", exe],
                   check=True)

    def run(cases):
        out = subprocess.run([exe], input="".join("%d %d %d %d %d %d %d\n" % c for c in cases), capture_output=True, text=True,
                             check=True).stdout.split("\n")
        return [[tuple(int(v) for v in g.split()) for g in line.split(";") if g] for line in out if line]
    return run


def draws(count, seed):
    rng = random.Random(seed)
    log_int = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    # the sizes at which a last group of 15 batches once needed more than a group of 16, for all metrics
    cases = [(dtype, 768, M, 64, 7, f, 31) for dtype in (B.SERE_F32, B.SERE_BF16) for M in range(120, 130) for f in METRICS]
    for _ in range(count):
        f = rng.choice(METRICS)
        cases.append((rng.choice((B.SERE_F32, B.SERE_BF16)), 64 * log_int(1, 64), log_int(1, 256), 64 * log_int(1, 224),
                      log_int(4 if f == B.SERE_FLAG_SIM_CKA_LINEAR else 1, 400), f, rng.choice((1, 2, 3, 7, 31, 31, 31))))
    return cases


def test_no_group_needs_more_than_a_larger_one(layouts):
    cases = draws(6000, 11)
    grouped = 0
    for case, groups in zip(cases, layouts(cases)):
        totals = [g[0] for g in groups]
        assert totals == sorted(totals), (case, totals)
        grouped += len(groups) > 1
    assert grouped > 1000      # otherwise the draw would say nothing


def test_layers_of_every_size_are_grouped(layouts):
    cases = [(B.SERE_BF16, 256, 16, 128 * k, 20, f, 64) for k in (1, 5, 6, 20) for f in METRICS]   # 3, 7.9, 9.4, 31 MB
    cases += [(B.SERE_F32, 256, 16, 128 * k, 20, f, 64) for k in (1, 2, 3, 10) for f in METRICS]   # 6, 13, 19, 63 MB
    for case, groups in zip(cases, layouts(cases)):
        assert len(groups) == 12, case


def test_plans_of_groups_can_be_run(layouts):
    """Items hold every row of a group, longer items than the decode kernels take go to the persistent ones, and the
    work list and the partial Gram matrices fit their places."""
    cases = draws(2000, 12)
    for case, groups in zip(cases, layouts(cases)):
        M, n, blocks = case[2], case[4], case[3] // 64
        for g, (_, items, rows, tile_gu, tile_dn, ksplit, splits, _, item_bytes, part_bytes, *_) in enumerate(groups, 1):
            assert M * items * 4 <= item_bytes and g * splits * (M * M + 96) * 8 <= part_bytes, case
            assert (items - 1) * rows < n * g <= items * rows, case
            assert rows == 32 or (tile_gu and tile_dn), case
            assert (ksplit - 1) * -(-blocks // ksplit) < blocks, case


def test_sums_of_alignment_fit_where_h_and_y_were(layouts):
    """The blocks of row sums of every expert's Gram matrix and the summands of every pair, 8 bytes each; 512 tokens and
    d_m = 64 have the least room."""
    cases = [(dtype, 64 * k, M, 64, n, B.SERE_FLAG_SIM_CKA_LINEAR, 3) for dtype in (B.SERE_F32, B.SERE_BF16) for k in (1, 2, 20)
             for M in (1, 2, 16, 17, 100, 256) for n in (4, 5, 16, 47, 48, 49, 100, 511, 512)]
    cases += [c for c in draws(6000, 16) if c[5] == B.SERE_FLAG_SIM_CKA_LINEAR]
    several = 0
    for case, groups in zip(cases, layouts(cases)):
        M, n = case[2], case[4]
        for g, (*_, y_bytes, h_bytes, parts, blocks, _, _) in enumerate(groups, 1):
            assert (blocks - 1) * (16 if n <= 48 else 32) < n <= blocks * (16 if n <= 48 else 32), case
            assert M * g * blocks * n * 8 <= h_bytes, case
            assert 1 <= parts <= 9 and (parts == 1 or g * parts * M * M * 8 <= y_bytes), case
            several += parts > 1
    assert several > 1000


def test_the_room_does_not_depend_on_the_number_of_batches(layouts):
    cases = draws(1500, 14)
    for case, few, many in zip(cases, layouts(cases), layouts([c[:6] + (64,) for c in cases])):
        assert [g[0] for g in few] == [g[0] for g in many][:len(few)], case


def test_sums_do_not_depend_on_the_group(layouts):
    """What decides the order of an expert's sums (the kernels, the slices of d_m) is the same for all groups of a call."""
    cases = draws(3000, 13)
    items = set()
    for case, groups in zip(cases, layouts(cases)):
        assert len({g[3:6] for g in groups}) == 1, case
        items.add(len({g[2] for g in groups}))
    assert max(items) > 3      # the item size does follow the group


def test_choice_of_the_gram_kernel(layouts):
    """Staged: Frobenius metric, outputs in one slice (by the slices that the plan takes, not by how many the layer's width
    would allow), and sizes at which it was measured to be the faster one."""
    cases = [c for c in draws(6000, 15)]
    wide = 0
    for case, groups in zip(cases, layouts(cases)):
        M, length = case[2], case[1] * case[4]
        for g, layout in enumerate(groups, 1):
            pays = (64 < M <= 128 and g * length >= 40960) or (M > 192 and g * length % 524288 == 0)
            assert layout[7] == (case[5] == 0 and layout[5] == 1 and pays), (case, g)
            wide += layout[7] and case[0] == B.SERE_BF16 and case[3] > 2048
    assert wide > 50


def test_gpu_cases_of_the_wide_gate_up_kernel_take_it(layouts):
    from . import test_gpu_wide_gate_up as gpu
    for case, groups in zip(gpu.CASES, layouts([(B.SERE_BF16, dh, M, dm, n, 0, b) for M, dh, dm, n, b in gpu.CASES])):
        assert (len(groups), groups[-1][2], groups[-1][10]) == (case[4], 256, 1), case


def test_gpu_cases_of_up_to_64_experts_run_the_loop_of_their_kernel(layouts):
    """More than one turn and a part of one, for every number of tiles and both metrics, and in groups of batches."""
    from . import test_gpu_pair_gram_few as gpu
    for flag in (0, B.SERE_FLAG_SIM_COSINE):
        tiles, grouped = set(), set()
        for (M, dh, n, batches, dtype, dm), groups in zip(gpu.LONG, layouts([(dtype, dh, M, dm, n, flag, b) for M, dh, n, b, dtype, dm in gpu.LONG])):
            *_, steps, turn = groups[-1]
            assert steps > turn and steps % turn != 0 and len(groups) == batches, (M, dh, n)
            tiles.add(-(-M // 16))
            grouped |= {-(-M // 16)} if batches > 1 else set()
        assert tiles == {1, 2, 3, 4} and grouped >= {3, 4}


def test_gpu_cases_of_alignment_are_grouped(layouts):
    from . import test_gpu_cka as gpu
    for case, groups in gpu.GROUPED.items():
        M, dh, n, batches, dtype, dm = case
        assert case in gpu.CASES
        assert len(layouts([(dtype, dh, M, dm, n, B.SERE_FLAG_SIM_CKA_LINEAR, batches)])[0]) == groups, case
    assert {n > 48 for _, _, n, _, _, _ in gpu.GROUPED} == {False, True}


def test_gpu_cases_of_the_gram_kernels_reach_them(layouts):
    from . import test_gpu_pair_gram as gpu
    for cases, staged in ((gpu.BLOCKS, 0), (gpu.STAGED, 1)):
        plans = layouts([(c[4], c[1], c[0], (*c, 64)[5], c[2], 0, c[3]) for c in cases])
        for case, groups in zip(cases, plans):
            assert groups[-1][7] == staged, case
