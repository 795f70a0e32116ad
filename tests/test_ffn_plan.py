"""The host's choice of FFN kernels (csrc/ffn_plan.hpp, compiled here with g++): over the range of
layers and batches the library accepts, every plan must be one that the kernels can run."""
import math
import os
import random
import subprocess

import pytest

from paper_2602_07616_amd import binding as B, workloads as wk
from . import test_gpu_ffn_tile as gpu, test_gpu_nonfinite as gpu_nonfinite, test_gpu_wide_gate_up as gpu_wide

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", os.path.join(HERE, "plan_main.cpp"), "-o", exe], check=True)

    def run(cases, *args):
        text = "".join(" ".join(map(str, c)) + "\n" for c in cases)
        out = subprocess.run([exe, *args], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        return [tuple(int(v) for v in line.split()) for line in out if line]
    return run


def shape(T, dh, M, K, dm, sh, kept):
    experts = max(1.0, M * (1.0 - (1.0 - kept / M) ** T))
    rows = T * K / experts
    return (dh, dm, sh, T, experts, rows, 1.5 * math.sqrt(rows) if K < M else 0.0, T * K / M, int(dm >= 4096), (dm + 2047) // 2048)


def test_every_plan_can_be_run(plans):
    rng = random.Random(5)
    cases, layers = [], []
    log_int = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    for _ in range(4000):
        M = log_int(1, 256)
        K = rng.randint(1, min(M, 12))
        layer = (log_int(1, 65536), 64 * log_int(1, 1024), M, K, 64 * log_int(1, 4096), rng.choice([0, 0, 1, 4, 16]), rng.randint(1, K))
        layers.append(layer)
        cases.append(shape(*layer))
    for layer, case, (rows, tile_gu, tile_dn, ksplit, wide) in zip(layers, cases, plans(cases)):
        blocks, split, max_ksplit = layer[4] // 64, case[8], case[9]
        assert rows in ((32, 64, 128) if split else (32, 64, 96, 128, 160, 192, 256)), layer
        if not (tile_gu and tile_dn):
            assert rows == 32, layer               # the other kernels take items of at most 32 rows
        assert 1 <= ksplit <= max_ksplit, layer
        assert (ksplit - 1) * -(-blocks // ksplit) < blocks, layer   # no slice of d_m is empty
        if not tile_dn:
            assert ksplit == max_ksplit, layer
        assert not wide or (rows == 256 and tile_gu and not split), layer


def test_choices_on_the_layers_the_rule_was_measured_on(plans):
    """Qwen3 shape: the persistent kernels from 8 rows per expert on, longer items with more rows."""
    got = plans([shape(T, 2048, 128, 8, 768, 0, 2) for T in (1, 32, 64, 128, 512, 1024, 2048, 3072)])
    assert [g[1] for g in got] == [0, 0, 0, 1, 1, 1, 1, 1]
    assert [g[0] for g in got] == [32, 32, 32, 32, 64, 96, 160, 256]


def test_fp32_plans(plans):
    """fp32 layers: items of 32 rows, no slices; batches of more than 8 tokens run on the persistent kernels."""
    layers = [(T, dh, 17, 4, dm, sh, 4) for T in (1, 2, 8, 9, 96, 4096) for dh in (64, 256, 1472) for dm in (64, 704) for sh in (0, 2)]
    cases = [shape(*layer)[:9] + (1,) for layer in layers]
    for layer, (rows, tile_gu, tile_dn, ksplit, wide) in zip(layers, plans(cases, "f32")):
        assert (rows, ksplit, wide) == (32, 1, 0) and tile_gu == tile_dn, layer
        assert tile_gu or layer[0] <= 8, layer


def call(dtype, T, dh, M, K, dm, sh, S, rho=0.0):
    return (dtype, T, dh, M, K, dm, sh, S, rho, 1)


# (T, d_h, M, d_m, shared) with K = M: the gate/up units of 256 weight rows took 4 % to 6 % less time for the whole call, or more
WIDE_IS_FASTER = [(1000, 2048, 5, 1536, 0), (1000, 512, 8, 2560, 1), (1000, 4096, 3, 1408, 1), (1500, 2048, 8, 512, 1),
                  (397, 1536, 3, 3584, 1), (200, 1024, 5, 3584, 1), (1137, 384, 10, 1216, 0)]
WIDE_IS_SLOWER = [(1500, 1024, 8, 1024, 0), (873, 1088, 10, 1216, 0), (2426, 384, 2, 3264, 1), (459, 512, 14, 1600, 1),
                  (1789, 576, 4, 1728, 0), (1475, 384, 3, 2624, 0)]


def test_wide_gate_up_units_only_where_their_rounds_are_shorter(plans):
    for layers, wide in ((WIDE_IS_FASTER, 1), (WIDE_IS_SLOWER, 0)):
        for reroute, S in ((0, 1), (1, 1)):
            cases = [(B.SERE_BF16, T, dh, M, M, dm, sh, S, 0.0, reroute) for T, dh, M, dm, sh in layers]
            assert [p[0] for p in plans(cases, "call")] == [256] * len(cases)
            assert [p[4] for p in plans(cases, "call")] == [wide] * len(cases), (layers, reroute)


def test_pairs_of_the_wide_kernel_and_the_narrow_one(plans):
    """What the comparison of their bits takes for granted: the longer batch by units of 128, all else alike."""
    for (dh, M, dm, sh), batches in gpu_wide.PAIRS:
        few, many = plans([(B.SERE_BF16, T, dh, M, M, dm, sh, M, 0.0, 0) for T in batches], "call")
        assert (few[4], many[4]) == (1, 0) and few[:4] == many[:4], (dh, M, dm, sh)


def test_gpu_cases_get_the_plans_they_are_there_for(plans):
    for S in (lambda K: 1, lambda K: K):         # both settings that the GPU test runs
        got = plans([call(B.SERE_BF16, *c, S(c[3])) for c in gpu.CASES], "call")
        assert dict(zip(gpu.CASES, got)) == gpu.CASES


def test_gpu_cases_of_fp32_layers_reach_the_kernels_that_they_name(plans):
    """What decode() does: the launches for few slots where they pay, else the plan's kernels."""
    calls = {call(B.SERE_F32, *c, S, rho): kind for c, kind in gpu.F32_CASES.items() for S, rho in ((1, 0.3),)}
    calls.update({call(B.SERE_F32, T, 1472, M, M, 192, 0, M): kind for (T, M), kind in gpu_nonfinite.F32_CALLS.items()})
    for c, plan, (fits, pays, *_) in zip(calls, plans(calls, "call"), plans(calls, "small")):
        assert ("few" if pays else "tile" if plan[1] else "alu") == calls[c] and plan[1] == plan[2], c
    assert set(gpu.F32_CASES.values()) == set(gpu_nonfinite.F32_CALLS.values()) == {"few", "alu", "tile"}


def test_gpu_cases_reach_every_kernel_of_a_plan(plans):
    """Over a draw of all accepted layers no plan launches a kernel that the GPU cases (and the Mixtral-shaped layer of the
    parity tests: gate/up by the decode kernels next to the persistent down kernel) do not."""
    def kernels(inter, plan):
        rows, tile_gu, tile_dn, _, wide = plan
        split = inter >= 4096
        return {("gate_up", rows if tile_gu else 0, wide), ("down", rows if tile_dn else 0, split)}
    spec = wk.SPECS["mixtral_b64"]
    mixtral = plans([call(spec.dtype, spec.tokens, spec.hidden, spec.experts, spec.top_k, spec.inter, spec.shared, 1)], "call")[0]
    assert mixtral == (32, 0, 1, 2, 0)
    tested = kernels(spec.inter, mixtral).union(*(kernels(c[4], p) for c, p in gpu.CASES.items()))
    rng = random.Random(6)
    log_int = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    cases = []
    for _ in range(20000):
        M = log_int(1, 256)
        K = rng.randint(1, min(M, 12))
        cases.append(call(B.SERE_BF16, log_int(1, 65536), 64 * log_int(1, 256), M, K, 64 * log_int(1, 512),
                          rng.choice([0, 0, 1, 4]), rng.randint(1, K), rng.choice([0.0, 0.3])))
    reached = set()
    for c, p in zip(cases, plans(cases, "call")):
        reached |= kernels(c[5], p)
    assert reached - tested <= {("down", 0, False), ("down", 0, True)}    # the decode kernels, which most other tests run
    assert {("gate_up", r, 0) for r in (32, 64, 96, 128, 160, 192, 256)} | {("gate_up", 256, 1)} <= reached
