"""The host's choice of the two launches for few slots (csrc/ffn_plan.hpp, compiled here with g++)."""
import os
import random
import subprocess

import pytest

from . import test_gpu_small_calls as gpu

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def small(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", os.path.join(HERE, "plan_main.cpp"), "-o", exe], check=True)

    def run(calls):
        text = "".join(" ".join(map(str, c)) + "\n" for c in calls)
        out = subprocess.run([exe, "small"], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        return [tuple(int(v) for v in line.split()) for line in out if line]
    return run


def test_the_gpu_cases_take_them(small):
    calls = [(dt, T, dh, M, K, dm, sh, S, rho, reroute) for dt, T, dh, M, K, dm, sh, S, rho in gpu.CASES for reroute in (0, 1)]
    calls += [(*c, 1) for c in gpu.SAME] + [(dt, 4, 256, 40, 5, 64, 0, S, rho, 1) for dt in (0, 1) for S, rho in ((1, 0.0), (2, 0.25), (2, 0.0))]
    calls += [(dt, 2, 64, M, K, 64, 0, K, 0.0, reroute) for dt in (0, 1) for M, K in ((3, 2), (19, 8), (130, 4)) for reroute in (0, 1)]
    for call, (fits, pays, _, _) in zip(calls, small(calls)):
        assert fits and pays, call


def test_what_fits_is_what_the_kernels_hold(small):
    rng = random.Random(3)
    calls = []
    for _ in range(5000):
        M = rng.choice([1, 2, 8, 16, 17, 64, 128, 129, 256])
        K = rng.randint(1, min(M, 12))
        calls.append((rng.randint(0, 1), rng.randint(1, 70), 64 * rng.randint(1, 70), M, K, 64 * rng.randint(1, 80), rng.choice([0, 0, 1, 2, 4, 16]),
                      rng.randint(1, K), rng.choice([0.0, 0.5]), rng.randint(0, 1)))
    taken = 0
    for (dt, T, dh, M, K, dm, sh, S, rho, re), (fits, pays, split, units) in zip(calls, small(calls)):
        if pays:
            taken += 1
            assert fits and K <= 8 and T <= (64 if dt == 0 else 16) and T * K + sh <= 64 and T * (K + sh) <= 128 and (dt == 0 or dm < 4096)
        assert split in (1, 2, 4, 8) and dm % (64 // split) == 0 and units * (64 // split) == dm
    assert taken > 300
