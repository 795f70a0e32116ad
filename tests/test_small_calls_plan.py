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
    for _ in range(8000):
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


# dtype, T, d_h, M, K, d_m, shared, S, rho, reroute: calls that these launches took and that were 0.68 to 0.90 times as fast by them as by the
# others, and calls that are 1.33 to 2.6 times as fast
SLOWER = [(1, 10, 448, 145, 4, 256, 4, 1, 0.5, 0), (1, 14, 896, 74, 2, 256, 4, 1, 0.5, 1), (1, 11, 2368, 147, 1, 128, 4, 1, 0.3, 1),
          (1, 14, 2816, 26, 1, 192, 2, 1, 0.3, 0), (1, 6, 2368, 129, 2, 192, 4, 2, 0.0, 1), (1, 13, 3584, 13, 4, 256, 1, 2, 0.0, 0),
          (0, 12, 256, 31, 4, 640, 0, 3, 0.0, 1), (0, 12, 448, 29, 2, 832, 1, 2, 0.0, 1), (0, 14, 384, 21, 2, 704, 0, 2, 0.5, 1),
          (0, 10, 448, 28, 2, 1024, 0, 1, 0.0, 0), (0, 12, 1344, 16, 4, 512, 4, 3, 0.0, 1), (1, 5, 320, 113, 4, 128, 0, 2, 0.4, 1)]
FASTER = [(1, 1, 1344, 3, 1, 1920, 0, 1, 0.0, 1), (1, 1, 2048, 128, 8, 768, 0, 2, 0.0, 1), (1, 2, 1600, 21, 6, 320, 4, 1, 0.0, 1),
          (1, 3, 896, 26, 2, 192, 0, 2, 0.5, 1), (1, 4, 256, 40, 5, 64, 0, 2, 0.25, 1), (0, 6, 1344, 16, 8, 256, 0, 1, 0.0, 1),
          (0, 8, 256, 16, 2, 128, 0, 1, 0.0, 1), (0, 18, 1280, 4, 2, 192, 0, 1, 0.5, 0), (0, 1, 640, 33, 2, 1024, 0, 2, 0.0, 1)]


def test_taken_where_they_are_faster(small):
    assert [pays for _, pays, _, _ in small(SLOWER)] == [0] * len(SLOWER)
    assert [pays for _, pays, _, _ in small(FASTER)] == [1] * len(FASTER)
