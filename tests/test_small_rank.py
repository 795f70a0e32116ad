"""The ranking behind the top-K of calls of few slots (csrc/rules.hpp, compiled here with g++): for every kind of logit the ids
are those of a stable sort, and none is a place without an expert."""
import os
import random
import struct
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def key_of(bits):
    """The router kernels' order-preserving key of a double's bits."""
    if bits == 1 << 63:
        bits = 0
    return bits ^ ((1 << 64) - 1) if bits >> 63 else bits | 1 << 63


def double_bits(x):
    return struct.unpack("<Q", struct.pack("<d", x))[0]


# fp32 and bf16 NaN of either sign, with all bits of the mantissa or one, as doubles; infinities; zeros; the lowest number
SPECIAL = [0xffffffffe0000000, 0x7fffffffe0000000, 0xfff8000000000000, 0x7ff8000000000000, 0xffffe00000000000, 0xfff0000020000000,
           0xfff0000000000000, 0x7ff0000000000000, 0x8000000000000000, 0, 0xffefffffffffffff, 0x8000000000000001]


def test_ids_are_those_of_a_stable_sort(tmp_path):
    exe = str(tmp_path / "rank")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", os.path.join(HERE, "small_rank_main.cpp"), "-o", exe], check=True)
    rng = random.Random(8)
    cases = []
    for M in (1, 2, 3, 7, 8, 9, 15, 16, 17, 23, 24, 33, 40, 127, 128, 129, 131, 255, 256):
        for K in sorted({1, min(2, M), min(8, M)}):
            cases += [(K, [s] * M) for s in SPECIAL]                                                   # all experts alike
            for _ in range(6):
                plain = [double_bits(rng.gauss(0, 1)) for _ in range(M)]
                few = [double_bits(rng.choice([-1.0, 0.0, 0.5])) for _ in range(M)]
                near = [double_bits(1.0) + rng.randrange(3) for _ in range(M)]                         # equal upper halves
                mixed = [rng.choice(SPECIAL) if rng.random() < 0.7 else b for b in plain]
                cases += [(K, bits) for bits in (plain, few, near, mixed)]
    text = "".join(f"{K} {len(bits)} " + " ".join("%x" % key_of(b) for b in bits) + "\n" for K, bits in cases)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
    for (K, bits), line in zip(cases, out):
        keys = [key_of(b) for b in bits]
        assert all(keys)
        want = sorted(range(len(keys)), key=lambda e: -keys[e])[:K]
        assert [int(v) for v in line.split()] == want, (K, ["%x" % b for b in bits])
