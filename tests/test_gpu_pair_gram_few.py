"""Frobenius and cosine similarity of up to 64 experts: every tile count of the Gram kernel, expert counts around the tiles,
outputs shorter than a group of loads and longer than one, groups of batches, y in slices; splits that take the kernel's loop
around more than once."""
import numpy as np
import pytest

import oracle
from paper_2602_07616_amd import workloads as wk
from .test_gpu_parity import dev  # noqa: F401

pytestmark = pytest.mark.gpu

# M, d_h, tokens, batches, dtype, d_m
CASES = [
    (2, 64, 1, 1, wk.F32, 64),         # four k steps, less than a wavefront's group
    (16, 192, 3, 2, wk.F32, 64),       # 36 steps, a whole tile
    (15, 448, 33, 1, wk.BF16, 192),    # a split is two groups with the cosine metric; tokens that change inside it
    (17, 64, 5, 3, wk.F32, 64),        # a second tile of one row; a token is one group
    (32, 320, 7, 1, wk.BF16, 64),
    (33, 128, 20, 1, wk.F32, 128),
    (48, 64, 9, 2, wk.F32, 64),
    (49, 192, 11, 1, wk.BF16, 128),
    (64, 128, 40, 1, wk.F32, 64),
    (20, 256, 30, 2, wk.BF16, 2112),   # two slices of d_m, a group of two batches
    (12, 512, 128, 2, wk.BF16, 256),
]
# splits of more than one turn of the loop, and a part of one (tests/test_similarity_plan.py), over several tokens
LONG = [
    (5, 320, 1275, 1, wk.F32, 64),     # 100 steps, 20 a token; a turn is 64, 32 with the cosine metric
    (19, 192, 700, 1, wk.F32, 64),     # 36 steps, 12 a token; 32 a turn
    (37, 192, 400, 1, wk.BF16, 64),    # 20 steps; 16 a turn
    (61, 128, 700, 1, wk.F32, 64),     # 24 steps, 8 a token
    (40, 1024, 64, 4, wk.BF16, 64),    # 24 steps, a group of four batches
    (50, 1024, 64, 4, wk.BF16, 64),
]


@pytest.mark.parametrize("metric", ["frobenius", "cosine"])
@pytest.mark.parametrize("case", CASES + LONG, ids=lambda c: "x".join(str(v) for v in c))
def test_few_experts(dev, case, metric):  # noqa: F811
    M, dh, n, batches, dtype, dm = case
    print(f"pair gram few {metric} {case}", flush=True)
    spec = wk.custom_spec("few", dtype, dh, M, 1, dm, 0, 4, 5700 + M + n, twin_src=0, twin_dst=M // 2, twin_n=M // 2,
                          calib_batches=batches, calib_tokens=n)
    wl = wk.make_workload(spec)
    got = dev.similarity_on_device(wl, metric=metric).cpu().numpy()
    ref = {"frobenius": oracle.similarity_frobenius, "cosine": oracle.similarity_cosine}[metric]
    want = ref(wl.calib, wl.w_gate_up, wl.w_down, dtype)
    # the experts' outputs carry the rounding of fp32 sums, or of h to bf16; everything after them is fp64
    tol = 1e-5 if dtype == wk.F32 else 5e-3
    assert np.abs(got - want).max() <= tol, np.abs(got - want).max()
    assert np.array_equal(got, got.T)
