"""Frobenius similarity of more than 64 experts through both Gram kernels: the one of 64 x 64 blocks, and the one that
stages its operands in LDS (a triangle of 128 experts, squares between triangles, lengths against its ring of eight
32-wide stages)."""
import numpy as np
import pytest

import oracle
from paper_2602_07616_amd import workloads as wk
from .test_gpu_parity import dev  # noqa: F401

pytestmark = pytest.mark.gpu

# M, d_h, tokens, batches, dtype, d_m (64 if not given)
BLOCKS = [
    (65, 64, 1, 1, wk.BF16),      # the smallest: one split, a second block of one row
    (66, 192, 1, 2, wk.F32),
    (128, 256, 5, 3, wk.BF16),    # three whole blocks
    (129, 128, 3, 1, wk.BF16),
    (192, 128, 4, 2, wk.F32),
    (256, 64, 7, 1, wk.BF16),     # ten whole blocks
    (130, 256, 200, 1, wk.BF16),  # long batches, too
    (70, 128, 40, 2, wk.BF16, 2112),  # two slices of d_m
]
STAGED = [
    (65, 64, 641, 1, wk.BF16),    # a last split of two stages; rows repeated up to 128
    (66, 192, 214, 1, wk.F32),    # ... of four, less than the ring holds
    (128, 256, 160, 2, wk.BF16),  # one whole triangle, splits of eight stages
    (100, 512, 90, 2, wk.F32),
    (70, 256, 100, 2, wk.BF16, 1088),   # two batches in a group
    (66, 192, 300, 1, wk.BF16, 2112),   # wide enough for two slices of d_m, of which the plan takes one
    (193, 128, 4096, 1, wk.BF16),  # rows 2 MiB apart: a second triangle of 65 rows, squares with one row
    (256, 128, 4096, 1, wk.F32),   # two whole triangles and the four squares between them
]


@pytest.mark.parametrize("case", BLOCKS + STAGED, ids=lambda c: "x".join(str(v) for v in c))
def test_frobenius(dev, case):  # noqa: F811
    M, dh, n, batches, dtype, dm = (*case, 64)[:6]
    print(f"pair gram {case}", flush=True)
    spec = wk.custom_spec("pairs", dtype, dh, M, 2, dm, 0, 4, 5200 + M, twin_src=0, twin_dst=32, twin_n=32,
                          calib_batches=batches, calib_tokens=n)
    wl = wk.make_workload(spec)
    got = dev.similarity_on_device(wl).cpu().numpy()
    want = oracle.similarity_frobenius(wl.calib, wl.w_gate_up, wl.w_down, dtype)
    # distances carry the rounding of the experts' outputs (fp32 sums; bf16: h rounded to bf16); the fp64 Gram
    # entries add ~1e-16 of the squared norms
    tol = 1e-5 if dtype == wk.F32 else 5e-3
    assert np.abs(got - want).max() <= tol, np.abs(got - want).max()
    assert np.array_equal(got, got.T)
