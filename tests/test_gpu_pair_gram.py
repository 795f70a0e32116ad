"""Frobenius similarity through the Gram kernel that stages its operands in LDS (more than 64 experts):
one triangle of 128 experts, a last triangle of one row, squares between triangles, batches of every
length against its ring of eight 32-wide stages."""
import numpy as np
import pytest

import oracle
from paper_2602_07616_amd import workloads as wk
from .test_gpu_parity import dev  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # M, d_h, tokens, batches, dtype
    (65, 64, 1, 1, wk.BF16),      # the smallest: one split of two stages
    (66, 192, 1, 2, wk.F32),      # fewer stages than the ring holds
    (128, 256, 5, 3, wk.BF16),    # one whole triangle, splits of eight stages
    (129, 128, 3, 1, wk.BF16),    # a second triangle of one row
    (192, 128, 4, 2, wk.F32),     # one square for each pair of groups
    (256, 64, 7, 1, wk.BF16),     # two whole triangles and the four squares between them
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(v) for v in c))
def test_frobenius(dev, case):  # noqa: F811
    M, dh, n, batches, dtype = case
    print(f"pair gram {case}", flush=True)
    spec = wk.custom_spec("pairs", dtype, dh, M, 2, 64, 0, 4, 5200 + M, twin_src=0, twin_dst=32, twin_n=32,
                          calib_batches=batches, calib_tokens=n)
    wl = wk.make_workload(spec)
    got = dev.similarity_on_device(wl).cpu().numpy()
    want = oracle.similarity_frobenius(wl.calib, wl.w_gate_up, wl.w_down, dtype)
    # distances carry the rounding of the experts' outputs (fp32 sums; bf16: h rounded to bf16); the fp64 Gram
    # entries add ~1e-16 of the squared norms
    tol = 1e-5 if dtype == wk.F32 else 5e-3
    assert np.abs(got - want).max() <= tol, np.abs(got - want).max()
    assert np.array_equal(got, got.T)
