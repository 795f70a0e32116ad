"""Centered kernel alignment at the edges of its kernels: token counts around the 16- and 32-row tiles and the change between
them, odd ones (rows of the Gram matrices that are only 8-byte aligned, a last group of products that is cut short), one
part of the products and several, expert counts around the 16-row tiles of the pair kernel."""
import numpy as np
import pytest

import oracle
from paper_2602_07616_amd import workloads as wk
from .test_gpu_parity import dev  # noqa: F401

pytestmark = pytest.mark.gpu

# M, d_h, tokens, batches, dtype, d_m
CASES = [
    (2, 64, 5, 1, wk.F32, 64),         # fewer groups of k than wavefronts
    (17, 64, 4, 2, wk.F32, 64),        # the fewest tokens; a second tile of one expert
    (16, 192, 15, 1, wk.F32, 64),
    (15, 128, 17, 3, wk.F32, 384),     # a second block of one token, a group of batches
    (33, 256, 31, 2, wk.BF16, 192),
    (200, 64, 9, 1, wk.F32, 64),       # no room for more than one part
    (9, 320, 48, 2, wk.F32, 64),       # the last count with blocks of 16
    (9, 320, 49, 2, wk.F32, 64),       # the first with blocks of 32
    (9, 320, 60, 3, wk.F32, 256),      # blocks of 32 in a group of batches
    (5, 192, 65, 1, wk.F32, 64),
    (20, 128, 100, 1, wk.BF16, 2112),  # two slices of d_m
    (3, 64, 129, 1, wk.F32, 64),
    (3, 64, 512, 1, wk.F32, 64),       # the most tokens: sixteen blocks of row sums to a row, in the place of a narrow h
]


# batches that a group holds (tests/test_similarity_plan.py)
GROUPED = {(15, 128, 17, 3, wk.F32, 384): 3, (33, 256, 31, 2, wk.BF16, 192): 2, (9, 320, 60, 3, wk.F32, 256): 3}


@pytest.mark.parametrize("kernel", ["linear", "rbf", "poly"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(v) for v in c))
def test_cka(dev, case, kernel):  # noqa: F811
    M, dh, n, batches, dtype, dm = case
    print(f"cka {kernel} {case}", flush=True)
    spec = wk.custom_spec("cka_edges", dtype, dh, M, 1, dm, 0, 4, 5400 + M + n, twin_src=0, twin_dst=M // 2, twin_n=M // 2,
                          calib_batches=batches, calib_tokens=n)
    wl = wk.make_workload(spec)
    a0 = oracle.moe_layer(wl.calib[0], wl.w_gate_up, wl.w_down, None, None, dtype, np.zeros((n, 1), dtype=np.int32), np.ones((n, 1)))
    norm2 = float(np.mean(np.sum(a0 * a0, axis=1)))
    p0, p1 = {"linear": (0.0, 0.0), "rbf": (np.sqrt(2.0 * norm2), 0.0), "poly": (norm2, 3.0)}[kernel]
    got = dev.similarity_on_device(wl, cka=(kernel, p0, p1)).cpu().numpy()
    want = oracle.similarity_cka(wl.calib, wl.w_gate_up, wl.w_down, dtype, kernel, p0, p1)
    # outputs carry the rounding of fp32 sums, or of h to bf16; everything after them is fp64
    tol = 1e-5 if dtype == wk.F32 else 5e-3
    assert np.abs(got - want).max() <= tol, np.abs(got - want).max()
    assert np.array_equal(got, got.T)
