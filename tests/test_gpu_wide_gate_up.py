"""The gate/up kernel with units of 256 weight rows x 256 token rows and two stages, which similarity calls and layers whose
tokens select every expert take for items of 256 rows: whole and part-filled token tiles, a last block of weight rows
that is half empty, one k step and several, more units than workgroups.  tests/test_similarity_plan.py and
tests/test_ffn_plan.py check on the CPU that the cases take it."""
import numpy as np
import pytest

import oracle
from paper_2602_07616_amd import workloads as wk
from . import pins
from .test_gpu_parity import dev  # noqa: F401

pytestmark = pytest.mark.gpu

# M, d_h, d_m, tokens, batches
CASES = [
    (64, 64, 448, 241, 1),     # one k step, a last token tile of one row, the last block of 128 indices half empty
    (40, 192, 448, 250, 1),    # three k steps
    (60, 192, 320, 128, 2),    # a group of two batches
    (40, 64, 512, 241, 1),     # whole blocks
    (100, 128, 576, 256, 1),   # 500 units
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(v) for v in c))
def test_wide_gate_up(dev, case):  # noqa: F811
    M, dh, dm, n, batches = case
    print(f"wide gate/up {case}", flush=True)
    spec = wk.custom_spec("wide", wk.BF16, dh, M, 2, dm, 0, 4, 5600 + M + n, twin_src=0, twin_dst=M // 2, twin_n=M // 2,
                          calib_batches=batches, calib_tokens=n)
    wl = wk.make_workload(spec)
    got = dev.similarity_on_device(wl).cpu().numpy()
    want = oracle.similarity_frobenius(wl.calib, wl.w_gate_up, wl.w_down, spec.dtype)
    # the experts' outputs carry the rounding of h to bf16; everything after them is fp64
    assert np.abs(got - want).max() <= 5e-3, np.abs(got - want).max()
    assert np.array_equal(got, got.T)


# (d_h, M, d_m, shared), K = M: a batch that takes the kernel and a longer one that takes units of 128 weight rows, the same
# item size and the same slices of d_m
PAIRS = [
    ((192, 8, 2112, 1), (241, 389)),     # a last token tile of one row, the last block half empty
    ((320, 8, 1472, 1), (1009, 1157)),   # more units than workgroups
    ((64, 8, 704, 1), (1009, 1031)),     # one k step
    ((320, 5, 2240, 0), (500, 774)),
]


@pytest.mark.parametrize("layer, batches", PAIRS, ids=lambda v: "x".join(str(i) for i in v))
def test_the_bits_of_the_narrow_kernel(dev, layer, batches):  # noqa: F811
    """A token's output in both batches: the same sums in the same order."""
    dh, M, dm, sh = layer
    few, many = batches
    spec = wk.custom_spec("widebits", wk.BF16, dh, M, M, dm, sh, many, 5800 + many, calib_batches=1, calib_tokens=4)
    wl = wk.make_workload(spec)
    print(f"wide bits {layer} {batches}", flush=True)
    sim = pins.rand_sim(5800, M)
    whole = dev.DeviceLayer.from_workload(wl, sim, M, 0.0)
    whole.run_baseline()
    want = whole.out[:few].clone()
    wl.hidden = np.ascontiguousarray(wl.hidden[:few])
    part = dev.DeviceLayer.from_workload(wl, sim, M, 0.0, weights=whole.weights())
    part.run_baseline()
    assert want.abs().max() > 0 and (part.out == want).all()
