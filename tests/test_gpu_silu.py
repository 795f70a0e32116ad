"""silu where 1 + exp(-z) is beyond 2^126 and its reciprocal below the smallest normal number: the result, some 1e-37 there, times
an up projection of its inverse's size is an ordinary number that the layer has to return."""
import numpy as np
import pytest

import oracle
from paper_2602_07616_amd import workloads as wk
from . import pins
from .test_gpu_parity import dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [wk.BF16, wk.F32])
@pytest.mark.parametrize("tokens, inter", [(4, 64), (300, 64), (4, 4160), (300, 4160)])    # small and large batches, one plane of h and two
def test_gate_whose_reciprocal_is_not_normal(dev, tokens, inter, dtype):  # noqa: F811
    spec = wk.custom_spec("silu", dtype, 64, 2, 2, inter, 0, tokens, 9100, calib_batches=1, calib_tokens=4)
    wl = wk.make_workload(spec)
    store = lambda a: wk.to_storage(np.asarray(a, dtype=np.float32), dtype)
    # gate z = -88 + offset, up 2^121 to 2^124, so that |silu(z) up| is 0.7 to 50; output r is intermediate r
    offsets = np.tile(np.linspace(-0.65, 1.5, 64, dtype=np.float32), inter // 64)
    hidden = np.zeros((tokens, 64), dtype=np.float32)
    hidden[:, 0] = hidden[:, 1] = 1.0
    hidden[:, 2] = 2.0 ** (np.arange(tokens) % 4)
    gate_up, down = np.zeros((2, 2 * inter, 64), dtype=np.float32), np.zeros((2, 64, inter), dtype=np.float32)
    gate_up[:, :inter, 0] = -88.0
    gate_up[:, :inter, 1] = offsets
    gate_up[:, inter:, 2] = 2.0 ** 121
    down[:, np.arange(64), np.arange(64)] = 1.0
    wl.hidden[:], wl.w_gate_up[:], wl.w_down[:] = store(hidden), store(gate_up), store(down)
    layer = dev.DeviceLayer.from_workload(wl, pins.rand_sim(9100, 2), 2, 0.0)
    print(f"silu {tokens} tokens, d_m {inter}, dtype {dtype}", flush=True)
    layer.run_baseline()
    got = layer.out_to_host_f64()
    ids, weights = layer.routing_to_host()["topk_ids"], layer.routing_to_host()["topk_weights"]
    want = oracle.moe_layer(wl.hidden, wl.w_gate_up, wl.w_down, None, None, dtype, ids, weights.astype(np.float64))
    assert np.abs(want).min() > 0.5 and np.abs(want).max() < 60
    # z is right to its last place, 2^-18, and so is the argument of the exponential: 1e-5; bf16: h and the output are rounded,
    # 2^-9 each
    tol = 2e-5 + (0.0 if dtype == wk.F32 else 2.0 ** -8)
    assert (np.abs(got - want) <= tol * np.abs(want)).all(), np.abs(got / want - 1).max()
