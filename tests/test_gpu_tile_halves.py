"""bf16 calls whose last round of units is cut into halves (csrc/ffn_tile.hpp): every expert, routed or shared, has every token
(K = M), so that the units of a launch are known.  tests/test_tile_units.py checks on the CPU that the cases have the plans and the
units that stand beside them, and that every kernel has a workgroup that goes on from whole units to a half."""
import numpy as np
import pytest

import oracle
from paper_2602_07616_amd import workloads as wk
from . import pins
from .test_gpu_parity import check_output, check_routing, dev, small_case  # noqa: F401

pytestmark = pytest.mark.gpu

# (T, d_h, M, d_m, shared): rows of an item, then of gate/up and of down the whole units and the halves of the launch (None: another kernel)
CASES = {
    (120, 576, 8, 512, 8): (192, (0, 256), (0, 144)),      # 16 gate/up units an XCD: halves for all workgroups; 10 down units, the last half of an item without rows
    (120, 320, 8, 576, 8): (192, (144, 0), (0, 80)),       # 18 gate/up units an XCD, just beyond the rule
    (120, 320, 8, 1088, 8): (192, (256, 32), (0, 80)),     # 34: a round and four halves
    (380, 576, 8, 1088, 8): (192, (512, 64), (160, 0)),    # 68 and 20: two items an expert
    (120, 704, 8, 1088, 8): (128, (144, 0), (0, 96)),      # items of 128 rows: 18, 6
    # whole units behind which halves come, every kernel
    (66, 320, 12, 832, 1): (32, (256, 31), None),
    (20, 1024, 64, 320, 1): (32, (195, 0), (256, 8)),
    (33, 320, 96, 320, 0): (64, (256, 48), (192, 0)),
    (43, 448, 128, 64, 2): (64, (34, 96), (256, 8)),
    (68, 320, 100, 320, 0): (96, (256, 73), (200, 0)),
    (74, 448, 128, 64, 2): (96, (34, 96), (256, 8)),
    (65, 320, 8, 4480, 1): (128, (256, 118), (0, 135)),
    (608, 960, 12, 64, 1): (128, (0, 65), (256, 8)),
    (577, 320, 96, 64, 0): (160, (256, 128), (768, 0)),
    (513, 192, 64, 64, 1): (160, (260, 0), (256, 8)),
    (33, 320, 64, 256, 1): (192, (256, 8), (195, 0)),
    (38, 256, 128, 64, 2): (192, (34, 192), (256, 8)),
    (807, 320, 12, 320, 1): (256, (256, 8), (156, 0)),
    (588, 64, 128, 64, 0): (256, (384, 0), (256, 128)),
    # two planes of h
    (17, 448, 64, 4224, 1): (32, None, (256, 8)),
    (34, 192, 128, 4224, 2): (64, (4290, 0), (256, 8)),
    (33, 128, 128, 4096, 2): (128, (4160, 0), (256, 8)),
    # gate/up of four k steps: no halves behind whole units
    (33, 256, 64, 256, 1): (32, (260, 0), None),
}


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(v) for v in c))
def test_halves(dev, case):  # noqa: F811
    T, dh, M, dm, n_sh = case
    print(f"halves {case}", flush=True)
    wl, layer, sim = small_case(dev, wk.BF16, T, dh, M, M, dm, n_sh, 9900 + T + dm, M, 0.0)
    # every token, or a dozen of them where the oracle would take long
    tokens = range(T) if T * (M + n_sh) * dh * dm < 5e9 else sorted(set(range(0, T, max(1, T // 12))) | {T - 1})
    ref = oracle.route(wl.hidden, wl.router_w, wk.BF16, M, sim, M, 0.0)
    assert ref.min_gap > 1e-9
    layer.out.fill_(9.0)
    layer.run_decode()
    check_routing(layer.routing_to_host(), ref, layer.cfg)
    want = oracle.moe_layer(np.ascontiguousarray(wl.hidden[tokens]), wl.w_gate_up, wl.w_down, wl.shared_gate_up, wl.shared_down, wk.BF16,
                            np.ascontiguousarray(ref.rerouted_ids[tokens]), np.ascontiguousarray(ref.topk_weights[tokens]))
    check_output(layer.out_to_host_f64()[tokens], want, wk.BF16, "sere")
    first = layer.out.clone()
    layer.workspace.fill_(0x5A)
    layer.run_decode()
    assert (layer.out == first).all()


# (d_h, M, d_m, shared): a batch whose gate/up or down units are cut behind whole ones, and one whose units of that launch are not cut,
# with the same slices of d_m
PAIRS = {
    (320, 4, 2240, 0): ("gate_up", 340, 406),     # items of 192 rows, two slices
    (320, 24, 256, 2): ("gate_up", 674, 561),     # 160
    (512, 32, 320, 2): ("gate_up", 336, 266),     # 128 and 160
    (512, 24, 64, 2): ("down", 526, 421),         # 128 and 256
    (384, 48, 64, 0): ("down", 327, 306),         # 192 and 160
    (640, 12, 2304, 1): ("down", 334, 299),       # 192 and 160, two slices
}


@pytest.mark.parametrize("layer", PAIRS, ids=lambda c: "x".join(str(v) for v in c))
def test_the_bits_of_whole_units(dev, layer):  # noqa: F811
    """A token's output in both batches: the same sums in the same order."""
    dh, M, dm, sh = layer
    _, *batches = PAIRS[layer]
    spec = wk.custom_spec("halfbits", wk.BF16, dh, M, M, dm, sh, max(batches), 5900 + dm, calib_batches=1, calib_tokens=4)
    wl = wk.make_workload(spec)
    print(f"half bits {layer} {batches}", flush=True)
    sim = pins.rand_sim(5900, M)
    outs, weights = [], None
    for T in batches:
        part = wk.Workload(**{**wl.__dict__, "hidden": np.ascontiguousarray(wl.hidden[:T])})
        device_layer = dev.DeviceLayer.from_workload(part, sim, M, 0.0, weights=weights)
        weights = device_layer.weights()
        device_layer.run_baseline()
        outs.append(device_layer.out[:min(batches)].clone())
    assert outs[0].abs().max() > 0 and (outs[0] == outs[1]).all()
