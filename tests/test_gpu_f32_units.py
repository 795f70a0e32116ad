"""fp32 calls whose work list has the items of more than 16 rows first, and the order in which the persistent workgroups
take their units (csrc/ffn_tile.hpp): against the oracle, at the edges of a round of 256 units.  tests/test_tile_units.py checks the
items that stand beside the cases on the CPU."""
import pytest

import oracle
from paper_2602_07616_amd import workloads as wk
from .test_gpu_parity import check_output, check_routing, dev, small_case  # noqa: F401

pytestmark = pytest.mark.gpu

# T, d_h, M, K, d_m, shared, S, rho; an item has d_m / 64 gate/up and d_h / 128 down units: items, of more than 16 rows, whether these come first
CASES = {
    (70, 64, 40, 4, 512, 2, 4, 0.0): (46, 4, True),        # 368 gate/up units, a round and a part; shared experts of two long items and a short one
    (130, 128, 30, 2, 512, 0, 2, 0.0): (30, 0, False),     # 240: about one round
    (66, 128, 64, 1, 256, 0, 1, 0.0): (40, 0, False),      # units for one round, no long item
    (200, 64, 33, 8, 1024, 0, 8, 0.0): (66, 49, True),     # 48 rows an expert: more long units than three rounds, an expert's items far apart
    (96, 576, 4, 4, 2048, 1, 4, 0.0): (15, 15, True),      # all items long
    (80, 64, 60, 8, 448, 1, 2, 0.4): (61, 8, True),        # re-routing with a threshold
    (300, 1088, 25, 1, 128, 4, 1, 0.0): (65, 39, False),   # one round of gate/up units, 2.3 of down units
    (48, 64, 255, 8, 320, 0, 8, 0.0): (193, 0, True),      # four rounds of short items
}


def seed(case):
    return 9700 + case[0] + case[2]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(v) for v in c))
def test_long_items_first(dev, case):  # noqa: F811
    T, dh, M, K, dm, n_sh, S, rho = case
    print(f"f32 units {case}", flush=True)
    wl, layer, sim = small_case(dev, wk.F32, T, dh, M, K, dm, n_sh, seed(case), S, rho)
    ref = oracle.layer(wl.hidden, wl.router_w, wl.w_gate_up, wl.w_down, wl.shared_gate_up, wl.shared_down, wk.F32, K, sim, S, rho)
    assert ref.min_gap > 1e-9
    layer.run_decode()
    check_routing(layer.routing_to_host(), ref, layer.cfg)
    check_output(layer.out_to_host_f64(), ref.out_sere, wk.F32, "sere")
    layer.run_baseline()
    check_output(layer.out_to_host_f64(), ref.out_base, wk.F32, "baseline")
