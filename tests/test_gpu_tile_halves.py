"""bf16 calls whose last round of units is cut into halves (csrc/ffn_tile.hpp), at the edges of that rule: every expert, routed
or shared, has every token, so that an XCD has two items' units, whole rounds of 32 and some behind them."""
import pytest

import oracle
from paper_2602_07616_amd import workloads as wk
from .test_gpu_parity import check_output, check_routing, dev, small_case  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,dh,dm", [
    # items of 192 rows: d_m / 64 gate/up and d_h / 128 down units of an item; of 128 rows (the last case): half as many
    (120, 576, 512),     # 16 gate/up units an XCD: halves for all workgroups; 10 down units, a fifth of their halves without rows
    (120, 320, 576),     # 18 and 6
    (120, 320, 1088),    # 34: a round and four halves
    (380, 576, 1088),    # 68 and 20: two items an expert
    (120, 704, 1088),    # 18, the last of an item without a second half; 6
])
def test_halves(dev, T, dh, dm):  # noqa: F811
    print(f"halves {T} {dh} {dm}", flush=True)
    wl, layer, sim = small_case(dev, wk.BF16, T, dh, 8, 8, dm, 8, 9900 + T + dm, 8, 0.0)
    ref = oracle.layer(wl.hidden, wl.router_w, wl.w_gate_up, wl.w_down, wl.shared_gate_up, wl.shared_down, wk.BF16, 8, sim, 8, 0.0)
    assert ref.min_gap > 1e-9
    layer.out.fill_(9.0)
    layer.run_decode()
    check_routing(layer.routing_to_host(), ref, layer.cfg)
    check_output(layer.out_to_host_f64(), ref.out_sere, wk.BF16, "sere")
