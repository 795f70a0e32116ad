"""The batch-wide routing step shared by many workgroups (batches from 1536 slots on) against the
oracle: at its threshold, with a last chunk of one token, with one expert, with more experts than one
wavefront row scans, and where a chunk's ids do not fit the workgroup's LDS (the one-workgroup step)."""
import numpy as np
import pytest

import oracle
from paper_2602_07616_amd import workloads as wk
from . import pins
from .test_gpu_parity import check_routing, dev  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # T, M, K, S, rho
    (191, 128, 8, 2, 0.0),     # 1528 slots: one workgroup
    (192, 128, 8, 2, 0.4),     # 1536 slots: 6 chunks of 32 tokens
    (193, 128, 8, 1, 0.0),     # a last chunk of one token
    (1100, 60, 4, 2, 0.3),     # chunks of 64 tokens
    (3000, 250, 6, 1, 0.4),    # chunks of 64 tokens, 16 lists per token
    (1100, 256, 70, 20, 0.3),  # a chunk's ids exceed the LDS array: the one-workgroup step
    (2000, 1, 1, 1, 0.0),      # one expert
    (1700, 3, 3, 1, 0.9),      # every expert primary or kept
    (5000, 17, 2, 2, 0.0),     # S = K: nothing to re-route
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(v) for v in c))
def test_route_and_reroute(dev, case):  # noqa: F811
    import torch
    from paper_2602_07616_amd import binding as B
    T, M, K, S, rho = case
    print(f"route chunks {case}", flush=True)
    spec = wk.custom_spec("chunks", wk.BF16, 192, M, K, 64, 1, T, 4100 + T + M, clusters=5, calib_batches=1, calib_tokens=4)
    wl = wk.make_workload(spec)
    sim = pins.rand_sim(4100 + M, M)
    layer = dev.DeviceLayer.from_workload(wl, sim, S, rho)
    ref = oracle.route(wl.hidden, wl.router_w, spec.dtype, K, sim, S, rho)
    for fill in (0x5A, 0xFF):
        layer.workspace.fill_(fill)           # stale scratch must not matter
        layer.run_route()
        got = layer.routing_to_host()
        if ref.min_gap > 1e-9:
            check_routing(got, ref, layer.cfg)
    # the shared experts' rows behind the routed ones are what the FFN reads: a whole step is finite and repeatable
    layer.run_decode()
    first = layer.out.clone()
    layer.workspace.fill_(0x33)
    layer.run_decode(with_outputs=False)
    assert torch.isfinite(layer.out.float()).all() and (layer.out == first).all()
    # re-routing alone from the ids just found
    ids = got["topk_ids"]
    bufs = B.RouteBuffers.allocate(layer.cfg)
    B.sere_reroute(layer.cfg, torch.from_numpy(ids).cuda(), layer.sim, bufs, layer.workspace)
    torch.cuda.synchronize()
    want, final, _, _ = oracle.reroute_sets(ids, sim, S, rho)
    cnt, offs, tok, slot, n_after = oracle.compact(want, M)
    for name, value in (("rerouted_ids", want), ("count_after", cnt), ("expert_offsets", offs), ("sorted_token", tok),
                        ("sorted_slot", slot), ("primary_mask", oracle.primary_mask(ids, S, M))):
        assert np.array_equal(getattr(bufs, name).cpu().numpy(), value), name
    assert bufs.num_active.cpu().numpy()[1] == n_after
