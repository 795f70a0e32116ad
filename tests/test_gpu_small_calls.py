"""Calls of at most 64 slots that take two launches behind the router logits (csrc/ffn_small.hpp), at the edges of what they
take: against the oracle, and against the launches for larger calls, which serve the same tokens given several times over.
tests/test_small_calls_plan.py checks on the CPU that the cases take them."""
import copy

import numpy as np
import pytest

import oracle
from paper_2602_07616_amd import workloads as wk
from . import pins
from .test_gpu_parity import TOL, check_output, check_routing, dev, small_case  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, T, d_h, M, K, d_m, shared, S, rho
    (wk.BF16, 1, 2048, 128, 8, 768, 0, 2, 0.0),     # eight blocks of a contraction to a wavefront's four
    (wk.BF16, 1, 64, 1, 1, 64, 0, 1, 0.0),          # the smallest layer
    (wk.F32, 1, 64, 3, 3, 64, 4, 1, 0.5),           # one token, shared experts
    (wk.F32, 8, 1024, 8, 8, 256, 0, 8, 0.0),        # 64 slots, all primary
    (wk.F32, 3, 192, 256, 8, 64, 0, 3, 0.0),        # 16 lists of experts, nine primary slots
    (wk.BF16, 2, 320, 129, 5, 128, 1, 4, 0.0),      # eight primary slots: every wavefront looks at all of them; nine lists
    (wk.BF16, 5, 320, 113, 3, 64, 0, 2, 0.4),       # ten: each looks at some; the last list has one expert
    (wk.F32, 16, 512, 16, 4, 256, 0, 3, 0.3),       # 64 slots
    (wk.F32, 16, 448, 2, 2, 192, 4, 1, 0.0),        # a whole tile of rows for every shared expert, 96 rows in all
    (wk.F32, 7, 1472, 33, 3, 320, 2, 1, 0.0),       # blocks that do not split evenly
    (wk.BF16, 3, 4096, 20, 3, 320, 0, 2, 0.6),      # two rounds of loads
    (wk.F32, 2, 512, 60, 4, 1088, 0, 1, 0.0),       # more units than workgroups without re-routing
    (wk.F32, 9, 1024, 64, 7, 128, 1, 3, 0.5),       # 63 slots and a shared expert: the longest work list
    (wk.F32, 17, 768, 9, 1, 320, 0, 1, 0.0),        # a tile and a row of tokens
    (wk.F32, 32, 1024, 1, 1, 256, 0, 1, 0.0),       # two whole tiles of one expert
    (wk.F32, 64, 1024, 3, 1, 256, 0, 1, 0.0),       # an output element of every thread
    (wk.F32, 32, 1024, 2, 1, 128, 3, 1, 0.0),       # two tiles of every shared expert, 128 rows in all
    (wk.F32, 32, 1088, 5, 2, 256, 0, 1, 0.6),       # 32 primary slots
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(v) for v in c))
def test_small_calls(dev, case):  # noqa: F811
    from paper_2602_07616_amd import binding as B
    dtype, T, dh, M, K, dm, n_sh, S, rho = case
    print(f"small {case}", flush=True)
    wl, layer, sim = small_case(dev, dtype, T, dh, M, K, dm, n_sh, 9300 + T + M, S, rho)
    ref = oracle.layer(wl.hidden, wl.router_w, wl.w_gate_up, wl.w_down, wl.shared_gate_up, wl.shared_down, dtype, K, sim, S, rho)
    assert ref.min_gap > 1e-9
    layer.run_decode()
    check_routing(layer.routing_to_host(), ref, layer.cfg)
    check_output(layer.out_to_host_f64(), ref.out_sere, dtype, "sere")
    first = layer.out.clone()
    layer.out.zero_()
    layer.run_decode(with_outputs=False)
    assert (layer.out == first).all()
    layer.cfg.flags = B.SERE_FLAG_RESIDUAL
    layer.run_decode()
    check_output(layer.out_to_host_f64(), ref.out_sere + layer.hidden.double().cpu().numpy(), dtype, "residual")
    layer.cfg.flags = 0
    layer.run_baseline()
    check_output(layer.out_to_host_f64(), ref.out_base, dtype, "baseline")
    small, before = layer.out.clone(), layer.routing_to_host()
    # while stages are timed the same launches run, each recorded for the stages that it does
    B.sere_stage_timing(True)
    layer.out.zero_()
    layer.run_baseline()
    ms, launches = B.sere_stage_timing_read()
    B.sere_stage_timing(False)
    assert all(launches[stage] == 1 and ms[stage] > 0 for stage in ("router", "route", "gate_up", "down", "combine"))
    assert ms["route"] == ms["gate_up"] and ms["down"] == ms["combine"]
    assert (layer.out == small).all()
    # more than 64 slots
    times = -(-65 // T)
    again = copy.copy(wl)
    again.hidden = np.concatenate([wl.hidden] * times)
    large = dev.DeviceLayer.from_workload(again, sim, S, rho, weights=layer.weights())
    large.run_baseline()
    after = large.routing_to_host()
    for name in ("topk_ids", "rerouted_ids"):
        assert np.array_equal(after[name], np.concatenate([before[name]] * times)), name
    for name in ("primary_mask", "num_active"):
        assert np.array_equal(after[name], before[name]), name
    for name in ("count_before", "count_after", "expert_offsets"):
        assert np.array_equal(after[name], times * before[name]), name
    # both are within half the tolerance of the exact result's rounding, so within it of each other
    small, rest = small.double().cpu().numpy(), large.out_to_host_f64()[:T]
    assert np.abs(small - rest).max() <= max(TOL[dtype][0], np.abs(small).max() * 2.0 ** -7 if dtype == wk.BF16 else 0.0)


@pytest.mark.parametrize("dtype", [wk.BF16, wk.F32])
def test_equal_logits_and_similarities(dev, dtype):  # noqa: F811
    """Equal router rows, in one list of sixteen experts and in two, and a similarity matrix of few values: the lower expert
    first.  Similarities of minus infinity and NaN (no precondition allows them) as in the launches for larger calls."""
    T, M, K = 4, 40, 5
    def mutate(wl):
        wl.router_w[5] = wl.router_w[3]
        wl.router_w[35] = wl.router_w[3]
        wl.router_w[20:26] = wl.router_w[20]
        wl.hidden[1] = wl.hidden[0]
    wl, layer, _ = small_case(dev, dtype, T, 256, M, K, 64, 0, 9500, 1, 0.0, mutate=mutate)
    logits = oracle.router_logits(wl.hidden, wl.router_w, dtype)
    ids, _, _ = oracle.topk_gate(logits, K)
    rng = np.random.default_rng(9500)
    few = rng.integers(0, 3, (M, M)).astype(np.float32) / 4
    holes = few.copy()
    holes[rng.random((M, M)) < 0.4] = np.nan
    holes[rng.random((M, M)) < 0.4] = -np.inf
    for sim in (few, holes, np.full((M, M), -np.inf, np.float32)):
        for S, rho in ((1, 0.0), (2, 0.25), (2, 0.0)):
            layer = dev.DeviceLayer.from_workload(wl, sim, S, rho, weights=layer.weights())
            layer.run_decode()
            got = layer.routing_to_host()
            assert np.array_equal(got["topk_ids"], ids)
            if sim is few:
                want, _, _, _ = oracle.reroute_sets(ids, sim, S, rho)
                assert np.array_equal(got["rerouted_ids"], want)
            layer.run_route()          # the launches for larger calls
            for name, value in layer.routing_to_host().items():
                if name != "topk_weights":
                    assert np.array_equal(got[name], value), name


SAME = [(wk.BF16, 8, 320, 40, 4, 192, 1, 1, 0.0), (wk.F32, 16, 512, 16, 4, 256, 0, 1, 0.0)]


@pytest.mark.parametrize("case", SAME, ids=lambda c: "x".join(str(v) for v in c))
def test_one_expert_has_every_slot(dev, case):  # noqa: F811
    """All tokens equal and one primary expert: 32 and 64 rows, two and four tiles."""
    dtype, T, dh, M, K, dm, n_sh, S, rho = case
    def mutate(wl):
        wl.hidden[:] = wl.hidden[0]
    wl, layer, sim = small_case(dev, dtype, T, dh, M, K, dm, n_sh, 9700 + T, S, rho, mutate=mutate)
    ref = oracle.layer(wl.hidden, wl.router_w, wl.w_gate_up, wl.w_down, wl.shared_gate_up, wl.shared_down, dtype, K, sim, S, rho)
    assert ref.min_gap > 1e-9 and ref.count_after.max() == T * K
    layer.run_decode()
    check_routing(layer.routing_to_host(), ref, layer.cfg)
    check_output(layer.out_to_host_f64(), ref.out_sere, dtype, "one expert")


@pytest.mark.parametrize("dtype", [wk.BF16, wk.F32])
@pytest.mark.parametrize("M,K", [(3, 2), (19, 8), (130, 4)])
def test_a_token_of_nan_chooses_experts(dev, dtype, M, K):  # noqa: F811
    """Hidden states whose bits are all set (memory that nobody wrote; no precondition allows them): the smallest keys there
    are.  The ids are those of the launches for larger calls, so experts, and the other token's output is what it is."""
    def mutate(wl):
        wl.hidden.view(np.uint32 if dtype == wk.F32 else np.uint16)[1] = 0xffffffff if dtype == wk.F32 else 0xffff
    wl, layer, sim = small_case(dev, dtype, 2, 64, M, K, 64, 0, 9800 + M, K, 0.0, mutate=mutate)
    print(f"small nan dtype {dtype} M {M}", flush=True)
    layer.run_route()
    want = layer.routing_to_host()
    assert want["topk_ids"].max() < M and all(len(set(row)) == K for row in want["topk_ids"].tolist())
    for run in (layer.run_decode, layer.run_baseline):
        run()
        got = layer.routing_to_host()
        for name in want:
            assert np.array_equal(got[name], want[name], equal_nan=True) or name == "topk_weights", name
        out = layer.out_to_host_f64()
        assert np.isnan(out[1]).all()
        alone = oracle.layer(wl.hidden[:1], wl.router_w, wl.w_gate_up, wl.w_down, None, None, dtype, K, sim, K, 0.0)
        check_output(out[:1], alone.out_base, dtype, "the other token")
