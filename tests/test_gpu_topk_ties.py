"""Top-K where logits are equal within a list of sixteen experts and across lists: the lower expert first, whatever the number of
lists, of entries kept of them and of workgroups (csrc/route_kernels.hpp, topk_merge)."""
import numpy as np
import pytest

import oracle
from paper_2602_07616_amd import workloads as wk
from .test_gpu_parity import dev, small_case  # noqa: F401

pytestmark = pytest.mark.gpu

# T, M, K
CASES = [(33, 40, 1), (33, 40, 7), (20, 64, 12), (9, 128, 8), (70, 128, 8), (33, 113, 16), (300, 128, 5), (40, 256, 8), (17, 200, 30),
         (5, 256, 256), (33, 17, 17),
         (33, 64, 9), (21, 64, 16), (9, 50, 17), (400, 64, 17), (33, 64, 32), (6, 33, 33)]      # up to 4, 8 and 16 logits of a lane


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(v) for v in c))
def test_equal_logits_go_to_the_lower_expert(dev, case):  # noqa: F811
    T, M, K = case
    rng = np.random.default_rng(T + M + K)

    def mutate(wl):
        wl.router_w[:] = wl.router_w[rng.integers(0, max(2, M // 3), M)]   # a third as many rows, each several times
    wl, layer, _ = small_case(dev, wk.BF16, T, 128, M, K, 64, 0, 9800 + M + K, 1, 0.0, mutate=mutate)
    logits = oracle.router_logits(wl.hidden, wl.router_w, wk.BF16)
    assert any(len(set(row)) < M for row in logits.tolist())
    ids, weights, _ = oracle.topk_gate(logits, K)
    layer.run_route()
    got = layer.routing_to_host()
    assert np.array_equal(got["topk_ids"], ids)
    assert np.abs(got["topk_weights"] - weights).max() <= 1e-6
