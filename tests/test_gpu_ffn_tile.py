"""The persistent FFN kernels (csrc/ffn_tile.hpp) against the oracle, at sizes where they can go
wrong: every kernel that a plan can launch, rows per expert around multiples of a 16-row tile and
of the item size, d_h and d_m that end inside a unit (64 mod 128, 64 mod 256), shared experts, two
slices of d_m, both planes of h.  Tolerances are those of the other bf16 parity tests.  The plan that a case
is there for stands beside it; tests/test_ffn_plan.py checks on the CPU that the host's rule gives that plan, and that
the cases reach every kernel."""
import numpy as np
import pytest

import oracle
from paper_2602_07616_amd import workloads as wk
from . import pins
from .test_gpu_parity import check_output, check_routing, dev, pairs_with_counts, plant_routing  # noqa: F401

pytestmark = pytest.mark.gpu

# (T, d_h, M, K, d_m, shared): (item rows, gate/up and down by the persistent kernels, slices of d_m, gate/up in units of
# 256 weight rows although the items have 256); d_m >= 4096: both planes
CASES = {
    (33, 320, 2, 2, 1472, 1): (32, 1, 0, 1, 0),     # down by the other kernels
    (500, 1024, 42, 2, 320, 1): (32, 1, 1, 1, 0),
    (230, 704, 33, 4, 704, 1): (64, 1, 1, 1, 0),
    (230, 320, 17, 4, 2112, 1): (64, 1, 1, 2, 0),
    (500, 320, 33, 4, 704, 1): (96, 1, 1, 1, 0),
    (777, 704, 33, 4, 704, 0): (128, 1, 1, 1, 0),
    (1100, 320, 33, 4, 2112, 1): (160, 1, 1, 2, 0),
    (330, 320, 17, 4, 704, 0): (192, 1, 1, 1, 0),
    (500, 320, 5, 4, 1472, 0): (256, 1, 1, 1, 0),
    (33, 320, 2, 2, 4160, 0): (32, 1, 0, 3, 0),
    (300, 512, 23, 1, 4160, 1): (32, 1, 1, 3, 0),
    (230, 320, 26, 4, 4160, 0): (64, 1, 1, 3, 0),
    (230, 320, 2, 2, 4160, 1): (128, 1, 1, 3, 0),
    (1600, 320, 5, 4, 4160, 1): (128, 1, 1, 1, 0),  # one slice
    (700, 64, 4, 4, 64, 0): (32, 1, 0, 1, 0),       # a single k step per gate/up unit, every expert sees every token
    (1200, 64, 226, 1, 64, 1): (192, 1, 1, 1, 0),   # a single k step per unit of both kernels
    (241, 192, 8, 8, 2112, 1): (256, 1, 1, 2, 1),  # gate/up units of 256 weight rows: the last block half empty, a token tile of one row
    (753, 64, 8, 8, 2112, 1): (256, 1, 1, 2, 1),   # ... a single k step, more units than workgroups
    (1009, 192, 6, 6, 1088, 0): (256, 1, 1, 1, 1),
}


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(v) for v in c))
def test_every_item_size(dev, case):  # noqa: F811
    T, dh, M, K, dm, n_sh = case
    spec = wk.custom_spec("tile" + "x".join(map(str, case)), wk.BF16, dh, M, K, dm, n_sh, T, 5000 + T + dm, clusters=3,
                          calib_batches=1, calib_tokens=4)
    wl = wk.make_workload(spec)
    sim = pins.rand_sim(5000 + T, M)
    layer = dev.DeviceLayer.from_workload(wl, sim, 1, 0.0)
    tokens = sorted(set(range(0, T, max(1, T // 24))) | {T - 1})
    for S, rho in ((1, 0.0), (K, 0.0)):
        print(f"tile {case} S={S}", flush=True)
        layer.set_knobs(S, rho)
        layer.out.fill_(9.0)
        layer.run_decode()
        ref = oracle.route(wl.hidden, wl.router_w, spec.dtype, K, sim, S, rho)
        if ref.min_gap <= 1e-9:
            pytest.skip("near-tie in the router ordering for this seed")
        check_routing(layer.routing_to_host(), ref, layer.cfg)
        want = oracle.moe_layer(np.ascontiguousarray(wl.hidden[tokens]), wl.w_gate_up, wl.w_down, wl.shared_gate_up,
                                wl.shared_down, spec.dtype, np.ascontiguousarray(ref.rerouted_ids[tokens]),
                                np.ascontiguousarray(ref.topk_weights[tokens]))
        check_output(layer.out_to_host_f64()[tokens], want, spec.dtype, f"tile {case} S={S}")
        first = layer.out.clone()
        layer.workspace.fill_(0x5A)
        layer.run_decode()
        assert (layer.out == first).all()          # the same bits again


F32_CASES = {
    # T, d_h, M, K, d_m, shared: the two launches of calls of few slots, the vector-ALU kernels (below 9 tokens, where those do not take the
    # call) or the persistent ones
    (1, 1472, 17, 4, 192, 1): "few", (8, 1472, 5, 2, 704, 0): "few", (8, 256, 16, 2, 128, 0): "few", (9, 1472, 5, 2, 704, 1): "few",
    (1, 1472, 17, 9, 192, 1): "alu", (8, 1472, 8, 8, 64, 1): "alu", (6, 2880, 11, 9, 128, 0): "alu",
    (33, 64, 2, 2, 64, 1): "tile", (70, 320, 3, 1, 448, 0): "tile", (300, 704, 8, 2, 1088, 2): "tile", (9, 1472, 9, 9, 192, 1): "tile",
}


@pytest.mark.parametrize("case", F32_CASES, ids=lambda c: "x".join(str(v) for v in c))
def test_fp32_layers(dev, case):  # noqa: F811
    """Every token against fp64; an fp32 sum of n products of independent terms rounds to about sqrt(n) 2^-24 of
    its size at worst, and the compensated sums stay near 2e-7: 1e-6 relative leaves a factor of five."""
    T, dh, M, K, dm, n_sh = case
    spec = wk.custom_spec("f32tile" + "x".join(map(str, case)), wk.F32, dh, M, K, dm, n_sh, T, 5400 + T + dm, clusters=3,
                          calib_batches=1, calib_tokens=4)
    wl = wk.make_workload(spec)
    sim = pins.rand_sim(5400 + T, M)
    layer = dev.DeviceLayer.from_workload(wl, sim, 1, 0.3)
    print(f"fp32 {case}", flush=True)
    ref = oracle.layer(wl.hidden, wl.router_w, wl.w_gate_up, wl.w_down, wl.shared_gate_up, wl.shared_down, wk.F32, K, sim, 1, 0.3)
    assert ref.min_gap > 1e-9
    layer.run_decode()
    check_routing(layer.routing_to_host(), ref, layer.cfg)
    got = layer.out_to_host_f64()
    assert np.linalg.norm(got - ref.out_sere) <= 1e-6 * np.linalg.norm(ref.out_sere)
    assert np.abs(got - ref.out_sere).max() <= 1e-5 * np.abs(ref.out_sere).max()


# 40 experts own 1, 15, 16, 17, ... rows up to two and three items (average about 90: items of 96 rows)
EDGE_COUNTS = [1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 79, 80, 81, 95, 96, 97, 111, 112, 113, 127, 128, 129,
               159, 160, 161, 191, 192, 193, 223, 288, 289, 90, 90, 90, 90, 90, 91]


def test_rows_around_tile_and_item_edges(dev):  # noqa: F811
    """Planted routing: expert e owns exactly EDGE_COUNTS[e] rows; every token is compared."""
    pairs = pairs_with_counts(EDGE_COUNTS)
    T, M, K, dh, dm = len(pairs), len(EDGE_COUNTS), 2, 448, 320
    spec = wk.custom_spec("tile_edges", wk.BF16, dh, M, K, dm, 1, T, 8800, calib_batches=1, calib_tokens=4)
    wl = wk.make_workload(spec)
    plant_routing(wl, pairs)
    sim = pins.rand_sim(8800, M)
    layer = dev.DeviceLayer.from_workload(wl, sim, K, 0.0)
    ref = oracle.layer(wl.hidden, wl.router_w, wl.w_gate_up, wl.w_down, wl.shared_gate_up, wl.shared_down, wk.BF16, K, sim, K, 0.0)
    assert ref.count_after.tolist() == EDGE_COUNTS
    layer.run_decode()
    check_routing(layer.routing_to_host(), ref, layer.cfg)
    check_output(layer.out_to_host_f64(), ref.out_sere, wk.BF16, "edges")


@pytest.mark.parametrize("n", [33, 64, 100, 129, 300])
def test_similarity_items(dev, n):  # noqa: F811
    """Calibration batches that are cut into several items per expert."""
    spec = wk.custom_spec(f"simtile{n}", wk.BF16, 320, 24, 2, 448, 0, 4, 6600 + n, twin_src=0, twin_dst=12, twin_n=12,
                          calib_batches=1, calib_tokens=n)
    wl = wk.make_workload(spec)
    got = dev.similarity_on_device(wl).cpu().numpy()
    want = oracle.similarity_frobenius(wl.calib, wl.w_gate_up, wl.w_down, spec.dtype)
    assert np.abs(got - want).max() <= 5e-3, np.abs(got - want).max()


@pytest.mark.parametrize("dtype", [wk.BF16, wk.F32])
@pytest.mark.parametrize("inter", [1216, 192])
@pytest.mark.parametrize("metric", ["frobenius", "cosine", "cka_linear"])
def test_similarity_groups_of_batches(dev, metric, inter, dtype):  # noqa: F811
    """Seven batches of 60 tokens on layers of 11 to 71 MB: groups of four and a smaller last one.  Against the oracle, and against workspaces that hold smaller groups: a batch's outputs take the
    same sums whatever group it is in, so only the fp64 sums of the pair stage are split differently, which the fp32 result
    shows in its last place at most (values up to 1: 6e-8, two results)."""
    import torch
    from paper_2602_07616_amd import binding as B
    spec = wk.custom_spec("simgroups", dtype, 512, 19, 2, inter, 0, 4, 6900, twin_src=0, twin_dst=9, twin_n=9,
                          calib_batches=7, calib_tokens=60)
    wl = wk.make_workload(spec)
    got = dev.similarity_on_device(wl, metric=metric).cpu().numpy()
    ref = {"frobenius": oracle.similarity_frobenius, "cosine": oracle.similarity_cosine,
           "cka_linear": oracle.similarity_cka_linear}[metric]
    want = ref(wl.calib, wl.w_gate_up, wl.w_down, spec.dtype)
    tol = 1e-5 if dtype == wk.F32 else 5e-3
    assert np.abs(got - want).max() <= tol, np.abs(got - want).max()
    flag = {"frobenius": 0, "cosine": B.SERE_FLAG_SIM_COSINE, "cka_linear": B.SERE_FLAG_SIM_CKA_LINEAR}[metric]
    cfg = B.make_config(60, 512, 19, 2, inter, 0, dtype, 1, 0.0, flag)
    gu, dn, calib = (dev.to_device(a, dtype) for a in (wl.w_gate_up, wl.w_down, wl.calib))
    sim = torch.empty((19, 19), dtype=torch.float32, device="cuda")
    whole = B.sere_similarity_workspace_bytes(cfg, 60)
    for share in (0.8, 0.6, 0.3):           # groups of three, two and one
        small = torch.empty(int(whole * share), dtype=torch.uint8, device="cuda")
        sim.fill_(-3.0)
        B.sere_similarity(cfg, calib, 7, 60, gu, dn, sim, small)
        diff = np.abs(sim.cpu().numpy() - got).max()
        print(f"groups {metric} d_m {inter} dtype {dtype}: {share} of the workspace, differs by {diff:.1e}", flush=True)
        assert diff <= 1.2e-7, (share, diff)
    with pytest.raises(B.SereError) as err:
        B.sere_similarity(cfg, calib, 7, 60, gu, dn, sim, torch.empty(whole // 16, dtype=torch.uint8, device="cuda"))
    assert err.value.status == B.SERE_ERR_WORKSPACE_TOO_SMALL


@pytest.mark.parametrize("metric", ["frobenius", "cosine", "cka_linear"])
def test_similarity_stays_inside_its_workspace(dev, metric):  # noqa: F811
    """31 batches of 7 tokens, groups of 16 and 15, at sizes where the smaller group has more Gram slices in all: nothing
    behind exactly the bytes asked for changes."""
    import torch
    from paper_2602_07616_amd import binding as B
    flag = {"frobenius": 0, "cosine": B.SERE_FLAG_SIM_COSINE, "cka_linear": B.SERE_FLAG_SIM_CKA_LINEAR}[metric]
    cfg = B.make_config(7, 768, 128, 1, 64, 0, B.SERE_F32, 1, 0.0, flag)
    g = torch.Generator(device="cuda").manual_seed(5)
    gu, dn, calib = (torch.empty(shape, device="cuda").normal_(0.0, std, generator=g)
                     for shape, std in (((128, 128, 768), 0.02), ((128, 768, 64), 0.02), ((31, 7, 768), 1.0)))
    sim = torch.full((128, 128), -3.0, device="cuda")
    need = B.sere_similarity_workspace_bytes(cfg, 7)
    room = torch.full((need + (1 << 20),), 0x5A, dtype=torch.uint8, device="cuda")
    B.sere_similarity(cfg, calib, 31, 7, gu, dn, sim, room[:need])
    assert (room[need:] == 0x5A).all()
    assert (torch.diagonal(sim) - 1.0).abs().max() <= 1e-6 and torch.isfinite(sim).all()


def test_every_launch_of_the_pair_stage_is_timed(dev):  # noqa: F811
    """The reported stage is everything after the experts' forward pass, for every metric."""
    from paper_2602_07616_amd import binding as B
    spec = wk.custom_spec("simtimed", wk.BF16, 320, 20, 2, 192, 0, 4, 6980, calib_batches=3, calib_tokens=12)
    wl = wk.make_workload(spec)
    weights = (None, dev.to_device(wl.w_gate_up, wk.BF16), dev.to_device(wl.w_down, wk.BF16))
    for kwargs, launches in (({"metric": "frobenius"}, 4), ({"metric": "cosine"}, 5), ({"metric": "cka_linear"}, 3),
                             ({"cka": ("rbf", 1.0, 0.0)}, 4)):
        B.sere_stage_timing(True)
        dev.similarity_on_device(wl, weights, **kwargs)
        ms, n = B.sere_stage_timing_read()
        B.sere_stage_timing(False)
        assert n["gate_up"] == 3 and n["sim_pairs"] == 3 * launches, (kwargs, n)


def test_cosine_of_zero_outputs_and_group_in_place_of_h(dev):  # noqa: F811
    """An expert whose down projection is zero has cosine 0 with every expert, itself included; d_m = 64 makes
    the Gram buffers larger than the place of h that they start in."""
    spec = wk.custom_spec("coszero", wk.BF16, 448, 70, 2, 64, 0, 4, 6950, calib_batches=2, calib_tokens=33)
    wl = wk.make_workload(spec)
    wl.w_down[5] = 0
    got = dev.similarity_on_device(wl, metric="cosine").cpu().numpy()
    want = oracle.similarity_cosine(wl.calib, wl.w_gate_up, wl.w_down, spec.dtype)
    assert (got[5] == 0).all() and (got[:, 5] == 0).all()
    assert np.abs(got - want).max() <= 5e-3
