"""Similarity on layers of at most 8 MiB of weights, whose batches are taken in groups as those of larger ones: against the
oracle, against smaller groups, and while stages are timed.  The CPU test checks the groups' layouts."""
import os
import subprocess

import numpy as np
import pytest

import oracle
from paper_2602_07616_amd import binding as B, workloads as wk
from .test_gpu_parity import dev  # noqa: F401
from .test_similarity_plan import HERE, METRICS, draws

# dtype, d_h, M, d_m, tokens, batches
CASES = [
    (wk.BF16, 320, 19, 192, 12, 20),     # groups of 16 and a rest of four
    (wk.F32, 256, 9, 128, 100, 9),       # ten batches would fit
    (wk.BF16, 128, 70, 128, 33, 3),      # more than 64 experts
    (wk.F32, 64, 5, 64, 4, 2),           # the smallest
]
FLAGS = {"frobenius": 0, "cosine": B.SERE_FLAG_SIM_COSINE, "cka_linear": B.SERE_FLAG_SIM_CKA_LINEAR}


@pytest.mark.gpu
@pytest.mark.parametrize("metric", list(FLAGS))
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(v) for v in c))
def test_small_layers_in_groups(dev, case, metric):  # noqa: F811
    import torch
    dtype, dh, M, dm, n, batches = case
    print(f"small similarity {case} {metric}", flush=True)
    spec = wk.custom_spec("simsmall", dtype, dh, M, 2, dm, 0, 4, 9900 + n, twin_src=0, twin_dst=M // 2, twin_n=M // 2,
                          calib_batches=batches, calib_tokens=n)
    wl = wk.make_workload(spec)
    got = dev.similarity_on_device(wl, metric=metric).cpu().numpy()
    ref = {"frobenius": oracle.similarity_frobenius, "cosine": oracle.similarity_cosine, "cka_linear": oracle.similarity_cka_linear}[metric]
    want = ref(wl.calib, wl.w_gate_up, wl.w_down, spec.dtype)
    tol = 1e-5 if dtype == wk.F32 else 5e-3
    assert np.abs(got - want).max() <= tol, np.abs(got - want).max()
    cfg = B.make_config(n, dh, M, 2, dm, 0, dtype, 1, 0.0, FLAGS[metric])
    gu, dn, calib = (dev.to_device(a, dtype) for a in (wl.w_gate_up, wl.w_down, wl.calib))
    sim = torch.full((M, M), -3.0, dtype=torch.float32, device="cuda")
    whole = B.sere_similarity_workspace_bytes(cfg, n)
    small = torch.empty(int(whole * 0.4), dtype=torch.uint8, device="cuda")
    B.sere_similarity(cfg, calib, batches, n, gu, dn, sim, small)
    assert np.abs(sim.cpu().numpy() - got).max() <= 1.2e-7       # the fp64 sums are split differently: values up to 1, two results
    # stage timing changes nothing but what is recorded, and every batch counts
    whole_ws = torch.empty(whole, dtype=torch.uint8, device="cuda")
    pairs = {"frobenius": 4, "cosine": 5, "cka_linear": 3}[metric]
    for ws in (small, whole_ws):
        sim.fill_(-3.0)
        B.sere_similarity(cfg, calib, batches, n, gu, dn, sim, ws)
        untimed = sim.clone()
        B.sere_stage_timing(True)
        sim.fill_(-3.0)
        B.sere_similarity(cfg, calib, batches, n, gu, dn, sim, ws)
        ms, launches = B.sere_stage_timing_read()
        B.sere_stage_timing(False)
        assert launches["gate_up"] == launches["down"] == batches and launches["sim_pairs"] == pairs * batches and ms["sim_pairs"] > 0
        assert torch.equal(sim, untimed)


def test_layouts_of_groups(tmp_path):
    exe = str(tmp_path / "plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", os.path.join(HERE, "similarity_plan_main.cpp"), "-o", exe], check=True)
    cases = [c for c in draws(6000, 21) if c[2] * 3 * c[1] * c[3] * (4 if c[0] == B.SERE_F32 else 2) <= 8 << 20]
    cases += [(dt, dh, M, dm, n, f, b) for dt, dh, M, dm, n, b in CASES for f in METRICS]
    out = subprocess.run([exe], input="".join("%d %d %d %d %d %d %d\n" % c for c in cases), capture_output=True, text=True,
                         check=True).stdout.split("\n")
    assert len(cases) > 1000
    for case, line in zip(cases, out):
        groups = [tuple(int(v) for v in g.split()) for g in line.split(";") if g]
        M, n, batches = case[2], case[4], case[6]
        assert len(groups) == min(batches, max(min(8, 1024 // n), min(16, 256 // n), 1)), case
        assert [g[0] for g in groups] == sorted(g[0] for g in groups) and groups[-1][0] <= 1 << 30, case
        assert len({g[3:6] for g in groups}) == 1, case                     # the kernels and the slices: a call's sums
        for g, (_, items, rows, tile_gu, tile_dn, _, splits, _, item_bytes, part_bytes, _, y, h, parts, blocks, *_) in enumerate(groups, 1):
            assert M * items * 4 <= item_bytes and (items - 1) * rows < n * g <= items * rows, case
            assert rows == 32 or (tile_gu and tile_dn), case
            if case[5] == B.SERE_FLAG_SIM_CKA_LINEAR:
                assert M * g * blocks * n * 8 <= h and (parts == 1 or g * parts * M * M * 8 <= y), case
            else:
                assert g * splits * (M * M + 96) * 8 <= part_bytes, case
