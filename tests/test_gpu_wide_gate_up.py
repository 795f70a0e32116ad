"""The gate/up kernel with units of 256 weight rows x 256 token rows and two stages, which similarity calls take for items of
256 rows: whole and part-filled token tiles, a last block of weight rows that is half empty, one k step and several, more
units than workgroups."""
import os
import subprocess

import numpy as np
import pytest

import oracle
from paper_2602_07616_amd import workloads as wk
from .test_gpu_parity import dev  # noqa: F401

# M, d_h, d_m, tokens, batches
CASES = [
    (64, 64, 448, 241, 1),     # one k step, a last token tile of one row, the last block of 128 indices half empty
    (40, 192, 448, 250, 1),    # three k steps
    (60, 192, 320, 128, 2),    # a group of two batches
    (40, 64, 512, 241, 1),     # whole blocks
    (100, 128, 576, 256, 1),   # 500 units
]
MAIN = """
#include <cstdio>
#include "csrc/similarity_plan.hpp"
int main() {
  sere_config c{};
  int n = 0, batches = 0;
  c.dtype = SERE_BF16;
  while (std::scanf("%d %d %d %d %d", &c.num_experts, &c.hidden, &c.inter, &n, &batches) == 5) {
    const int most = sere::sim_group(c, n), g = batches < most ? batches : most;
    const sere::SimLayout l = sere::make_sim_layout(c, n, g, g);
    std::printf("%d %d\\n", l.plan.item_rows, l.plan.wide_gate_up);
  }
}
"""


def test_the_cases_take_the_wide_kernel(tmp_path):
    src, exe = str(tmp_path / "main.cpp"), str(tmp_path / "main")
    with open(src, "w") as f:
        f.write(MAIN)
    pkg = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_07616_amd")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", pkg, src, "-o", exe], check=True)
    out = subprocess.run([exe], input="".join("%d %d %d %d %d\n" % c for c in CASES), capture_output=True, text=True, check=True)
    assert out.stdout.split("\n")[:-1] == ["256 1"] * len(CASES)


@pytest.mark.gpu
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
