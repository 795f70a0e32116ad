"""Infinities and NaN in the experts' weights or from overflow: what a layer or a similarity estimation returns where
a plain sum gives one.  (Hidden states, router and similarities have to be finite; expert weights need not be.)"""
import numpy as np
import pytest

import oracle
from paper_2602_07616_amd import workloads as wk
from . import pins
from .test_gpu_parity import dev  # noqa: F401

pytestmark = pytest.mark.gpu

HUGE = np.float32(2.5e38)    # finite; the sum of two is not


def f32_layer(wl, ref):
    """The layer in numpy, every projection rounded to fp32 (which is where a sum becomes infinite)."""
    out = np.zeros(wl.hidden.shape, dtype=np.float64)
    x = wl.hidden.astype(np.float64)
    dm = wl.spec.inter
    with np.errstate(all="ignore"):
        for e in range(wl.spec.experts):
            t, k = np.nonzero(ref.rerouted_ids == e)
            if len(t) == 0:
                continue
            gu = np.einsum("tk,jk->tj", x[t], wl.w_gate_up[e].astype(np.float64)).astype(np.float32)
            g, u = gu[:, :dm], gu[:, dm:]
            h = (g / (1.0 + np.exp(-g.astype(np.float64)))).astype(np.float32) * u
            y = np.einsum("tj,rj->tr", h.astype(np.float64), wl.w_down[e].astype(np.float64)).astype(np.float32)
            out[t] += ref.topk_weights[t, k][:, None] * y
    return out


# (tokens, experts = K): the two launches of calls of few slots, the vector-ALU kernels, the persistent ones
F32_CALLS = {(4, 3): "few", (4, 9): "alu", (40, 3): "tile"}


@pytest.mark.parametrize("tokens,M", F32_CALLS)
@pytest.mark.parametrize("where", ["up_inf_first", "up_inf_last", "up_overflow", "up_overflow_far", "down_inf", "down_neg_inf"])
def test_fp32_sum_that_overflows_is_infinite(dev, tokens, M, where):  # noqa: F811
    """One infinite weight, or two finite ones whose products overflow (in one 32-wide step, or in two), in the first,
    a middle or the last step of the contraction: the sums are infinite, with the sign of the exact sum."""
    dh, K, dm = 1472, M, 192
    spec = wk.custom_spec("nonfinite", wk.F32, dh, M, K, dm, 0, tokens, 7300, calib_batches=1, calib_tokens=4)
    wl = wk.make_workload(spec)
    up, down = wl.w_gate_up[2][dm:], wl.w_down[2]
    if where == "up_inf_first":
        up[7, 3] = np.inf
    elif where == "up_inf_last":
        up[7, dh - 1] = np.inf
    elif where == "up_overflow":
        up[7, 640] = up[7, 641] = HUGE
        wl.hidden[:, 640:642] = 1.0
    elif where == "up_overflow_far":
        up[7, 5] = up[7, dh - 2] = HUGE
        wl.hidden[:, [5, dh - 2]] = 1.0
    else:
        down[11, dm // 2] = np.inf if where == "down_inf" else -np.inf
    sim = pins.rand_sim(7300, M)
    layer = dev.DeviceLayer.from_workload(wl, sim, K, 0.0)
    ref = oracle.route(wl.hidden, wl.router_w, wk.F32, K, sim, K, 0.0)
    assert (ref.rerouted_ids == 2).any()
    print(f"nonfinite {where} {tokens} {M}", flush=True)
    layer.run_decode()
    got, want = layer.out_to_host_f64(), f32_layer(wl, ref)
    assert np.isinf(want).any() and not np.isnan(want).any()
    assert not np.isnan(got).any(), np.argwhere(np.isnan(got))[:4]
    assert np.array_equal(np.isinf(got), np.isinf(want)) and np.array_equal(np.signbit(got), np.signbit(want))
    fin = np.isfinite(want)
    # as in the finite fp32 tests: compensated sums stay near 2e-7
    assert np.linalg.norm(got[fin] - want[fin]) <= 1e-6 * np.linalg.norm(want[fin])


@pytest.mark.parametrize("M", [70, 60, 12])     # blocks of 64 x 64 experts; 16 tiles of the kernel of up to 64 experts, one
@pytest.mark.parametrize("dtype", [wk.F32, wk.BF16])
def test_cosine_of_nonfinite_outputs(dev, dtype, M):  # noqa: F811
    """A token contributes the quotient where the product of the two norms is positive (that is NaN if one of them is
    infinite), and 0 where it is not: a zero output or one with a NaN, whatever the other one is."""
    spec = wk.custom_spec("cosnan", dtype, 320, M, 2, 64, 0, 4, 6960, calib_batches=2, calib_tokens=17)
    wl = wk.make_workload(spec)
    zero, nan, inf = 5, 7, 9
    wl.w_down[zero] = 0
    wl.w_down[nan, 100, 3] = wk.to_storage(np.float32([np.nan]), dtype)[0]
    wl.w_down[inf, 200, 60] = wk.to_storage(np.float32([np.inf]), dtype)[0]
    print(f"cosine nonfinite dtype {dtype}, {M} experts", flush=True)
    got = dev.similarity_on_device(wl, metric="cosine").cpu().numpy()
    want = oracle.similarity_cosine(wl.calib, wl.w_gate_up, wl.w_down, dtype)
    assert (want[nan] == 0).all() and np.isnan(want[inf]).sum() == M - 2       # the oracle has the same reading
    assert np.array_equal(np.isnan(got), np.isnan(want))
    fin = ~np.isnan(want)
    assert (got[[zero, nan]] == 0).all() and (got[:, [zero, nan]] == 0).all()
    # as in the finite cosine tests
    assert np.abs(got[fin] - want[fin]).max() <= (1e-5 if dtype == wk.F32 else 5e-3)


def test_cosine_of_one_token_with_nan_outputs(dev):  # noqa: F811
    """A token whose outputs overflow to NaN in fp32 contributes 0: the others' mean is left, over all tokens."""
    n = 20
    spec = wk.custom_spec("costoken", wk.F32, 320, 33, 2, 64, 0, 4, 6970, calib_batches=1, calib_tokens=n)
    wl = wk.make_workload(spec)
    others = np.delete(wl.calib, 6, axis=1)
    want = oracle.similarity_cosine(others, wl.w_gate_up, wl.w_down, wk.F32) * (n - 1) / n
    wl.calib[0, 6] *= np.float32(1e30)
    got = dev.similarity_on_device(wl, metric="cosine").cpu().numpy()
    assert np.abs(got - want).max() <= 1e-5


@pytest.mark.parametrize("kernel", ["linear", "rbf", "poly"])
@pytest.mark.parametrize("n", [17, 60])     # blocks of 16 and of 32 rows
def test_alignment_with_nonfinite_outputs(dev, n, kernel):  # noqa: F811
    """An expert whose outputs are zero, infinite or NaN has no positive self-term, so its similarities are 0; the others' are
    what they are without it."""
    spec = wk.custom_spec("ckanan", wk.F32, 320, 20, 2, 64, 0, 4, 6975, calib_batches=2, calib_tokens=n)
    wl = wk.make_workload(spec)
    zero, nan, inf = 5, 7, 18
    finite = [e for e in range(20) if e not in (nan, inf)]
    outs = oracle.moe_layer(wl.calib[0], wl.w_gate_up, wl.w_down, None, None, wk.F32, np.zeros((n, 1), dtype=np.int32), np.ones((n, 1)))
    norm2 = float(np.mean(np.sum(outs * outs, axis=1)))
    p0, p1 = {"linear": (0.0, 0.0), "rbf": (np.sqrt(2.0 * norm2), 0.0), "poly": (norm2, 3.0)}[kernel]
    wl.w_down[zero] = 0
    wl.w_down[nan, 100, 3] = np.nan
    wl.w_down[inf, 200, 60] = np.inf
    print(f"alignment nonfinite {kernel}, {n} tokens", flush=True)
    got = dev.similarity_on_device(wl, cka=(kernel, p0, p1)).cpu().numpy()
    want = oracle.similarity_cka(wl.calib, wl.w_gate_up[finite], wl.w_down[finite], wk.F32, kernel, p0, p1)
    assert (got[[nan, inf]] == 0).all() and (got[:, [nan, inf]] == 0).all()
    # as in the finite tests; the zero expert's kernels are constant, so its self-term is 0 but for rounding
    rest = [e for e in finite if e != zero]
    at = [finite.index(e) for e in rest]
    assert np.abs(got[np.ix_(rest, rest)] - want[np.ix_(at, at)]).max() <= 1e-5
    if kernel == "linear":
        assert (got[zero] == 0).all() and (got[:, zero] == 0).all()
