"""Network ticks that leave as graphs of several (a call with many of them, in
a context past its first 64 ticks) against the same ticks one call each, bit
for bit: with residuals and before the first check, in gain mode, after new
weights and a new state, with a caller's state buffer, in one dimension."""
import numpy as np
import pytest

from paper_2105_09688_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    return torch


def _run(d, precision, mode, whole, N=1500, check=24):
    from paper_2105_09688_amd.ssm import SSM, mlp_init
    h = 2.0 ** -9
    w = (W.surrogate_d2(N=N, h=h, h_fine=h / 2) if d == 2 else
         W.with_systems(W.small_parity(n_ens=1, h=h, h_fine=h / 2), [(N, 0, h), (700, 1, 2 * h)]))
    w["T"] = 400 * h

    def go(n):
        for k in [n] if whole else [1] * n:
            s.step(k)

    out = []
    with SSM(w, precision=precision, persistent=-1) as s:
        s.surrogate_load(0.3 * mlp_init(d, seed=2))
        go(2)
        s.surrogate_enable(check_every=check, tol=1e9, mode=mode)
        go(120)
        out.append(s.states())
        s.surrogate_load(0.5 * mlp_init(d, seed=3))
        go(60)
        s.set_state(0, 0.5 * s.state(0), step=200)
        go(70)
        out.append(s.states())
        if d == 2:
            X = s.bind_state()
            go(50)
            s.sync()
            out.append([X.cpu().numpy()])
        info = s.info()
    return out, {k: info[k] for k in ("tick", "surr_ticks", "surr_checks", "surr_fallback_ticks", "surr_last_err", "newton_max_seen")}


@pytest.mark.parametrize("d,precision,mode", [(2, "fp32_kahan", "residual"), (2, "fp64", "residual"), (2, "fp32", "gain"),
                                              (1, "fp64", "residual")])
def test_graphs_equal_single_ticks(d, precision, mode):
    a, ia = _run(d, precision, mode, True)
    b, ib = _run(d, precision, mode, False)
    print(f"[gpu-surrogate-graphs] d={d} {precision} {mode} {ia}", flush=True)
    assert ia == ib and ia["surr_ticks"] > 150
    for p, q in zip(a, b):
        for x, y in zip(p, q):
            assert np.array_equal(x, y)
