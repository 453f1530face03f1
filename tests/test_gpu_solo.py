"""Small one-dimensional systems, one workgroup each (the library's default up
to 2048 particles), against the oracle pathwise: the least and largest systems
of each kernel shape, several step sizes, clouds summed directly (too wide for
modes), no pair term, the mean in the implicit part; a run split over calls and
resumed in a new context, bit for bit.

Tolerances: a step moves a particle by h times its pair term (|K| < 1), whose
FP64 error from the modes is below 40 rounding units, and the implicit solve
and the update add a few roundings: 1e-13 over 8 steps.  The FP32 modes carry
their state in 24 bits: 2e-6."""
import numpy as np
import pytest

import oracle
from paper_2105_09688_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-13, "fp32_kahan": 2e-6}
H = 2.0 ** -6


@pytest.fixture(scope="module", autouse=True)
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    return torch


def _ssm(w, precision, **kw):
    from paper_2105_09688_amd.ssm import SSM
    return SSM(w, precision=precision, **kw)


def _w(kind, top):
    sizes = [1, top - 1, 2, top, top // 2 + 1]
    w = (W.ginzburg_landau(version=2, h_fine=H / 4) if kind == "mean" else
         W.ou(x0_std=0.5, h=H, h_fine=H / 4) if kind == "free" else W.small_parity(n_ens=1, h=H, h_fine=H / 4))
    w = W.with_systems(w, [(n, e, H * 2 ** (e % 2)) for e, n in enumerate(sizes)])
    if kind == "wide":  # some 2500 widths: every system is summed directly
        w["b"]["ell"] = 0.002
    w["T"] = 8 * H
    return w


@pytest.mark.parametrize("precision", ["fp64", "fp32_kahan"])
@pytest.mark.parametrize("kind", ["modes", "wide", "mean", "free"])
@pytest.mark.parametrize("top", [256, 512, 1024, 2048])
def test_against_the_oracle(kind, top, precision):
    w = _w(kind, top)
    print(f"[gpu-solo] {kind} {top} {precision}", flush=True)
    ref = oracle.run(w)
    with _ssm(w, precision) as s:
        s.run()
        assert s.info()["persistent_ticks"] == 8
        for k, r in enumerate(ref):
            err = np.max(np.abs(s.state(k) - r) / np.maximum(1.0, np.abs(r)))
            assert err <= TOL[precision], (k, err)
        whole = s.states()
    with _ssm(w, precision) as s:
        for n in (2, 4, 2):
            s.step(n)
            if n == 4:
                mid = s.states()
        assert all(np.array_equal(a, b) for a, b in zip(whole, s.states()))
    with _ssm(w, precision) as s:
        for k, x in enumerate(mid):
            s.set_state(k, x, step=6 // (1 + k % 2))
        s.step(2)
        assert all(np.array_equal(a, b) for a, b in zip(whole, s.states()))
