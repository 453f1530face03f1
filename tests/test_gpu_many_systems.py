"""Contexts of very many small one-dimensional systems: the buffers of the mode
sums and of the one-workgroup launches grow with the particles they serve and
not by fixed rows per system (device memory against a context of the pair
kernels), and such contexts step as the oracle does, by one launch and by
launches per tick, split over calls bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2105_09688_amd import workloads as W

pytestmark = pytest.mark.gpu
H = 2.0 ** -6


@pytest.fixture(scope="module", autouse=True)
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    return torch


def _w(n_sys, N):
    w = W.with_systems(W.small_parity(n_ens=1, h=H, h_fine=H), [(N, e, H) for e in range(n_sys)])
    w["T"] = 32 * H
    return w


@pytest.mark.parametrize("precision", ["fp64", "fp32_kahan"])
@pytest.mark.parametrize("persistent", [0, -1])
def test_memory(precision, persistent):
    """Increments of a tick and rows of 2 KB a system beside about 5 (FP32) or 8 KB that a system has in any case."""
    from paper_2105_09688_amd.ssm import SSM
    w = _w(20000, 50)
    with SSM(w, precision=precision, persistent=persistent) as a, SSM(w, precision=precision, pair_scheme="symmetric") as b:
        ma, mb = a.info()["device_bytes"], b.info()["device_bytes"]
    print(f"[gpu-many] {precision} persistent={persistent}: {ma / 1e6:.0f} MB, pair kernels {mb / 1e6:.0f}", flush=True)
    assert ma <= 1.5 * mb


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-13), ("fp32_kahan", 2e-6)])
@pytest.mark.parametrize("n_sys,N", [(9000, 30), (300, 700), (140000, 3)])
def test_steps(precision, tol, n_sys, N):
    """140000: totals of the rows are made (more than 2^17 row reads)."""
    from paper_2105_09688_amd.ssm import SSM
    w = _w(n_sys, N)
    some = [0, 1, n_sys // 2, n_sys - 1]
    ref = oracle.run(dict(W.with_systems(w, [w["systems"][k] for k in some]), T=4 * H))
    whole = None
    for persistent, plan in ((0, (4,)), (0, (1, 3)), (-1, (4,))):
        with SSM(w, precision=precision, persistent=persistent) as s:
            for n in plan:
                s.step(n)
            got = [s.state(k) for k in some]
        err = max(float(np.max(np.abs(g - r) / np.maximum(1.0, np.abs(r)))) for g, r in zip(got, ref))
        print(f"[gpu-many] {n_sys} x {N} {precision} persistent={persistent} {plan}: {err:.1e}", flush=True)
        assert err <= tol
        if persistent == 0:
            whole = whole or got
            assert all(np.array_equal(a, b) for a, b in zip(whole, got))


@pytest.mark.parametrize("precision", ["fp64", "fp32_kahan"])
@pytest.mark.parametrize("n_sys,N", [(1024, 50), (4096, 50), (2048, 300), (1024, 1000)])
def test_no_slower_than_the_pair_kernels(n_sys, N, precision):
    """Ordinary clouds in one workgroup each take a third to a half of the pair kernels' time; 1.2 times it is allowed."""
    import time

    from paper_2105_09688_amd.ssm import SSM
    w = _w(n_sys, N)
    w["T"] = 2048 * H

    def tick(**kw):
        with SSM(w, precision=precision, **kw) as s:
            s.step(72)
            s.sync()
            best = 1.0
            for _ in range(6):
                t = time.perf_counter()
                s.step(16)
                s.sync()
                best = min(best, (time.perf_counter() - t) / 16)
            return 1e6 * best, s.info()["persistent_ticks"] > 0

    (own, one), (pairs, _) = tick(), tick(pair_scheme="symmetric", persistent=-1)
    print(f"[gpu-many] {n_sys} x {N} {precision}: {own:.1f} us a tick, pair kernels {pairs:.1f}", flush=True)
    assert one and own <= 1.2 * pairs
