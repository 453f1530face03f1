"""One-dimensional clouds that are wide against the kernel.  Where a context's
cloud is drawn so wide that its mode sums would be slower than sums over pairs,
it takes the pair kernels (or the tiled kernel of small systems) as before, bit
for bit, and is no slower than a context that asks for them by name.  Where a
cloud becomes that wide later, its sums run directly inside the mode kernels,
the sources in shares over several blocks: against the oracle.

Tolerances: a step moves a particle by h times its pair term (|K| < 1), summed
in at most 8 shares with a rounding each: 1e-13 in FP64; the FP32 modes carry
their state in 24 bits, 2e-6 (as in test_gpu_modes.py)."""
import time

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


def _w(sizes, ell, steps=8):
    w = W.with_systems(W.small_parity(n_ens=1, h=H, h_fine=H / 4), [(n, e, H) for e, n in enumerate(sizes)])
    w["b"]["ell"] = ell
    w["T"] = steps * H
    return w


@pytest.mark.parametrize("precision", ["fp64", "fp32_kahan"])
@pytest.mark.parametrize("sizes,ell,asked", [([1000], 0.02, dict(persistent=1)), ([2048], 0.005, dict(persistent=1)),
                                             ([300, 900], 0.02, dict(persistent=1)), ([4096], 0.005, dict(pair_scheme="symmetric")),
                                             ([8191], 0.002, dict(pair_scheme="symmetric")),
                                             ([20011, 3000], 0.001, dict(pair_scheme="symmetric"))])
def test_drawn_wide(sizes, ell, asked, precision):
    w = _w(sizes, ell)
    out = []
    for kw in ({}, asked):
        with _ssm(w, precision, **kw) as s:
            s.step(4)
            out.append(s.states())
    assert all(np.array_equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("precision", ["fp64", "fp32_kahan"])
@pytest.mark.parametrize("N,ell", [(300, 0.02), (1000, 0.005), (2048, 0.05), (2048, 0.005), (4096, 0.02), (8191, 0.02), (8191, 0.005),
                                   (65536, 0.002)])
def test_no_slower_than_asked_for_by_name(N, ell, precision):
    """Within 1.5 of the faster of what can be asked for (small differences are measured, not tested)."""
    w = _w([N], ell, steps=4096)

    def tick(**kw):
        with _ssm(w, precision, **kw) as s:
            s.step(72)
            s.sync()
            best = 1.0
            for _ in range(6):
                t = time.perf_counter()
                s.step(16)
                s.sync()
                best = min(best, (time.perf_counter() - t) / 16)
        return 1e6 * best

    own = tick()
    pairs = tick(pair_scheme="symmetric", persistent=-1)
    if N <= 2048:
        pairs = min(pairs, tick(persistent=1))
    print(f"[gpu-wide] N={N} ell={ell} {precision}: {own:.1f} us a tick, by name {pairs:.1f}", flush=True)
    assert own <= 1.5 * pairs


@pytest.mark.parametrize("precision", ["fp64", "fp32_kahan"])
@pytest.mark.parametrize("sizes", [[300], [1000, 257], [2048], [2049], [8191, 70], [40000], [65536]])
def test_wide_later(sizes, precision):
    """A context drawn narrow is given a cloud of thousands of widths and one with a particle far away."""
    w = _w(sizes, 1.0)
    rng = np.random.default_rng(7)
    for kind in ("wide", "outlier"):
        with _ssm(w, precision) as s:
            for k, (N, e, h) in enumerate(w["systems"]):
                x = rng.normal(size=(1, N)) * (400.0 if kind == "wide" else 0.7)
                if kind == "outlier":
                    x[0, N // 3] = 3000.0
                s.set_state(k, x)
            start = s.states()
            s.step(1)
            got = s.states()
        for k, (N, e, h) in enumerate(w["systems"]):
            at = np.unique(np.linspace(0, N - 1, 200).astype(int)) if N > 5000 else np.arange(N)
            ref = oracle.step_at(w, e, h, 0, start[k], at)
            err = np.max(np.abs(got[k][:, at] - ref) / np.maximum(1.0, np.abs(ref)))
            print(f"[gpu-wide] {kind} {sizes} {precision} system {k}: {err:.1e}", flush=True)
            assert err <= TOL[precision]


def test_wide_later_in_rows_of_1024():
    """As above past 2^19 particles, at sampled particles, in FP32 (a tick is 3.6e11 pairs)."""
    w = _w([600_001], 1.0)
    x = np.random.default_rng(8).normal(size=(1, 600_001)) * 4000.0
    with _ssm(w, "fp32_kahan") as s:
        s.set_state(0, x)
        x = s.states()[0]
        s.step(1)
        got = s.state(0)
    at = np.array([0, 1, 1023, 1024, 300_000, 600_000])
    ref = oracle.step_at(w, 0, H, 0, x, at)
    assert np.max(np.abs(got[:, at] - ref) / np.maximum(1.0, np.abs(ref))) <= TOL["fp32_kahan"]
