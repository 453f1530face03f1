"""The interaction sums in one dimension by their modes (the library's default
there) against the oracle's sums over every pair, pathwise, and against the
pair kernels: sizes around a block and a partial row, several systems, both
sizes of a row, clouds so wide that many modes or none are taken, particles
that are not finite.

Tolerances: a step moves a particle by h times its pair term (|K| < 1), whose
FP64 error from the modes is below 40 rounding units at the widths tried
here, so states stay within 1e-13; the FP32 modes carry their state in 24
bits, 2e-6 over a few steps as for the pair kernels' summation order."""
import sys

import numpy as np
import pytest

import oracle
from paper_2105_09688_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-13, "fp32": 2e-6, "fp32_kahan": 2e-6}
H = 2.0 ** -6


def _say(msg):
    print(f"[gpu-modes] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    return torch


def _ssm(w, precision, **kw):
    from paper_2105_09688_amd.ssm import SSM
    return SSM(w, precision=precision, **kw)


def _err(got, ref):
    return float(np.max(np.abs(got - ref) / np.maximum(1.0, np.abs(ref))))


def _w(sizes, ell=1.0, steps=2):
    w = W.with_systems(W.small_parity(n_ens=1, h=H, h_fine=H / 4), [(n, e, H) for e, n in enumerate(sizes)])
    w["b"]["ell"] = ell
    w["T"] = steps * H
    return w


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_kahan"])
def test_sizes_match_oracle(precision):
    """One context of systems of 1 to 4099 particles (a block is 256)."""
    w = _w([1, 2, 63, 255, 256, 257, 1000, 4099])
    ref = oracle.run(w)
    with _ssm(w, precision, persistent=-1) as s:
        s.run()
        errs = [_err(s.state(k), r) for k, r in enumerate(ref)]
    _say(f"sizes {precision}: {['%.1e' % e for e in errs]}")
    assert max(errs) <= TOL[precision]


@pytest.mark.parametrize("ell,N", [(0.25, 3000), (0.01, 1000), (0.01, 20011), (0.002, 20011), (30.0, 3000)])
def test_width_of_the_cloud(ell, N):
    """Kernel widths from far below the spacing of the particles (direct sums
    take over: too many modes for the particle count) to far above the cloud
    (16 modes), in FP64 and FP32, against the oracle and the pair kernels."""
    w = _w([N], ell=ell, steps=1)
    ref = oracle.run(w)[0]
    for precision in ("fp64", "fp32_kahan"):
        with _ssm(w, precision, persistent=-1) as a, _ssm(w, precision, pair_scheme="symmetric") as b:
            a.run()
            b.run()
            got, pairs = a.state(0), b.state(0)
        _say(f"ell={ell} N={N} {precision}: oracle {_err(got, ref):.1e}, pair kernel {_err(got, pairs):.1e}")
        assert _err(got, ref) <= TOL[precision] and _err(got, pairs) <= TOL[precision]


def test_rows_of_1024_and_totals():
    """A context of more than 2^19 particles: rows of 1024 particles, added up
    once per system; ragged sizes, the largest system sampled."""
    w = _w([600_001, 700, 1025], steps=1)
    idx = np.array([0, 1, 255, 1023, 1024, 299_999, 600_000])
    for precision in ("fp64", "fp32"):
        with _ssm(w, precision) as s:
            s.run()
            got = s.states()
        for k, (N, e, h) in enumerate(w["systems"]):
            at = idx[idx < N] if N > 5000 else np.arange(N)
            ref = oracle.step_at(w, e, h, 0, oracle.init_state(w, e, N), at)
            _say(f"system {k} {precision}: {_err(got[k][:, at], ref):.1e}")
            assert _err(got[k][:, at], ref) <= TOL[precision]


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_a_particle_that_is_not_finite_spreads(bad):
    """As through the pair kernels: every particle of its system that meets a
    NaN becomes one (an infinite particle gives inf x 0), other systems stay."""
    from paper_2105_09688_amd import SSMError
    w = _w([700, 300], steps=2)
    ref = oracle.run(w)
    out = []
    for kw in (dict(persistent=-1), dict(pair_scheme="symmetric")):
        with _ssm(w, "fp64", **kw) as s:
            X = s.state(0)
            X[0, 5] = bad
            with pytest.raises(SSMError):
                s.set_state(0, X)
            s.step(2)
            out.append(_states_despite_flag(s))
    assert np.isnan(out[0][0]).all() and np.array_equal(np.isnan(out[0][0]), np.isnan(out[1][0]))
    assert _err(out[0][1], ref[1]) <= TOL["fp64"]


def _states_despite_flag(s):
    """Final states of a context whose sync reports non-finite particles (the copy is made all the same)."""
    import ctypes as C
    from paper_2105_09688_amd import _lib
    got = []
    for k, N in enumerate(s.N):
        a, n = np.zeros((1, N)), C.c_int64()
        _lib.load().ssm_get_state(s._h, k, 0, a.ctypes.data_as(C.POINTER(C.c_double)), C.byref(n))
        got.append(a)
    return got


def test_sampler_after_persistent_ticks():
    """Training rows drawn after ticks of the small-system kernel: the exact
    term of the rows equals the oracle's at the current Y*."""
    w = _w([900], steps=4)
    with _ssm(w, "fp64") as s:
        s.step(3)
        U, T = s.surrogate_samples(2000, seed=4)
        Y = s.state(0, "y")
    K = oracle.pair_sum(Y, 1.0)
    order = np.argsort(Y[0])
    at = order[np.searchsorted(Y[0], U[:, 0].double().cpu().numpy() , sorter=order).clip(0, 899)]
    near = np.abs(Y[0][at] - U[:, 0].cpu().numpy()) <= 1e-6
    assert near.mean() > 0.4
    assert np.max(np.abs(K[0][at] - T[:, 0].cpu().numpy())[near]) <= 1e-6


@pytest.mark.parametrize("case", ["one", "strides"])
def test_graphs_of_several_ticks_are_the_launches(case):
    """Past 64 ticks a context's longer step calls leave as graphs of 4, 8 or
    16 ticks; steps of one tick never do.  Both runs are equal bit for bit,
    with reads and moments between replays, ticks left over (the device tick
    counter is set again), a state moved to another step and a newly bound
    state buffer (the graphs are made again)."""
    w = (_w([3000], steps=400) if case == "one" else
         W.batched(n_ens=2, levels=(5, 6, 7), h_fine=2.0 ** -9, sizes=[3000, 300]))
    w["T"] = 400 * max(s[2] for s in w["systems"])
    with _ssm(w, "fp32_kahan", persistent=-1) as a, _ssm(w, "fp32_kahan", persistent=-1) as b:
        def same(note):
            for k in range(len(w["systems"])):
                assert np.array_equal(a.state(k), b.state(k)), (note, k)

        def both(n):
            for _ in range(n):
                a.step(1)
            b.step(n)

        for n in (64, 4, 4, 8, 16, 10, 12, 32, 7, 1, 60):
            both(n)
            same(n)
            assert np.array_equal(a.moments(0)[0], b.moments(0)[0])
        for s in (a, b):
            for k, (N, e, h) in enumerate(w["systems"]):
                s.set_state(k, s.state(k), step=round(64 * max(x[2] for x in w["systems"]) / h))
        both(36)
        same("moved")
        buf = b.bind_state()
        both(20)
        same("bound")
        assert buf.shape[0] == 1


def test_graphs_stay_out_of_a_callers_capture(torch_cuda):
    """A context on a stream that the caller is capturing launches tick by
    tick into the capture, also past 64 ticks; the caller's graph then takes
    the same four ticks as a context without it."""
    torch = torch_cuda
    w = _w([3000], steps=200)
    st = torch.cuda.Stream()
    with _ssm(w, "fp64", persistent=-1, stream=st) as a, _ssm(w, "fp64", persistent=-1) as b:
        a.step(80)
        b.step(80)
        a.sync()
        X = a.state(0)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            a.step(4)
        g.replay()
        torch.cuda.synchronize()
        b.step(4)
        assert np.array_equal(a.state(0), b.state(0)) and not np.array_equal(a.state(0), X)
