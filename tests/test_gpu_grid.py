"""The interaction sums of one large system in three dimensions by way of a
grid (the library's default there, and in two dimensions with a surrogate) against sums over every pair in 64 bits, at
the least size and beyond it, for clouds of one bin, of many, and flat ones;
clouds that it leaves to the pair kernels (too wide, or with a particle that
is not finite), bit for bit as an explicit choice of them; a step repeated
from the same state, and a context resumed after steps of both kinds.

Tolerances.  With the drift g K alone a step from x gives x + h g K / N, so
(x_1 - x) / h is the pair term K / N, |K / N| <= 0.6 ell.  FP64: the grid's
error is 1.1e-15 of the root mean square of K in one dimension, three of them
and the roundings of W^3 products are taken as 1e-13 of ell.  FP32: 4.6e-9 a
dimension, K / N and x_1 rounded to 24 bits (h = 1024 makes x_1 of the size of
h K / N): 8e-8 of ell, taken as 2e-7.  To both, the rounding u |x| of a scaled
coordinate, own and others', which moves K / N by at most as much, and the one
that is left of x_0 in the difference."""
import ctypes as C

import numpy as np
import pytest

from paper_2105_09688_amd import workloads as W

pytestmark = pytest.mark.gpu
H = 1024.0
TOL = {"fp64": 1e-13, "fp32": 2e-7, "fp32_kahan": 2e-7}
U = {"fp64": 2.0 ** -53, "fp32": 2.0 ** -24, "fp32_kahan": 2.0 ** -24}


@pytest.fixture(scope="module", autouse=True)
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    return torch


def _ssm(w, precision, **kw):
    from paper_2105_09688_amd.ssm import SSM
    return SSM(w, precision=precision, **kw)


def _w(N, std, ell=0.5, mean=(0.0, 0.0, 0.0)):
    w = W.precision_d3(N=N)
    w.update(T=4 * H, h_fine=H, systems=[(N, 0, H)], x0_mean=list(mean), x0_std=list(std),
             v=dict(rho=0.0, a=0.0, kappa=0.0, lam=0.0), sigma=dict(s0=[0.0] * 3, s1=[0.0] * 3, s2=[0.0] * 3))
    w["b"]["ell"] = ell
    w["allow_unstable_h"] = True
    return w


def _pairs(torch, X, ell, idx):
    Y = torch.tensor(X, device="cuda", dtype=torch.float64)
    out = torch.empty(len(X), len(idx), dtype=torch.float64, device="cuda")
    for a in range(0, len(idx), 256):
        z = Y[:, None, :] - Y[:, idx[a:a + 256], None]
        t = torch.exp((z * z).sum(0) * (-0.5 / ell ** 2))
        out[:, a:a + 256] = (z * t).sum(2) / Y.shape[1]
    return out.cpu().numpy()


CLOUDS = [((1.0, 1.0, 1.0), 0.5), ((0.02, 0.02, 0.02), 0.5), ((2.0, 0.1, 0.001), 0.5), ((1.0, 1.0, 0.0), 0.7), ((1.0, 2.0, 0.5), 4.0)]


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_kahan"])
@pytest.mark.parametrize("N", [20000, 65537])
def test_pair_term(torch_cuda, precision, N):
    for k, (std, ell) in enumerate(CLOUDS):
        w = _w(N, std, ell, mean=(0.0, 5.0, -300.0) if k == 0 and precision == "fp64" else (0.0, 0.0, 0.0))
        print(f"[gpu-grid] {precision} N={N} cloud {std} ell={ell}", flush=True)
        with _ssm(w, precision) as s:
            x0 = s.state(0)
            s.step(1)
            x1 = s.state(0)
        idx = np.unique(np.concatenate([np.arange(64), np.argsort(x0[0])[[0, 1, -2, -1]], np.linspace(0, N - 1, 800).astype(int)]))
        err = np.abs((x1 - x0)[:, idx] / H - _pairs(torch_cuda, x0, ell, idx)).max() / ell
        print(f"[gpu-grid] error {err:.1e}", flush=True)
        assert err <= TOL[precision] + 2 * (1 + 1 / H) * U[precision] * np.abs(x0).max() / ell


def _set(s, X, step):
    """As set_state, which reports a particle that is not finite after it has copied it."""
    from paper_2105_09688_amd import _lib
    X = np.ascontiguousarray(X)
    _lib.load().ssm_set_state(s._h, 0, X.ctypes.data_as(C.POINTER(C.c_double)), step)


def _get(s):
    from paper_2105_09688_amd import _lib
    X, n = np.zeros((3, s.N[0])), C.c_int64()
    _lib.load().ssm_get_state(s._h, 0, 0, X.ctypes.data_as(C.POINTER(C.c_double)), C.byref(n))
    return X


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_left_to_the_pair_kernels(torch_cuda, precision):
    """Too wide, NaN and infinite: as the pair kernels asked for by name; and the grid again after them."""
    w = _w(32768, (1.0, 1.0, 1.0))
    rng = np.random.default_rng(5)
    clouds = [rng.normal(size=(3, 32768)) * 40.0, rng.normal(size=(3, 32768)), rng.normal(size=(3, 32768))]
    clouds[1][1, 77] = np.nan
    clouds[2][0, 9] = np.inf
    for n, x in enumerate(clouds):
        print(f"[gpu-grid] left to the pair kernels {precision} {n}", flush=True)
        with _ssm(w, precision) as s, _ssm(w, precision, pair_scheme="symmetric") as p:
            for c in (s, p):
                _set(c, x, 0)
                c.step(1)
            assert np.array_equal(_get(s), _get(p), equal_nan=True)
            y = rng.normal(size=(3, 32768))
            with _ssm(w, precision) as f:
                for c in (s, f):
                    _set(c, y, 2)
                    c.step(1)
                assert np.array_equal(_get(s), f.state(0))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("graphs", [False, True])
def test_two_dimensions(torch_cuda, precision, graphs):
    """A context takes the grid from its first check on, then in its captured ticks too."""
    from paper_2105_09688_amd.ssm import mlp_init
    N, ell = 24000, 0.6
    w = _w(N, (1.0, 1.0, 1.0), ell)
    w.update(d=2, x0_mean=[0.0, 2.0], x0_std=[1.0, 0.3], sigma=dict(s0=[0.0] * 2, s1=[0.0] * 2, s2=[0.0] * 2))
    out = []
    with _ssm(w, precision, graphs=graphs) as s:
        x0 = s.state(0)
        s.surrogate_load(mlp_init(2, seed=1))
        for every in (0, 16, 0):  # an exact tick, a check, an exact tick
            s.surrogate_enable(check_every=every, tol=1e9, mode="residual")
            s.set_state(0, x0, step=0)
            s.step(1)
            out.append(s.state(0))
    assert np.array_equal(out[1], out[2])
    out.pop()
    assert not np.array_equal(*out)  # two ways, to the same result:
    idx = np.linspace(0, N - 1, 800).astype(int)
    ref = _pairs(torch_cuda, x0, ell, idx)
    err = [np.abs((x1 - x0)[:, idx] / H - ref).max() / ell for x1 in out]
    print(f"[gpu-grid] two dimensions {precision}: pair kernels {err[0]:.1e}, grid {err[1]:.1e}", flush=True)
    assert err[1] <= TOL[precision] + 2 * (1 + 1 / H) * U[precision] * np.abs(x0).max() / ell


@pytest.mark.parametrize("precision", ["fp64", "fp32_kahan"])
def test_repeats_bit_for_bit(torch_cuda, precision):
    """Steps in one call, one by one, in graphs, and resumed in a new context."""
    w = W.precision_d3(N=40001)
    out = []
    for kw, plan in (({}, (4,)), ({}, (1, 1, 2)), ({"graphs": True}, (1, 3))):
        with _ssm(w, precision, **kw) as s:
            for n in plan:
                s.step(n)
            out.append(s.state(0))
    with _ssm(w, precision) as s:
        s.step(3)
        mid = s.state(0)
    with _ssm(w, precision) as s:
        s.set_state(0, mid, step=3)
        s.step(1)
        out.append(s.state(0))
    for x in out[1:]:
        assert np.array_equal(out[0], x)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_two_dimensions_by_configuration(torch_cuda, precision):
    """How exact ticks are summed follows from how a context was configured: rows sampled
    in between change nothing, nor does which ticks were checks, and a context resumed
    from the state repeats the run bit for bit."""
    from paper_2105_09688_amd.ssm import mlp_init
    N = 24000
    w = _w(N, (1.0, 1.0, 1.0), 0.6)
    w.update(d=2, x0_mean=[0.0, 2.0], x0_std=[1.0, 0.3], sigma=dict(s0=[0.1] * 2, s1=[0.0] * 2, s2=[0.0] * 2))

    def run(enabled, samples, check, resume=False):
        with _ssm(w, precision) as s:
            s.surrogate_load(mlp_init(2, seed=1))
            if enabled:
                s.surrogate_enable(check_every=check, tol=1e9, mode="residual")
                s.surrogate_enable(check_every=0)
            s.step(1)
            if samples:
                s.surrogate_samples(512, seed=3)
            s.step(1)
            mid = s.state(0)
            if not resume:
                s.step(1)
                return s.state(0)
        with _ssm(w, precision) as s:
            s.surrogate_load(mlp_init(2, seed=1))
            if enabled:
                s.surrogate_enable(check_every=check, tol=1e9, mode="residual")
                s.surrogate_enable(check_every=0)
            s.set_state(0, mid, step=2)
            s.step(1)
            return s.state(0)

    pairs, grid = run(False, False, 1), run(True, False, 1)
    assert not np.array_equal(pairs, grid)
    assert np.array_equal(pairs, run(False, True, 1)) and np.array_equal(grid, run(True, True, 1))
    assert np.array_equal(grid, run(True, False, 16))
    assert np.array_equal(pairs, run(False, True, 1, resume=True)) and np.array_equal(grid, run(True, True, 1, resume=True))


def _rms_error(w, x0, x1, ell, targets=48):
    """RMS error of the step's pair term over its RMS, against sums in long double."""
    N = x0.shape[1]
    idx = np.linspace(0, N - 1, targets).astype(int)
    X = x0.astype(np.longdouble)
    err = ref = 0.0
    for i in idx:
        z = X - X[:, i:i + 1]
        K = (z * np.exp(-(z * z).sum(0) / (2 * np.longdouble(ell) ** 2))).sum(1) / N
        err += float((((x1[:, i].astype(np.longdouble) - X[:, i]) / H - K) ** 2).sum())
        ref += float((K * K).sum())
    return np.sqrt(err / ref)


@pytest.mark.parametrize("d,N", [(3, 20000), (3, 50021), (3, 262144), (3, 1048577), (2, 50021)])
def test_fp64_error_does_not_grow(torch_cuda, d, N):
    """FP64 at every size: 6e-16 by this arithmetic on the CPU (normal clouds, 2e4 to
    2^20), 1e-16 for x_1 and x_0 in the difference, 1e-15 allowed."""
    from paper_2105_09688_amd.ssm import mlp_init
    w = _w(N, (1.0, 1.0, 1.0))
    if d == 2:
        w.update(d=2, x0_mean=[0.0] * 2, x0_std=[1.0] * 2, sigma=dict(s0=[0.0] * 2, s1=[0.0] * 2, s2=[0.0] * 2))
    out = []
    for kw in ({}, dict(pair_scheme="symmetric")):
        if kw and N > 300000:
            break
        with _ssm(w, "fp64", **kw) as s:
            if d == 2:
                s.surrogate_load(mlp_init(2, seed=1))
                s.surrogate_enable(check_every=1, tol=1e9, mode="residual")
            x0 = s.state(0)
            s.step(1)
            out.append(_rms_error(w, x0, s.state(0), 0.5))
    print(f"[gpu-grid] d={d} N={N} FP64 relative RMS error: grid, pair kernels {['%.1e' % e for e in out]}", flush=True)
    assert out[0] <= 1e-15


def _contracted(kind, N):
    """Coordinates in which the grid's error, a fraction of Phi, is too large a part of K."""
    rng = np.random.default_rng(11)
    x = rng.normal(size=(3, N))
    if kind == "cluster":      # one cluster of 0.034 kernel widths (scaled)
        return 0.02 * x + np.array([[0.3], [-4.0], [1.0]])
    x *= 1e-3
    if kind == "two":          # two tight ones far apart
        x[0, N // 2:] += 5.0
    elif kind == "far":        # a tight one, and a few particles that make its spread large
        x[1, :1000] += 2.0
    elif kind == "near":       # two tight ones at the kernel's width: K is of its size
        x[2, : N // 2] += 0.5
    return x


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("kind,grid", [("cluster", False), ("two", False), ("far", False), ("near", True), ("normal", True)])
def test_contracted_clouds(torch_cuda, precision, kind, grid):
    """Bit for bit the pair kernels' where K is small against Phi, and not so elsewhere."""
    N = 32768
    w = _w(N, (1.0, 1.0, 1.0))
    out = []
    for kw in ({}, dict(pair_scheme="symmetric")):
        with _ssm(w, precision, **kw) as s:
            if kind != "normal":
                s.set_state(0, _contracted(kind, N), step=0)
            x0 = s.state(0)
            s.step(1)
            out.append(s.state(0))
    assert np.array_equal(*out) != grid


@pytest.mark.parametrize("std", [0.06, 0.12, 0.6])
def test_fp64_error_of_a_contracting_cloud(torch_cuda, std):
    """As test_fp64_error_does_not_grow: down to where the pair kernels take over 3e-16 by
    this arithmetic on the CPU."""
    with _ssm(_w(30000, (std,) * 3), "fp64") as s:
        x0 = s.state(0)
        s.step(1)
        err = _rms_error(s, x0, s.state(0), 0.5)
    print(f"[gpu-grid] std {std}: FP64 relative RMS error {err:.1e}", flush=True)
    assert err <= 1e-15
