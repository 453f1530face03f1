"""The mode sums of the one-dimensional interaction (ssm_modes.hpp) on the
CPU: with the gap, the largest wavenumber and the constants of the kernel
source, the Fourier sum over a cloud's extent equals the sums over all pairs
to the error that the source states for each precision, for clouds of one
particle up to hundreds of kernel widths.

Tolerances: image and truncation errors are below 5e-18 (FP64) and 1e-11
(FP32 modes) per pair term, whose largest value is 0.52; the FP64 bound adds
the rounding of the phases, 2^-52 per radian of the largest one that carries
weight (wavenumber 4 in the scaled coordinate) and as much per mode for the
repeated rotation."""
import math
import os
import re

import numpy as np
import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2105_09688_amd", "csrc",
                   "ssm_modes.hpp")
ALPHA = math.log(2.0)


def _source():
    with open(SRC) as fh:
        s = fh.read()
    lim = re.search(r"fp64 \? ModeLimits\{([\d.]+), ([\d.]+)\} : ModeLimits\{([\d.]+), ([\d.]+)\}", s)
    c0 = float(re.search(r"delta \* ([\d.]+);\s*// 1 / sqrt\(4 pi a\)", s).group(1))
    e = float(re.search(r"exp2_fast<double>\(k \* k \* -([\d.]+)\)", s).group(1))
    ia = float(re.search(r"c0 \* \(k \* ([\d.]+)\)", s).group(1))
    return [float(x) for x in lim.groups()], c0, e, ia


def test_constants():
    _, c0, e, ia = _source()
    assert c0 == pytest.approx(1 / math.sqrt(4 * math.pi * ALPHA), rel=1e-15)
    assert e == pytest.approx(1 / (4 * ALPHA ** 2), rel=1e-15) and ia == pytest.approx(1 / ALPHA, rel=1e-15)


def test_limits_bound_images_and_truncation():
    (g64, k64, g32, k32), *_ = _source()
    for gap, kmax, bound in ((g64, k64, 5e-18), (g32, k32, 1e-11)):
        images = 2 * (gap * 2.0 ** -(gap * gap))
        tail = 2 / math.sqrt(4 * math.pi * ALPHA) * math.exp(-kmax * kmax / (4 * ALPHA))
        assert images <= 2 * bound and tail <= bound


def _modes(s, gap, kmax):
    _, c0, e, ia = _source()
    lo, hi = s.min(), s.max()
    c, L = 0.5 * (lo + hi), hi - lo + gap
    M = (int(math.ceil(kmax / (2 * math.pi) * L)) + 7) // 8 * 8
    delta = 2 * math.pi / L
    z = np.exp(2j * np.pi * ((s - c) * (1.0 / L)))
    w, g = z.copy(), []
    for m in range(1, M + 1):
        k = m * delta
        cm = delta * c0 * k * ia * 2.0 ** (-k * k * e)
        g.append(cm * (w.imag.sum() + 1j * w.real.sum()))
        w = w * z
    p = np.zeros_like(z)
    for gm in reversed(g):
        p = p * z + gm
    return (p * z).real, M


@pytest.mark.parametrize("N,scale", [(1, 0.0), (2, 3.0), (300, 0.05), (300, 0.5), (500, 2.0), (500, 12.0), (300, 100.0)])
def test_equals_the_sum_over_pairs(N, scale):
    s = np.random.default_rng(N).normal(size=N) * scale + 0.8
    z = s.astype(np.longdouble)[None] - s.astype(np.longdouble)[:, None]
    ref = (z * np.exp2(-z * z)).sum(1)
    (g64, k64, g32, k32), *_ = _source()
    for gap, kmax, eps in ((g64, k64, 5e-18), (g32, k32, 1e-11)):
        got, M = _modes(s, gap, kmax)
        ext = float(s.max() - s.min())
        tol = N * (3 * eps + 2.0 ** -52 * (4 * ext / 2 + M))
        assert float(np.abs(got - ref).max()) <= tol, (N, scale, gap, float(np.abs(got - ref).max()), tol)
