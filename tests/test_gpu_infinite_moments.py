"""The implicit step where the second moment of mu^X is infinite or NaN (a
corrupted particle in a system whose v depends on that moment): the finite
particles' equation has the root 0 in the limit (alpha = 1 - h (rho - kappa m2)
infinite), no solve counts as failed, and the corrupted particle is what is
reported, as through the bracketed form alone.  Next to it the ordinary range
up to moments of 1e307, against the root in 60 digits."""
from decimal import Decimal, localcontext

import numpy as np
import pytest

from paper_2105_09688_amd import workloads as W

pytestmark = pytest.mark.gpu
X1 = np.array([1e-100, 1e-20, 0.3, 1.0, 7.0, 1e10, 1e100, 1e153])


@pytest.fixture(scope="module", autouse=True)
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    return torch


@pytest.mark.parametrize("d", [1, 2, 3])
def test_infinite_second_moment(torch_cuda, d):
    from paper_2105_09688_amd.ssm import implicit_solve
    x = np.concatenate([X1, -X1, [0.0, np.inf, np.nan]])
    X = np.stack([x] + [0.5 * x] * (d - 1))
    Y, it = implicit_solve(torch_cuda.tensor(X, device="cuda"), 2.0 ** -4, 0.0, 1.0, 0.5, 0.0, np.zeros(d), np.inf)
    Y, it = Y.cpu().numpy(), it.cpu().numpy()
    assert (Y[:, :17] == 0.0).all() and (it[:17] >= 0).all()
    assert (it[17:] == -2).all() and np.array_equal(Y[:, 17:], X[:, 17:], equal_nan=True)


def _root(x, alpha, ha):
    """s with ha s^3 + alpha s = x by Newton from the smaller upper bound, in 60 digits."""
    with localcontext() as c:
        c.prec = 60
        x, alpha, ha = Decimal(x), Decimal(alpha), Decimal(ha)
        s = min(x / alpha, (x / ha) ** (Decimal(1) / 3))
        for _ in range(60):
            s -= (ha * s ** 3 + alpha * s - x) / (3 * ha * s * s + alpha)
        return float(s)


@pytest.mark.parametrize("m2", [0.0, 1e10, 1e100, 1e300, 1e307])
def test_large_second_moments(torch_cuda, m2):
    from paper_2105_09688_amd.ssm import implicit_solve
    h, kappa = 2.0 ** -4, 0.5
    Y, it = implicit_solve(torch_cuda.tensor(X1[None], device="cuda"), h, 0.0, 1.0, kappa, 0.0, np.zeros(1), m2)
    ref = np.array([_root(x, 1.0 + h * kappa * m2, h) for x in X1])
    assert (it.cpu().numpy() >= 0).all()
    # a few roundings; roots below the normal numbers to one unit there
    assert np.allclose(Y.cpu().numpy()[0], ref, rtol=1e-13, atol=1e-307)


@pytest.mark.parametrize("bad", [np.inf, np.nan])
@pytest.mark.parametrize("persistent", [0, -1])
def test_context_reports_the_particle(bad, persistent):
    """One corrupted particle under v_kappa: non-finite particles are counted, no Newton failure."""
    from paper_2105_09688_amd import SSMError
    from paper_2105_09688_amd.ssm import SSM
    h = 2.0 ** -6
    w = W.with_systems(W.small_parity(n_ens=1, h=h, h_fine=h), [(500, 0, h), (500, 1, h)])
    w["v"] = dict(rho=-1.0, a=1.0, kappa=0.5, lam=0.0)
    w["b"]["g"] = 0.0
    with SSM(w, precision="fp64", persistent=persistent) as s:
        clean = s.state(1)
        x = s.state(0)
        x[0, 7] = bad
        with pytest.raises(SSMError):
            s.set_state(0, x)
        s.step(2)
        info = s.info()
        print(f"[gpu-infinite-moments] {bad} persistent={persistent}: {info['nonfinite']} {info['newton_failures']}", flush=True)
        assert info["nonfinite"] > 0 and info["newton_failures"] == 0
    assert np.isfinite(clean).all()
