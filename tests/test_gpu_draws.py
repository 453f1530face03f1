"""Brownian increments of large systems, around the counts from which fewer
lanes share a particle's draws, and gradients of batches of every remainder of
the weight-gradient kernel's chunks.

Tolerances: FP64 increments as in the parity tests (1e-13 over a step); a
gradient against the oracle's in 64 bits 2e-2 of each tensor's norm, as in the
surrogate's tests (BF16 operands); a chunk of 64 rows left out of the largest
batch would be 17 %."""
import numpy as np
import pytest

import oracle
from test_gpu_surrogate import D, IN, IN_NET, _expand, _kernel_params
from paper_2105_09688_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    return torch


@pytest.mark.parametrize("N", [2 ** 15, 2 ** 16 + 1, 2 ** 17 + 1, 2 ** 18 + 1, 2 ** 19 + 1])
def test_increments_of_large_systems(N):
    from paper_2105_09688_amd.ssm import SSM
    h = 2.0 ** -6
    w = W.with_systems(W.ou(x0_std=0.5, h=h, h_fine=h / 64), [(N, 0, h)])
    w["T"] = 2 * h
    at = np.unique(np.concatenate([[0, 63, 64, 255, 256, N - 1], np.linspace(0, N - 1, 200).astype(int)]))
    ref = oracle.step_at(w, 0, h, 0, oracle.init_state(w, 0, N), at)
    print(f"[gpu-draws] N={N}", flush=True)
    with SSM(w, precision="fp64") as s:
        s.step(1)
        assert np.max(np.abs(s.state(0)[:, at] - ref)) <= 1e-13


@pytest.mark.parametrize("precision", ["fp64", "fp32_kahan"])
@pytest.mark.parametrize("kind", ["free", "mean", "two sizes"])
def test_many_ticks_of_a_call_equal_single_ones(kind, precision):
    """Without a pair term a call's ticks leave as graphs too, past a context's first 64."""
    from paper_2105_09688_amd.ssm import SSM
    h = 2.0 ** -7
    w = W.ginzburg_landau(version=2, h_fine=h / 4) if kind == "mean" else W.ou(x0_std=0.5, h=h, h_fine=h / 4)
    w = W.with_systems(w, [(2500, 0, h), (3001, 1, 2 * h if kind == "two sizes" else h)])
    w["T"] = 128 * h
    out = []
    for plan in ((70, 31, 27), (1,) * 128):
        with SSM(w, precision=precision) as s:
            for n in plan:
                s.step(n)
            out.append(s.states())
    assert all(np.array_equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("rows", [64, 128, 512, 576, 1088, 2112])
def test_gradients_of_every_remainder(torch_cuda, rows):
    from paper_2105_09688_amd.ssm import mlp_init, mlp_loss_grad
    torch = torch_cuda
    rng = np.random.default_rng(rows)
    p = mlp_init(D, seed=3)
    p += rng.normal(size=p.size).astype(np.float32) * 0.05
    U = rng.normal(size=(rows, IN)).astype(np.float32)
    T = rng.normal(size=(rows, D)).astype(np.float32) * 0.3
    print(f"[gpu-draws] gradient of {rows} rows", flush=True)
    loss, g = mlp_loss_grad(D, torch.tensor(p, device="cuda"), torch.tensor(U, device="cuda"), torch.tensor(T, device="cuda"))
    g = g.cpu().numpy().astype(np.float64)
    loss_ref, g_ref = oracle.mlp_loss_grad(_kernel_params(p), _expand(U), T.astype(np.float64), IN_NET, 64, D)
    assert loss == pytest.approx(loss_ref, rel=1e-2)
    off = 0
    for k, n in enumerate([64 * IN_NET, 64, 64 * 64, 64, 64 * 64, 64, D * 64, D]):
        a, b = g[off:off + n], g_ref[off:off + n]
        assert np.linalg.norm(a - b) <= 2e-2 * np.linalg.norm(b), k
        off += n
