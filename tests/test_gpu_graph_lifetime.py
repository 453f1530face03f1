"""Network ticks replayed as graphs of several, with the surrogate enabled again
(its residuals dropped) while earlier replays may still be queued, and in a
context with tick graphs of its own (graphs = 1) whose first check starts the
grid: equal bit for bit to single ticks of a context that waits in between."""
import numpy as np
import pytest

from paper_2105_09688_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    return torch


@pytest.mark.parametrize("N,graphs", [(1500, False), (40000, False), (24000, True)])
def test_enabled_again_between_queued_replays(N, graphs):
    from paper_2105_09688_amd.ssm import SSM, mlp_init
    h = 2.0 ** -9
    w = W.surrogate_d2(N=N, h=h, h_fine=h)
    w["T"] = 800 * h

    def run(whole):
        with SSM(w, precision="fp32_kahan", persistent=-1, graphs=graphs) as s:
            s.surrogate_load(0.3 * mlp_init(2, seed=2))

            def go(n):
                for k in [n] if whole else [1] * n:
                    s.step(k)
                    if not whole:
                        s.sync()

            go(3)  # exact ticks
            s.surrogate_enable(check_every=48, tol=1e9, mode="residual")
            go(3 + 48 + 94)  # past 64 ticks; ends with replays that add residuals
            for _ in range(4):
                s.surrogate_enable(check_every=48, tol=1e9, mode="residual")  # without: until the next check
                go(40)
                go(56)
            return s.state(0), s.info()["surr_checks"]

    (a, ca), (b, cb) = run(True), run(False)
    print(f"[gpu-graph-lifetime] N={N} graphs={graphs}: {ca} checks", flush=True)
    assert ca == cb >= 10 and np.array_equal(a, b)
