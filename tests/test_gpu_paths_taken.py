"""That the paths other tests compare do run: steps of many ticks past a context's
64th leave as graph launches (a failed capture would fall back to the same
kernels one by one, and equal results would show nothing)."""
import pytest

from paper_2105_09688_amd import workloads as W

pytestmark = pytest.mark.gpu
H = 2.0 ** -9


@pytest.fixture(scope="module", autouse=True)
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    return torch


def _calls(torch, step):
    """Runtime calls by name during step()."""
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as p:
        step()
        torch.cuda.synchronize()
    n = {}
    for e in p.events():
        if e.name.startswith("hip"):
            n[e.name] = n.get(e.name, 0) + 1
    return n


@pytest.mark.parametrize("case", ["modes", "free", "network"])
def test_graph_launches(torch_cuda, case):
    from paper_2105_09688_amd.ssm import SSM, mlp_init
    w = (W.surrogate_d2(N=1500, h=H, h_fine=H) if case == "network" else
         W.with_systems(W.small_parity(n_ens=1, h=H, h_fine=H) if case == "modes" else W.ou(x0_std=0.5, h=H, h_fine=H),
                        [(3000, 0, H)]))
    w["T"] = 512 * H
    with SSM(w, precision="fp32_kahan", persistent=-1) as s:
        if case == "network":
            s.surrogate_load(mlp_init(2, seed=1))
            s.surrogate_enable(check_every=128, tol=1e9, mode="residual")
        s.step(80)
        s.sync()

        def go():
            s.step(16)
            s.sync()

        go()  # captures it
        calls = _calls(torch_cuda, go)
        print(f"[gpu-paths] {case}: {calls}", flush=True)
        assert calls.get("hipGraphLaunch", 0) >= 1
        assert calls.get("hipLaunchKernel", 0) + calls.get("hipExtLaunchKernel", 0) + calls.get("hipModuleLaunchKernel", 0) <= 4
