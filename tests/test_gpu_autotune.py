"""The autotuner's choice against a context without a tiling: where that has a
faster way than the pair kernels the choice passes nothing to SSM, and a cache
entry that does not know the default's time is measured again."""
import json

import pytest

from paper_2105_09688_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    return torch


def test_no_tiling_is_a_candidate(tmp_path, monkeypatch):
    from paper_2105_09688_amd import tune
    path = tmp_path / "tune.json"
    monkeypatch.setenv("SSM_TUNE_CACHE", str(path))
    w = W.single_gpu_d1(N=32768)  # 12 us a tick by modes, 112 by the pair kernels
    path.write_text(json.dumps({tune._key(w, "fp32_kahan"): {"targets_per_lane": 4, "sources_per_item": 320,
                                                            "pair_scheme": "symmetric", "tick_ms": 0.1}}))
    c = tune.autotune(w, "fp32_kahan", steps=4)
    print(f"[gpu-autotune] {c}", flush=True)
    assert c["kwargs"] == {} and c["default_tick_ms"] < c["tiled_tick_ms"]
    assert c["targets_per_lane"] in (2, 4, 8) and tune.autotune(w, "fp32_kahan") == c


def test_a_tiling_is_passed_where_the_pair_kernels_run(tmp_path, monkeypatch):
    """Two dimensions without a surrogate: both run the pair kernels, so either choice is near the other."""
    from paper_2105_09688_amd import tune
    monkeypatch.setenv("SSM_TUNE_CACHE", str(tmp_path / "tune.json"))
    w = W.surrogate_d2(N=6000, h=2.0 ** -9, h_fine=2.0 ** -9)
    c = tune.autotune(w, "fp32_kahan", steps=8)
    print(f"[gpu-autotune] {c}", flush=True)
    assert c["kwargs"] == {} or c["kwargs"]["pair_scheme"] == c["pair_scheme"]
    assert min(c["default_tick_ms"], c["tiled_tick_ms"]) <= tune.tick_ms(w, "fp32_kahan", steps=8, **c["kwargs"]) * 1.5
