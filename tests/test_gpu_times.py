"""The profiler's categories: every addition counts as addition, also where one pass
makes them all and writes the outputs."""
import numpy as np
import pytest

from gpu_util import run_gpu
from paper_2101_10881_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,passes", [(20, 1), (200, 2)])
def test_addition_passes_count_as_additions(N, passes):
    import torch
    from paper_2101_10881_amd import mdpe
    rng = np.random.default_rng(2)
    w = W.make("times", 4, 40, 9, W.random_supports(rng, 9, N, rng.integers(2, 5, size=N)), seed=1)
    P = mdpe.Polynomial.for_workload(w, torch.device("cuda", 0), fused_layers=False)
    prof = mdpe.Profiler()
    run_gpu(w, profiler=prof, poly=P)
    t = prof.read()
    assert t["n_add"] == passes and t["add_ms"] > 0 and t["n_gather"] == 1
    assert t["gather_ms"] < t["add_ms"]


def test_without_additions_the_pass_is_the_gather():
    import torch
    from paper_2101_10881_amd import mdpe
    w = W.make("none", 2, 9, 3, [], seed=1)
    P = mdpe.Polynomial.for_workload(w, torch.device("cuda", 0), fused_layers=False)
    prof = mdpe.Profiler()
    run_gpu(w, profiler=prof, poly=P)
    t = prof.read()
    assert t["n_add"] == 0 and t["n_gather"] == 1 and t["gather_ms"] > 0
