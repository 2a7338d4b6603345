"""Which instances of a batch run whole components as tasks (no GPU needed): not
those whose longest component would outlast the rest of the queue, one product
after the other on one wavefront."""
import numpy as np
import pytest

from paper_2101_10881_amd import mdpe, workloads as W


def _plan(n, N, lo, hi, m, d, seed):
    rng = np.random.default_rng(seed)
    return mdpe.Plan.for_workload(W.make("b", m, d, n, W.random_supports(rng, n, N, rng.integers(lo, hi + 1, size=N)),
                                         seed=1), device=-1)


def _conv_tasks(plans):
    rows = mdpe.Batch(plans).tasks()
    return [int(np.sum((rows[:, 0] == p) & (rows[:, 1] == 1))) for p in range(len(plans))]


# a few deep, medium and long-series instances beside many small ones
@pytest.mark.parametrize("n,N,lo,hi,d", [(64, 4, 50, 60, 128), (64, 40, 8, 12, 128), (64, 40, 3, 3, 191)])
def test_long_components_among_small_instances_keep_their_layers(n, N, lo, hi, d):
    small = [_plan(20, 300, 2, 4, 4, 8, q) for q in range(120 if d < 191 else 60)]
    large = [_plan(n, N, lo, hi, 4, d, 1000 + q) for q in range(16)]
    tasks = _conv_tasks(small + large)
    for p in large:
        sizes, _ = p.layer_sizes()
        assert len(sizes) >= 3
    for q, p in enumerate(large):  # one job per group at these degrees: every layer of the monomials has its tasks
        assert tasks[len(small) + q] >= sum(-(-s // 2) for s in p.layer_sizes()[0])
    assert all(t <= 300 for t in tasks[: len(small)])  # the small ones: at most a task per component


@pytest.mark.parametrize("m", [2, 4])
def test_equal_instances_run_whole_components(m):
    plans = [_plan(23, 211, 1, 12, m, 37, q) for q in range(16)]
    assert all(t <= 422 for t in _conv_tasks(plans))
