"""The chain launch against the fused launch at one double per coefficient (no GPU needed)."""
import numpy as np
import pytest

from paper_2101_10881_amd import mdpe, workloads as W


def _info(n, N, lo, hi, d):
    rng = np.random.default_rng(6)
    return mdpe.Plan.for_workload(W.make("cf", 1, d, n, W.random_supports(rng, n, N, rng.integers(lo, hi + 1, size=N)),
                                         seed=1), device=-1).info


# measured on MI355X (us), fused and chain launch: 17.8 and 25.7, 22.8 and 28.0, 22.4 and 26.6
@pytest.mark.parametrize("args", [(9, 199, 2, 9, 3), (19, 6, 16, 16, 4), (53, 192, 13, 13, 5)])
def test_short_series_stay_fused(args):
    i = _info(*args)
    assert i["fused_components"] > 0 and i["chain_layers"] == 0


# 27.0 and 23.7, 35.1 and 24.4, 43.1 and 29.2
@pytest.mark.parametrize("args", [(13, 234, 8, 13, 12), (16, 40, 1, 11, 43), (31, 68, 27, 27, 11)])
def test_longer_series_take_the_chain_launch(args):
    assert _info(*args)["chain_layers"] > 0
