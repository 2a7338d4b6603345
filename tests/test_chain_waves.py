"""Wavefronts per chain of the chain launch where workgroups of one or two spread
unevenly over a CU's SIMDs, and of long series at eight doubles (no GPU needed)."""
import numpy as np
import pytest

from paper_2101_10881_amd import mdpe, workloads as W


def _waves(n, N, lo, hi, m, d, emax=1, cx=False):
    rng = np.random.default_rng(11)
    w = W.make("waves", m, d, n, W.random_supports(rng, n, N, rng.integers(lo, hi + 1, size=N)), seed=1, cx=cx)
    if emax > 1:
        rng, q = np.random.default_rng(7), len(w.vars)
        w.exps = np.where(rng.uniform(size=q) < 0.5, rng.integers(2, emax + 1, size=q), 1).astype(np.int32)
    info = mdpe.Plan.for_workload(w, device=-1).info
    assert info["chain_layers"] > 0
    return info["chain_waves"]


# many long chains: four (measured 1781 us against 2575 on two, 740 against 1144)
@pytest.mark.parametrize("args", [(40, 261, 15, 15, 5, 130, 2), (45, 310, 19, 39, 4, 80), (41, 511, 23, 33, 5, 69)])
def test_many_long_chains_take_four_wavefronts(args):
    assert _waves(*args) >= 4


@pytest.mark.parametrize("args", [(51, 14, 23, 25, 8, 176), (50, 90, 27, 27, 4, 146, 1, True)])
def test_long_series_up_to_eight_doubles_take_eight_wavefronts(args):
    assert _waves(*args) == 8


# many chains of short series stay on one (216 us against 347 on two; 73 against 109)
@pytest.mark.parametrize("args", [(29, 286, 13, 13, 10, 10), (28, 759, 23, 23, 4, 6)])
def test_many_chains_of_short_series_take_one_wavefront(args):
    assert _waves(*args) == 1
