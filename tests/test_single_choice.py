"""Which small plans take the single launch: those that it serves faster than the
launches that are made (a launch per layer and one or two addition passes).  No GPU
needed; both sides of each measured on MI355X."""
import numpy as np
import pytest

from paper_2101_10881_amd import mdpe, workloads as W


def _single(n, N, lo, hi, m, d):
    rng = np.random.default_rng(4)
    return mdpe.Plan.for_workload(W.make("s", m, d, n, W.random_supports(rng, n, N, rng.integers(lo, hi + 1, size=N)),
                                         seed=1), device=-1).info["single_launch"]


# one workgroup and launches per layer (us): 77 and 26, 51 and 19, 75 and 28, 40 and 17, 97 and 47
@pytest.mark.parametrize("args", [(3, 103, 3, 3, 5, 2), (12, 81, 2, 3, 3, 3), (11, 51, 1, 3, 3, 16), (12, 19, 2, 2, 2, 29),
                                  (14, 40, 2, 2, 10, 3)])
def test_many_additions_or_long_products_take_a_launch_per_layer(args):
    assert not _single(*args)


# 5.6 and 12.4, 8.3 and 24.1, 8.1 and 12.4, 12.4 and 19.0, 15 and 22
@pytest.mark.parametrize("args", [(3, 4, 1, 1, 2, 4), (7, 17, 2, 3, 1, 3), (14, 20, 1, 1, 2, 5), (8, 17, 3, 3, 2, 5),
                                  (8, 16, 3, 3, 2, 8)])
def test_the_smallest_take_one_workgroup(args):
    assert _single(*args)


def _kept(n, r, m, d, flags):
    return mdpe.Plan.for_workload(W.make("s", m, d, n, W.all_subsets(n, r), seed=1), device=-1,
                                  flags=flags).info["single_launch"]


# through autograd 107 and 122, 113 and 122, 114 and 122 us, alone 19 and 14, 24 and 15, 22 and 15
@pytest.mark.parametrize("args", [(16, 2, 1, 15), (15, 2, 1, 14), (13, 2, 2, 6)])
def test_a_plan_with_a_reverse_pass_takes_one_workgroup_for_fewer_launches(args):
    assert _kept(*args, mdpe.MDPE_KEEP_MONOMIAL_VALUES) and not _kept(*args, 0)


# 86 and 43, 119 and 38, 124 and 45 with the reverse pass
@pytest.mark.parametrize("args", [(8, 3, 2, 12), (10, 2, 2, 31), (14, 3, 1, 13)])
def test_but_not_where_the_device_is_what_takes_time(args):
    assert not _kept(*args, mdpe.MDPE_KEEP_MONOMIAL_VALUES)
