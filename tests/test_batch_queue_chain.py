"""Instances of one, eight or ten doubles whose plan takes the chain launch run their
products at the earliest layers in a batch (no GPU needed): as many stages as the longest monomial has
variables, every product once, after the products that it reads."""
import numpy as np
import pytest

from paper_2101_10881_amd import mdpe, workloads as W


@pytest.mark.parametrize("m,count", [(8, 16), (1, 16), (10, 1)])
def test_chain_plans_run_at_their_earliest_layers(m, count):
    plans = []
    for q in range(count):
        rng = np.random.default_rng(q)
        w = W.make("c", m, 37, 23, W.random_supports(rng, 23, 211, rng.integers(1, 13, size=211)), seed=1)
        plans.append(mdpe.Plan.for_workload(w, device=-1))
        assert plans[-1].info["chain_layers"] > 0
    rows = mdpe.Batch(plans).tasks()
    for p, plan in enumerate(plans):
        conv = rows[(rows[:, 0] == p) & (rows[:, 1] == 1)]
        assert conv[:, 3].sum() == plan.info["n_conv"]
        nv = int(plan.nvars.max())
        sizes = [conv[conv[:, 2] == need, 3].sum() for need in np.unique(conv[:, 2])]
        assert len(sizes) == nv < plan.info["n_layers"]
