"""Plans of short chains stay within the allocation-free entry's workspace where
the plan without the chain launch does (no GPU needed)."""
import numpy as np

from paper_2101_10881_amd import mdpe, workloads as W

SCRATCH = 64 << 20


def test_short_chains_do_not_outgrow_the_scratch_workspace():
    rng = np.random.default_rng(5)
    sup = W.random_supports(rng, 31, 700, rng.integers(8, 14, size=700))

    def plan(d, flags=0):
        return mdpe.Plan.for_workload(W.make("sc", 2, d, 31, sup, seed=1), device=-1, flags=flags).info

    slots = plan(20, mdpe.MDPE_NO_CHAIN_LAUNCH)["n_series"]
    chained = plan(20)
    assert chained["chain_layers"] > 0 and chained["n_series"] > slots
    d = SCRATCH // (slots * 16) - 1  # the largest degree that fits without the fresh slots
    assert chained["n_series"] * (d + 1) * 16 > SCRATCH
    info = plan(d)
    assert info["workspace_bytes"] <= SCRATCH and info["chain_layers"] == 0
