"""Long chains that pay take the chain launch even where its fresh slots pass the
allocation-free entry's workspace (no GPU needed)."""
import numpy as np

from paper_2101_10881_amd import mdpe, workloads as W

SCRATCH = 64 << 20


def test_long_chains_that_pay_outgrow_the_scratch_workspace():
    # measured on MI355X: 3080 us by layers, 1790 by the chain launch
    rng = np.random.default_rng(11)
    w = W.make("long", 5, 130, 40, W.random_supports(rng, 40, 261, rng.integers(15, 16, size=261)), seed=1)
    rng, q = np.random.default_rng(7), len(w.vars)
    w.exps = np.where(rng.uniform(size=q) < 0.5, 2, 1).astype(np.int32)
    info = mdpe.Plan.for_workload(w, device=-1).info
    without = mdpe.Plan.for_workload(w, device=-1, flags=mdpe.MDPE_NO_CHAIN_LAUNCH).info
    assert without["workspace_bytes"] <= SCRATCH < info["workspace_bytes"]
    assert info["chain_layers"] >= 16
