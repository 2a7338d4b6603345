"""The chain launch, chosen by a plan itself, never takes a plan past the
allocation-free entry's workspace that fits without it: deep plans (power tables
and common factors, long chains) like shallow ones.  No GPU needed."""
import numpy as np
import pytest

from paper_2101_10881_amd import mdpe, workloads as W

SCRATCH = 64 << 20


# powers and common factors make 31 layers around chains of 12 products; one
# double per coefficient has chains of 21
@pytest.mark.parametrize("n,N,lo,hi,m,d,emax", [(30, 410, 4, 14, 4, 184, 8), (60, 2510, 8, 21, 1, 81, 1)])
def test_deep_plans_do_not_outgrow_the_scratch_workspace(n, N, lo, hi, m, d, emax):
    rng = np.random.default_rng(3)
    w = W.make("deep", m, d, n, W.random_supports(rng, n, N, rng.integers(lo, hi + 1, size=N)), seed=1)
    if emax > 1:
        rng, q = np.random.default_rng(7), len(w.vars)
        w.exps = np.where(rng.uniform(size=q) < 0.5, rng.integers(2, emax + 1, size=q), 1).astype(np.int32)

    def plan(flags=0):
        return mdpe.Plan.for_workload(w, device=-1, flags=flags).info

    without, asked, info = plan(mdpe.MDPE_NO_CHAIN_LAUNCH), plan(mdpe.MDPE_CHAIN_LAUNCH), plan()
    assert without["n_layers"] >= 16 and without["workspace_bytes"] <= SCRATCH
    assert asked["chain_layers"] > 0 and asked["workspace_bytes"] > SCRATCH  # asked for, it is made whatever it takes
    assert info["workspace_bytes"] <= SCRATCH
