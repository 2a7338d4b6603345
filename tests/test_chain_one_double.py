"""The chain launch at one double per coefficient and high degrees (no GPU needed)."""
import pytest

from paper_2101_10881_amd import mdpe, workloads as W


# p2 measured on MI355X: 200 to 224 us with the chain launch, 545 to 568 by layers
@pytest.mark.parametrize("d", [160, 161, 165, 176, 190])
def test_chain_launch_at_one_double_up_to_190(d):
    assert mdpe.Plan.for_workload(W.p2(m=1, d=d), device=-1).info["chain_layers"] > 0
