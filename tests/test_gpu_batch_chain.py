"""A batch of instances whose plans take the chain launch, by layers (eight doubles,
one instance dealt over the queues) and by component sets, against the oracle."""
import numpy as np
import pytest

from gpu_util import assert_bitexact
from paper_2101_10881_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,d,count", [(8, 9, 4), (1, 20, 9), (4, 12, 1), (3, 25, 16)])
def test_batch_of_chain_plans(oracle_lib, m, d, count):
    import torch
    from paper_2101_10881_amd import mdpe
    dev = torch.device("cuda", 0)
    ws = []
    for q in range(count):
        rng = np.random.default_rng(q)
        ws.append(W.make(f"bc{q}", m, d, 23, W.random_supports(rng, 23, 90, rng.integers(1, 13, size=90)), seed=q + 1))
    B = mdpe.BatchedPolynomials(ws, dev)
    assert all(P.plan.info["chain_layers"] > 0 for P in B.polys)
    vs, gs = B.eval_and_diff([torch.from_numpy(w.coeff).to(dev) for w in ws], [torch.from_numpy(w.z).to(dev) for w in ws])
    B.batch.status()
    torch.cuda.synchronize()
    for q in (0, count - 1):
        want_v, want_g = oracle_lib.eval_workload(ws[q])
        assert_bitexact(vs[q].cpu().numpy(), want_v, f"value {q}")
        assert_bitexact(gs[q].cpu().numpy(), want_g, f"grad {q}")
