"""The addition passes on the GPU: output lists around the sizes where a run of
a thread, a workgroup's part and a pass end, against the oracle bit for bit."""
import numpy as np
import pytest

from gpu_util import assert_bitexact, run_gpu
from paper_2101_10881_amd import workloads as W

pytestmark = pytest.mark.gpu


# a part covers 16 runs of eight leaves up to eight doubles per coefficient, of
# four beyond; the value list has N + 1 leaves, variable 0's list N
@pytest.mark.parametrize("m,d,N", [(1, 0, 1), (2, 1, 7), (2, 15, 8), (4, 16, 9), (3, 17, 126), (1, 33, 127), (4, 8, 128),
                                   (5, 3, 129), (10, 2, 63), (10, 17, 64), (8, 16, 65), (10, 1, 64 * 64 + 2),
                                   (2, 2, 128 * 128 + 130)])
def test_list_sizes(oracle_lib, m, d, N):
    import torch
    from paper_2101_10881_amd import mdpe
    # variable 0 in every monomial, variable 1 in every third, variable 2 absent
    sup = [(0, 1) if k % 3 == 0 else (0,) for k in range(N)]
    w = W.make(f"lists_{m}_{d}_{N}", m, d, 3, sup, seed=N)
    # one launch per layer: tiny plans would run their additions in the single launch
    val, grad = run_gpu(w, poly=mdpe.Polynomial.for_workload(w, torch.device("cuda", 0), fused_layers=False))
    want_v, want_g = oracle_lib.eval_workload(w)
    assert_bitexact(val, want_v, "value")
    assert_bitexact(grad, want_g, "grad")
    assert not np.any(grad[:, 2])
