"""Where the blocked convolutions change their terms per iteration (three to five
doubles: two below d = 24, four from there), also with second operands at the workspace's
end (common factors) and in the reverse pass; whole components as batch tasks; against the oracle bit for bit."""
import numpy as np
import pytest

from gpu_util import assert_bitexact, run_gpu
from paper_2101_10881_amd import workloads as W

pytestmark = pytest.mark.gpu


def _supports(n, N, lo, hi, seed):
    rng = np.random.default_rng(seed)
    return W.random_supports(rng, n, N, rng.integers(lo, hi + 1, size=N))


@pytest.mark.parametrize("m,d", [(3, 23), (3, 24), (3, 26), (4, 23), (4, 25), (4, 27), (5, 24), (5, 31), (5, 66)])
@pytest.mark.parametrize("emax,fused", [(1, False), (1, True), (3, False)])
def test_terms_per_iteration(oracle_lib, m, d, emax, fused):
    import torch
    from paper_2101_10881_amd import mdpe
    w = W.make(f"terms_{m}_{d}", m, d, 8, _supports(8, 33, 1, 5, d), seed=d + m)
    if emax > 1:
        w = W.with_exponents(w, emax, seed=d)
    P = mdpe.Polynomial.for_workload(w, torch.device("cuda", 0), fused_layers=fused)
    want_v, want_g = oracle_lib.eval_workload(w)
    got = run_gpu(w, poly=P)
    assert_bitexact(got[0], want_v, "value")
    assert_bitexact(got[1], want_g, "grad")


@pytest.mark.parametrize("m,d", [(3, 23), (3, 25), (4, 24), (4, 28), (5, 29)])
def test_reverse_pass_terms(oracle_lib, m, d):
    import torch
    from paper_2101_10881_amd import mdpe
    w = W.make("corr_terms", m, d, 8, _supports(8, 40, 1, 5, d), seed=d + 3)
    dev = torch.device("cuda", 0)
    P = mdpe.Polynomial.for_workload(w, dev, keep_monomials=True, fused_layers=False)
    value, grad = P.eval_and_diff(torch.from_numpy(w.coeff).to(dev), torch.from_numpy(w.z).to(dev))
    ybar = W.upstream_adjoint(m, d, 5)
    cbar, zbar = P.adjoint(torch.from_numpy(ybar).to(dev), grad)
    torch.cuda.synchronize()
    _, want_g = oracle_lib.eval_workload(w)
    assert_bitexact(grad.cpu().numpy(), want_g, "grad")
    want_c, want_z = oracle_lib.eval_adjoint(w.m, w.d, w.n, w.nvars, w.vars, w.z, want_g, ybar)
    assert_bitexact(cbar.cpu().numpy(), want_c, "coeff_bar")
    assert_bitexact(zbar.cpu().numpy(), want_z, "z_bar")


# 16 equal instances, two per queue, 2 x 140 components each: more than 256 on a
# queue, so whole components are the tasks
@pytest.mark.parametrize("m,d", [(2, 5), (3, 4), (3, 33), (4, 8), (5, 6)])
def test_batch_components_as_tasks(oracle_lib, m, d):
    import torch
    from paper_2101_10881_amd import mdpe
    dev = torch.device("cuda", 0)
    ws = [W.make(f"set{q}", m, d, 12, _supports(12, 140, 1, 6, q), seed=q + 1) for q in range(16)]
    B = mdpe.BatchedPolynomials(ws, dev)
    vs, gs = B.eval_and_diff([torch.from_numpy(w.coeff).to(dev) for w in ws], [torch.from_numpy(w.z).to(dev) for w in ws])
    B.batch.status()
    torch.cuda.synchronize()
    for q in (0, 7, 15):
        want_v, want_g = oracle_lib.eval_workload(ws[q])
        assert_bitexact(vs[q].cpu().numpy(), want_v, f"value {q}")
        assert_bitexact(gs[q].cpu().numpy(), want_g, f"grad {q}")
