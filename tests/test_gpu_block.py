"""The blocked convolutions at the edges of their blocks, groups and schedules:
per-layer and fused launches (several terms per iteration, four coefficients per
lane at one double), the reverse pass and the chain launch, against the oracle
bit for bit."""
import numpy as np
import pytest

from gpu_util import assert_bitexact, run_gpu
from paper_2101_10881_amd import workloads as W

pytestmark = pytest.mark.gpu


def _poly(w, **kw):
    import torch
    from paper_2101_10881_amd import mdpe
    return mdpe.Polynomial.for_workload(w, torch.device("cuda", 0), **kw)


def _check(oracle_lib, w, **kw):
    want_v, want_g = oracle_lib.eval_workload(w)
    got = run_gpu(w, poly=_poly(w, **kw))
    assert_bitexact(got[0], want_v, "value")
    assert_bitexact(got[1], want_g, "grad")


def _supports(n, N, lo, hi, seed):
    rng = np.random.default_rng(seed)
    return W.random_supports(rng, n, N, rng.integers(lo, hi + 1, size=N))


# degrees around one and two blocks of two and four terms and 64 lanes; two
# doubles and one stage both operands; beyond five doubles blocks run up to d = 16
@pytest.mark.parametrize("m,d,cx", [(m, d, False) for m in (1, 2, 3, 5) for d in (0, 1, 2, 3, 4, 7, 63, 64, 65)] +
                         [(8, 1, False), (8, 16, False), (10, 15, False), (10, 16, False)] +
                         [(1, 2, True), (1, 64, True), (2, 5, True), (5, 9, True), (2, 66, True)])
@pytest.mark.parametrize("fused", [False, True])
def test_layer_and_fused_launches(oracle_lib, m, d, cx, fused):
    w = W.make(f"blk_{m}_{d}", m, d, 9, _supports(9, 37, 1, 6, d), seed=d + 1, cx=cx)
    _check(oracle_lib, w, fused_layers=fused)


# one double runs blocks, of four coefficients where that is cheapest, in layers
# of more than 6144 jobs
@pytest.mark.parametrize("d,n", [(128, 12), (131, 80), (3, 80), (10, 80), (67, 80)])
def test_four_coefficients_per_lane(oracle_lib, d, n):
    _check(oracle_lib, W.make("quad", 1, d, n, W.all_subsets(n, 2 if n > 20 else 3), seed=d), fused_layers=False)


@pytest.mark.parametrize("m,d", [(1, 129), (2, 0), (2, 3), (2, 17), (3, 1), (3, 34), (4, 63), (5, 32), (8, 15)])
def test_reverse_pass(oracle_lib, m, d):
    import torch
    w = W.make("corr", m, d, 8, _supports(8, 40, 1, 5, d), seed=d + 3)
    P = _poly(w, keep_monomials=True, fused_layers=False)
    dev = torch.device("cuda", 0)
    value, grad = P.eval_and_diff(torch.from_numpy(w.coeff).to(dev), torch.from_numpy(w.z).to(dev))
    ybar = W.upstream_adjoint(m, d, 5)
    cbar, zbar = P.adjoint(torch.from_numpy(ybar).to(dev), grad)
    torch.cuda.synchronize()
    _, want_g = oracle_lib.eval_workload(w)
    assert_bitexact(grad.cpu().numpy(), want_g, "grad")
    want_c, want_z = oracle_lib.eval_adjoint(w.m, w.d, w.n, w.nvars, w.vars, w.z, want_g, ybar)
    assert_bitexact(cbar.cpu().numpy(), want_c, "coeff_bar")
    assert_bitexact(zbar.cpu().numpy(), want_z, "z_bar")


# few and many chains (one and two wavefronts per chain from 64 chains on),
# chains longer than their LDS slots, chains of 9 to 12 products by default
@pytest.mark.parametrize("m,d,N,nk", [(1, 0, 3, 5), (1, 9, 40, 20), (1, 130, 4, 20), (2, 3, 40, 18), (2, 96, 5, 17),
                                      (3, 33, 130, 6), (4, 2, 70, 9), (4, 65, 6, 30), (5, 37, 60, 12), (8, 31, 4, 18),
                                      (10, 150, 2, 20), (10, 8, 3, 20)])
def test_chain_launch(oracle_lib, m, d, N, nk):
    n = max(nk, 24)
    w = W.make(f"chain_{m}_{d}", m, d, n, _supports(n, N, max(1, nk - 3), nk, d + nk), seed=d + nk)
    _check(oracle_lib, w, chain_launch=True)
    if nk <= 12:
        _check(oracle_lib, w)
