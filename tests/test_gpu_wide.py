"""The kernels of workspaces of 4 GiB and more (asked for on small ones) against the
oracle, and the blocked kernels on a workspace between 2 and 4 GiB, whose byte
offsets use the top bit, against those."""
import numpy as np
import pytest

from gpu_util import assert_bitexact
from paper_2101_10881_amd import workloads as W

pytestmark = pytest.mark.gpu


def _supports(n, N, lo, hi, seed):
    rng = np.random.default_rng(seed)
    return W.random_supports(rng, n, N, rng.integers(lo, hi + 1, size=N))


def _run(w, flags):
    import torch
    from paper_2101_10881_amd import mdpe
    dev = torch.device("cuda", 0)
    plan = mdpe.Plan.for_workload(w, 0, flags | mdpe.MDPE_WIDE_OFFSETS)
    lead = (2, w.m) if w.cx else (w.m,)
    value = torch.empty(lead + (w.d + 1,), dtype=torch.float64, device=dev)
    grad = torch.empty(lead + (w.n, w.d + 1), dtype=torch.float64, device=dev)
    ws = torch.empty(plan.info["workspace_bytes"] // 8, dtype=torch.float64, device=dev)
    mdpe.eval_and_diff(plan, torch.from_numpy(w.coeff).to(dev), torch.from_numpy(w.z).to(dev), value, grad, ws)
    torch.cuda.synchronize()
    return plan, value, grad, ws


def _check(oracle_lib, w, flags):
    plan, value, grad, ws = _run(w, flags)
    want_v, want_g = oracle_lib.eval_workload(w)
    assert_bitexact(value.cpu().numpy(), want_v, "value")
    assert_bitexact(grad.cpu().numpy(), want_g, "grad")
    return plan, grad, ws


@pytest.mark.parametrize("m,d,N,nk,cx", [(1, 40, 12, 17, False), (2, 33, 70, 10, False), (3, 9, 5, 20, False),
                                         (4, 65, 6, 18, False), (5, 12, 8, 17, False), (8, 7, 9, 18, False),
                                         (10, 20, 3, 20, False), (2, 18, 6, 17, True)])
def test_chain_launch(oracle_lib, m, d, N, nk, cx):
    from paper_2101_10881_amd import mdpe
    w = W.make("wc", m, d, 24, _supports(24, N, nk - 2, nk, d), seed=d, cx=cx)
    plan, _, _ = _check(oracle_lib, w, mdpe.MDPE_CHAIN_LAUNCH)
    assert plan.info["chain_layers"] > 0


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("m,d,cx", [(1, 63, False), (2, 4, False), (2, 64, False), (3, 30, False), (4, 7, False),
                                    (4, 66, False), (5, 33, False), (8, 9, False), (2, 20, True)])
def test_layer_and_fused_launches(oracle_lib, m, d, cx, fused):
    from paper_2101_10881_amd import mdpe
    w = W.make("wl", m, d, 9, _supports(9, 37, 1, 6, d), seed=d + 1, cx=cx)
    plan, _, _ = _check(oracle_lib, w, mdpe.MDPE_FUSED_LAYERS if fused else mdpe.MDPE_LAYER_LAUNCHES)
    assert (plan.info["fused_components"] > 0) == fused


@pytest.mark.parametrize("m,d", [(2, 17), (3, 34), (4, 24), (5, 8)])
def test_reverse_pass(oracle_lib, m, d):
    import torch
    from paper_2101_10881_amd import mdpe
    w = W.make("wr", m, d, 8, _supports(8, 40, 1, 5, d), seed=d + 3)
    plan, grad, ws = _check(oracle_lib, w, mdpe.MDPE_KEEP_MONOMIAL_VALUES | mdpe.MDPE_LAYER_LAUNCHES)
    ybar = W.upstream_adjoint(m, d, 5)
    cbar = torch.empty((m, w.N + 1, d + 1), dtype=torch.float64, device="cuda")
    zbar = torch.empty((m, w.n, d + 1), dtype=torch.float64, device="cuda")
    mdpe.eval_adjoint(plan, torch.from_numpy(ybar).to("cuda"), ws, grad, cbar, zbar)
    torch.cuda.synchronize()
    want_c, want_z = oracle_lib.eval_adjoint(w.m, w.d, w.n, w.nvars, w.vars, w.z, grad.cpu().numpy(), ybar)
    assert_bitexact(cbar.cpu().numpy(), want_c, "coeff_bar")
    assert_bitexact(zbar.cpu().numpy(), want_z, "z_bar")


@pytest.mark.parametrize("ms", [(2,), (3,), (4,), (5,), (2, 4)])
def test_batch(oracle_lib, ms):
    import torch
    from paper_2101_10881_amd import mdpe
    dev = torch.device("cuda", 0)
    ws = [W.make(f"wb{q}", ms[q % len(ms)], 11 + q, 9, _supports(9, 30, 1, 6, q), seed=q + 1) for q in range(10)]
    plans = [mdpe.Plan.for_workload(w, 0, mdpe.MDPE_WIDE_OFFSETS) for w in ws]
    B = mdpe.Batch(plans)
    c, z = [torch.from_numpy(w.coeff).to(dev) for w in ws], [torch.from_numpy(w.z).to(dev) for w in ws]
    v = [torch.empty((w.m, w.d + 1), dtype=torch.float64, device=dev) for w in ws]
    g = [torch.empty((w.m, w.n, w.d + 1), dtype=torch.float64, device=dev) for w in ws]
    B.eval_and_diff(c, z, v, g, torch.empty(B.info()["workspace_bytes"] // 8, dtype=torch.float64, device=dev))
    B.status()
    for q in (0, 1, 9):
        want_v, want_g = oracle_lib.eval_workload(ws[q])
        assert_bitexact(v[q].cpu().numpy(), want_v, f"value {q}")
        assert_bitexact(g[q].cpu().numpy(), want_g, f"grad {q}")


# 790000 products of two of three variables: 3.0 GiB, the products' slots from 0.75 on
@pytest.mark.parametrize("m,d", [(2, 63), (4, 31)])
def test_offsets_beyond_two_gib(m, d):
    import torch
    from paper_2101_10881_amd import mdpe
    dev = torch.device("cuda", 0)
    N = 790000
    vars_ = np.tile(np.array([0, 1, 0, 2, 1, 2], dtype=np.int32), N // 3 + 1)[: 2 * N]
    nvars = np.full(N, 2, dtype=np.int32)
    gen = torch.Generator(device=dev).manual_seed(m)
    coeff = torch.randn((m, N + 1, d + 1), dtype=torch.float64, device=dev, generator=gen)
    z = torch.randn((m, 3, d + 1), dtype=torch.float64, device=dev, generator=gen)
    out = []
    for flags in (0, mdpe.MDPE_WIDE_OFFSETS):
        plan = mdpe.Plan(3, nvars, vars_, d, m, 0, flags | mdpe.MDPE_LAYER_LAUNCHES)
        size = plan.info["workspace_bytes"]
        assert 2 << 30 < size < 4 << 30
        value = torch.empty((m, d + 1), dtype=torch.float64, device=dev)
        grad = torch.empty((m, 3, d + 1), dtype=torch.float64, device=dev)
        ws = torch.empty(size // 8, dtype=torch.float64, device=dev)
        mdpe.eval_and_diff(plan, coeff, z, value, grad, ws)
        torch.cuda.synchronize()
        out.append((value.cpu().numpy(), grad.cpu().numpy()))
        del plan, ws
    assert np.isfinite(out[1][0]).all() and np.any(out[1][0])
    assert_bitexact(out[0][0], out[1][0], "value")
    assert_bitexact(out[0][1], out[1][1], "grad")
